"""Which form lf_sparse_attn_split takes (no GPU: the rule and the validation in front of it, compiled for the CPU)."""
import shutil
import subprocess

import pytest

from paper_2602_04789_amd import build as B

MAIN = r"""
#include <stdio.h>
#include <string.h>
#include "lf_common.h"
LAUNCHERS
int main(int argc, char** argv) {
  int d, heads, n, f, hist, keep;
  while (scanf("%d %d %d %d %d %d", &d, &heads, &n, &f, &hist, &keep) == 6) {
    lf_shape h;
    memset(&h, 0, sizeof(h));
    h.heads = heads; h.head_dim = d; h.frame_len = n; h.block = 64; h.q_len = f * n; h.kv_len = (hist + f) * n;
    h.q_stride_tok = h.k_stride_tok = h.v_stride_tok = h.o_stride_tok = d;
    lf_budget b;
    memset(&b, 0, sizeof(b));
    b.n_hist_frames = hist; b.frames_per_chunk = f; b.k_frames = hist; b.k_blocks = keep; b.current_mandatory = 1;
    b.list_len = keep + f * ((n + 63) / 64);
    lf_dims m;
    if (lf_derive(&h, &b, &m) != LF_OK) return 1;
    printf("%d\n", (int)lf_two_phases(m));
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def two_phases(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("g++ not found")
    d = tmp_path_factory.mktemp("line")
    with open(f"{B.ROOT}/tests/host_sanitize_driver.cpp") as f:
        driver = f.read()
    launchers = driver[driver.index("static int g_launches"): driver.index("static int g_fail")]
    (d / "line.cpp").write_text(MAIN.replace("LAUNCHERS", launchers))
    subprocess.run([gxx, "-std=c++17", "-O1", "-I", f"{B.ROOT}/include", "-I", B.CSRC, f"{B.CSRC}/lf_host.cpp", str(d / "line.cpp"),
                    "-o", str(d / "line")], check=True)

    def ask(*call):
        out = subprocess.run([str(d / "line")], input=" ".join(map(str, call)), check=True, stdout=subprocess.PIPE, text=True).stdout
        return out.strip() == "1"
    return ask


# d, heads, frame length, frames in the chunk, frames before it, retrieved blocks
@pytest.mark.parametrize("call,expected", [
    # frames that leave much of their blocks empty, in large calls: 1.2 to 2.3 times as fast in two phases
    ((128, 5, 97, 150, 30, 30), True), ((64, 5, 97, 150, 30, 30), True), ((64, 40, 200, 12, 40, 30), True), ((128, 60, 200, 12, 40, 30), True),
    ((64, 60, 33, 60, 40, 30), True), ((128, 60, 33, 60, 40, 30), True), ((128, 44, 65, 30, 40, 60), True),
    # whole frames and frames of 1 560: one pass, whatever the number of blocks
    ((128, 5, 64, 225, 70, 60), False), ((128, 8, 64, 300, 70, 60), False), ((64, 20, 64, 225, 70, 60), False), ((128, 40, 1560, 3, 18, 150), False),
    ((128, 12, 1560, 3, 9, 90), False), ((64, 24, 1560, 9, 9, 90), False),
    # few query blocks, and short chunks whose saving is less than the state costs
    ((128, 2, 33, 60, 40, 30), False), ((64, 2, 65, 60, 40, 30), False), ((64, 200, 97, 4, 40, 30), False), ((128, 200, 200, 2, 40, 100), False)])
def test_two_phases_where_padding_costs_more_than_the_state(two_phases, call, expected):
    assert two_phases(*call) is expected
