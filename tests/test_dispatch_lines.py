"""Which kernel a call takes, on both sides of each line (no GPU: the rules of lf_common.h, compiled for the CPU)."""
import shutil
import subprocess

import pytest

from paper_2602_04789_amd import build as B

MAIN = r"""
#include <stdio.h>
#include <string.h>
#include "lf_common.h"
int main() {
  char rule[16];
  int a, b, c, d, e;
  while (scanf("%15s %d %d %d %d %d", rule, &a, &b, &c, &d, &e) == 6) {
    int out = -1;
    if (!strcmp(rule, "kv")) out = (int)lf_kv_form_of(a, b, c, d, e);
    printf("%d\n", out);
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("g++ not found")
    d = tmp_path_factory.mktemp("lines")
    (d / "lines.cpp").write_text(MAIN)
    subprocess.run([gxx, "-std=c++17", "-I", f"{B.ROOT}/include", "-I", B.CSRC, str(d / "lines.cpp"), "-o", str(d / "lines")], check=True)

    def ask(rule, *numbers):
        numbers = numbers + (0,) * (5 - len(numbers))
        out = subprocess.run([str(d / "lines")], input=" ".join(map(str, (rule,) + numbers)), check=True, stdout=subprocess.PIPE, text=True).stdout
        return int(out)
    return ask


HALVES, GROUPS, BLOCK, WIDE = range(4)


# d, (head, KV block) pairs, list length, query and KV blocks of a head
@pytest.mark.parametrize("call,form", [
    ((64, 256, 64, 64, 64), HALVES), ((64, 352, 70, 70, 88), HALVES), ((64, 353, 70, 70, 88), BLOCK), ((64, 3000, 5, 75, 75), BLOCK),
    # past 256 blocks: lists of a few query blocks each that hold at least half of all
    ((64, 333, 3, 3, 3), BLOCK), ((64, 256, 3, 3, 3), HALVES), ((64, 318, 3, 3, 6), BLOCK), ((64, 300, 4, 10, 10), HALVES), ((64, 300, 5, 8, 10), BLOCK),
    ((64, 300, 5, 9, 10), HALVES),
    # d = 128: long lists of few blocks go to the kernel with one wavefront per SIMD
    ((128, 128, 48, 128, 128), WIDE), ((128, 128, 47, 128, 128), HALVES), ((128, 64, 64, 64, 64), WIDE), ((128, 129, 17, 43, 43), GROUPS),
    ((128, 129, 18, 43, 43), WIDE), ((128, 256, 17, 64, 64), GROUPS), ((128, 257, 17, 257, 257), BLOCK), ((128, 512, 18, 64, 64), WIDE),
    ((128, 513, 14, 57, 57), BLOCK), ((128, 513, 15, 57, 57), WIDE), ((128, 6300, 188, 75, 525), WIDE), ((128, 6300, 100, 75, 525), BLOCK)])
def test_the_form_of_dk_and_dv(ask, call, form):
    assert ask("kv", *call) == form
