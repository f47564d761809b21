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
    if (!strcmp(rule, "attn")) out = (int)lf_attn_form(a, b, c, d);
    if (!strcmp(rule, "dq")) out = (int)lf_dq_form(a, b, c);
    if (!strcmp(rule, "apart")) out = (int)lf_full_rounds_apart(a, b, c);
    if (!strcmp(rule, "four")) {             // the last call that divides lists in four, of all up to 1 536 blocks and lists of 1 200
      for (int n_k = 1; n_k <= 1200; n_k += 109)
        for (int blocks = 1; blocks <= 1536; ++blocks)
          for (int len = 1; len <= n_k; ++len) {
            if (lf_attn_form(a, blocks, len, n_k) == LF_FORM_FOUR && blocks > out) out = blocks;
            if (lf_dq_form(a, blocks, len) == LF_FORM_FOUR && blocks > out) out = blocks;
          }
    }
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
    ((64, 351, 7, 9, 9), BLOCK), ((64, 351, 9, 9, 9), HALVES), ((64, 320, 7, 10, 10), HALVES), ((64, 320, 8, 10, 10), BLOCK),
    # d = 128: long lists of few blocks go to the kernel with one wavefront per SIMD
    ((128, 128, 48, 128, 128), WIDE), ((128, 128, 47, 128, 128), HALVES), ((128, 64, 64, 64, 64), WIDE), ((128, 129, 17, 43, 43), GROUPS),
    ((128, 129, 18, 43, 43), WIDE), ((128, 256, 17, 64, 64), GROUPS), ((128, 257, 17, 257, 257), BLOCK), ((128, 512, 18, 64, 64), WIDE),
    ((128, 513, 14, 57, 57), BLOCK), ((128, 513, 15, 57, 57), WIDE), ((128, 6300, 188, 75, 525), WIDE), ((128, 6300, 100, 75, 525), BLOCK)])
def test_the_form_of_dk_and_dv(ask, call, form):
    assert ask("kv", *call) == form


ROWS, TWO, FOUR, ONE, PAIR = range(5)      # row halves, lists in two, in four, a wavefront a block, a pair of wavefronts a block


# d, query blocks, list length
@pytest.mark.parametrize("d,blocks,length,form", [
    (128, 1, 1, PAIR), (128, 1, 2, ROWS), (128, 128, 188, ROWS), (128, 129, 1, PAIR), (128, 129, 2, TWO), (128, 256, 14, TWO), (128, 256, 15, FOUR),
    (128, 257, 7, PAIR), (128, 257, 8, TWO), (128, 448, 8, TWO), (128, 449, 15, PAIR), (128, 512, 16, TWO), (128, 512, 188, TWO), (128, 513, 15, PAIR),
    (128, 513, 16, ONE), (128, 1024, 16, ONE), (128, 1025, 188, PAIR), (128, 1536, 188, PAIR), (128, 1537, 16, ONE), (128, 3000, 188, ONE),
    (64, 128, 1, PAIR), (64, 128, 2, TWO), (64, 128, 3, ROWS), (64, 129, 10, TWO), (64, 256, 11, FOUR), (64, 257, 5, PAIR), (64, 257, 6, TWO), (64, 512, 200, TWO),
    (64, 513, 1, PAIR), (64, 513, 2, TWO), (64, 768, 200, TWO), (64, 769, 200, PAIR)])
def test_the_form_of_the_attention(ask, d, blocks, length, form):
    assert ask("attn", d, blocks, length, 525) == form


@pytest.mark.parametrize("d,blocks,length,form", [
    (128, 128, 3, PAIR), (128, 128, 4, ROWS), (128, 129, 4, TWO), (128, 256, 14, TWO), (128, 256, 15, FOUR), (128, 257, 7, PAIR), (128, 512, 8, TWO),
    (128, 512, 300, TWO), (128, 513, 7, PAIR), (128, 513, 8, ONE), (128, 1024, 188, ONE), (128, 1280, 188, PAIR), (128, 1281, 188, ONE),
    (128, 2048, 8, ONE), (128, 2096, 8, PAIR), (128, 2097, 8, ONE), (64, 128, 3, PAIR), (64, 128, 5, TWO), (64, 128, 6, ROWS), (64, 256, 4, TWO), (64, 256, 15, FOUR),
    (64, 257, 9, PAIR), (64, 512, 10, TWO), (64, 513, 188, PAIR)])
def test_the_form_of_dq(ask, d, blocks, length, form):
    assert ask("dq", d, blocks, length) == form


@pytest.mark.parametrize("call,apart", [((128, 1024, 188), 0), ((128, 1025, 16), 1), ((128, 1025, 15), 0), ((128, 1280, 16), 1), ((128, 1281, 31), 0),
                                        ((128, 1281, 32), 1), ((128, 1472, 32), 1), ((128, 1473, 188), 0), ((128, 2049, 188), 1), ((64, 1025, 188), 0)])
def test_full_rounds_apart(ask, call, apart):
    assert ask("apart", *call) == apart


@pytest.mark.parametrize("d", [64, 128])
def test_lists_are_divided_in_four_up_to_256_blocks(ask, d):
    assert ask("four", d) == 256
