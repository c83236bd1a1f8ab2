"""The prompt pass's tiles that are cut to the prompt's rows: their rules without a GPU, and the lengths at which a rule or its number of row
tiles changes against the float64 model of test_gpu_prefill_tiles.py (whose bars these are)."""
import os
import subprocess

import pytest

import test_gpu_prefill_tiles as tiles

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "la_prefill_plan.h"
using namespace la;
int main(int, char **v) {  // d, q columns, k and v columns, ffn, compute units
  const int d = atoi(v[1]), qd = atoi(v[2]), kvd = atoi(v[3]), F = atoi(v[4]), cus = atoi(v[5]);
  for (int M = 1; M <= 2048; ++M) {
    const int RT = (M + 63) / 64 * 4, part_rows = pf_layout(PfDims{(size_t)d, (size_t)qd, 128, (size_t)F}, M < PF_LONG ? PF_LONG : PF_ROWS).part_rows;
    int So = 0, Sd = 0;
    const int q = pf_qkv_rows(PfProduct{RT, M, d / 32, (qd + 2 * kvd) / 16, d}, cus);
    const int o = pf_part_rows(PfProduct{RT, M, qd / 32, d / 16, d}, part_rows, cus, So), w = pf_part_rows(PfProduct{RT, M, F / 32, d / 16, d}, part_rows, cus, Sd);
    printf("%d %d %d %d %d %d %d %d\n", M, q, o, So, w, Sd, pf_gateup_rows(PfProduct{RT, M, d / 32, 2 * F / 16, d}, cus), part_rows);
  }
}
"""


@pytest.fixture(scope="module")
def rows(tmp_path_factory):
    d = tmp_path_factory.mktemp("rows")
    (d / "rows.cpp").write_text(PROGRAM)
    exe = str(d / "rows")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2602_16760_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
                    str(d / "rows.cpp"), "-o", exe], check=True)
    return lambda *a: [[int(x) for x in line.split()] for line in
                       subprocess.run([exe, *map(str, a)], check=True, capture_output=True, text=True).stdout.splitlines()]


@pytest.mark.parametrize("dims,cus", [((4096, 4096, 1024, 14336), 256), ((5120, 4096, 1024, 14336), 256), ((4096, 4096, 4096, 14336), 256),
                                      ((4096, 4096, 1024, 14336), 64), ((512, 1024, 256, 1408), 256), ((384, 384, 128, 1056), 256)])
def test_rules_stay_within_their_kernels_and_buffers(rows, dims, cus):
    d, qd, kvd, F = dims
    up = lambda a, b: -(-a // b)
    for M, q, o, So, w, Sd, g, part_rows in rows(*dims, cus):
        rt = up(M, 16)
        assert q in (0, 3, 4, 5, 6, 7, 8) and (not q or (128 < M <= 512 and up(rt, q) <= 4 and up(rt, q) * up((qd + 2 * kvd) // 16, 6) <= cus))
        for r, S, K in ((o, So, qd), (w, Sd, F)):
            if r:  # every row in one workgroup's tile, each slice's products in the buffer, a slice of four k-tiles or more
                assert 64 < M <= 128 and r == rt and 1 <= S <= 8 and S * M <= part_rows and (S == 1 or K // 32 // S >= 4) and up(d // 16, 8) * S <= cus
        assert g in ((0, rt) if M <= 128 else (0, 10, 12))
        if M <= 64:
            assert (q, o, w, g) == (0, 0, 0, 0)


# Widths at which a rule's line lies, with what is faster on each side of it (the figures are beside the rules): d, q columns, k and v columns, ffn
def test_gate_up_is_cut_where_the_smallest_tiles_are_more_than_the_chip(rows):
    for F, cut in ((8192, False), (8704, True), (14336, True)):
        for d in (2048, 3072, 4096, 6144):
            for M, *_, g, _ in rows(d, d, 1024, F, 256):
                if 64 < M <= 128:
                    assert g == (-(-M // 16) if cut else 0), (d, F, M)


def test_o_and_down_are_cut_where_the_smallest_tiles_are_not_taken(rows):
    for (d, qd, F), at in (((4096, 4096, 8192), [(77, 8, 8), (90, 0, 7), (128, 0, 7)]), ((5120, 4096, 14336), [(97, 6, 6), (112, 0, 6)]), ((3072, 3072, 8192), [(70, 0, 8), (96, 0, 0), (128, 0, 0)])):
        t = {M: (So if o else 0, Sd if w else 0) for M, _, o, So, w, Sd, _, _ in rows(d, qd, 1024, F, 256)}
        for M, So, Sd in at:  # slices, 0: not cut
            assert t[M] == (So, Sd), (d, M)


def test_narrow_qkv_is_cut_beyond_256_rows_only_where_the_contraction_is_short(rows):
    last = {64: 320, 128: 256, 32: 384, 16: 384}  # k-tiles: the last length that is cut (the last layer's K and V, all of a narrow model's QKV)
    for KT, end in last.items():
        for M, q, *_ in rows(32 * KT, 0, 1024, 32 * KT, 256):
            assert (q != 0) == (128 < M <= end), (KT, M)
    # more columns than one round of the smallest tiles
    assert all((q != 0) == (128 < M <= 512) for M, q, *_ in rows(4096, 4096, 1024, 14336, 256))


# 7B and 12B widths: QKV by 3 .. 8 row tiles (first and last length of each), gate/up by 10 and 12, one row into a row tile and a full one
SIZES = [("mistral7b", "bf16", [(66, 1), (96, 0), (112, 33), (129, 0), (192, 5), (256, 0), (320, 64), (321, 0), (384, 7), (385, 0), (448, 1), (449, 0), (512, 31), (640, 0)]),
         ("mistral7b", "f16", [(80, 0), (310, 3)]),
         ("nemo12b", "bf16", [(65, 0), (128, 0), (133, 0), (500, 9)])]


@pytest.mark.gpu
@pytest.mark.parametrize("name,dtype,cases", SIZES)
def test_prompt_lengths_at_the_edges_of_the_rules(name, dtype, cases):
    tiles.test_prompt_pass_sizes(name, dtype, cases)


def test_the_lengths_above_reach_every_kernel_of_the_rules(rows):
    want, have = set(), set()
    for name, dtype, cases in SIZES:
        sh = tiles.shape_of(name, dtype)
        for M, q, o, So, w, Sd, g, _ in rows(sh.d_model, sh.q_dim, sh.kv_dim, sh.d_ffn, 256):
            used = {("qkv", q), ("part", o), ("part", w), ("gateup", g)}
            want |= used
            if M in {n for n, _ in cases}:
                have |= used
    assert want == have and len(want) == 7 + 5 + 7
