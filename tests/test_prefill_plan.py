"""The prompt pass's host decisions (la_prefill_plan.h, plain C++): a small program prints them, checked here without a GPU."""
import os
import subprocess

import pytest

from test_gpu_prefill_tiles import SIZES, shape_of

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_16760_amd", "csrc")
SHAPES = {"7b": (4096, 4096, 128, 14336), "12b": (5120, 4096, 128, 14336), "small64": (384, 384, 64, 1056)}  # d, Hq dh, dh, F

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <initializer_list>
#include "la_prefill_plan.h"
using namespace la;
static void show(const PfLayout &l) {
  printf("%d %d %zu %zu %zu %zu %zu %zu %zu %zu %zu\n", l.rows, l.part_rows, l.x, l.part, l.ss, l.cs, l.A, l.Q, l.attn, l.act, l.total);
}
int main(int, char **v) {
  const auto num = [&](int i) { return (size_t)atoll(v[i]); };
  if (!strcmp(v[1], "layout")) show(pf_layout(PfDims{num(2), num(3), num(4), num(5)}, (int)num(6)));
  if (!strcmp(v[1], "fit"))
    show(pf_fit(PfDims{num(2), num(3), num(4), num(5)}, PF_ROWS, PF_LONG, [&](size_t bytes) { return bytes <= num(6); }));
  if (!strcmp(v[1], "routes")) {  // the products of every layer, then of the last one (its K and V columns): prompt lengths v[6] .. v[7]
    const int d = (int)num(2), qd = (int)num(3), kvd = (int)num(4), F = (int)num(5);
    for (int n = (int)num(6); n <= (int)num(7); ++n) {
      const int rows = n < PF_LONG ? PF_LONG : PF_ROWS, part_rows = pf_layout(PfDims{(size_t)d, (size_t)qd, 128, (size_t)F}, rows).part_rows;
      for (int done = 0; done < n; done += rows) {
        const int M = n - done < rows ? n - done : rows, RT = (M + 63) / 64 * 4;
        int tile = 0, S = 0;
        for (int cols : {qd + 2 * kvd, 2 * kvd}) {
          pf_choose(PfProduct{RT, M, d / 32, cols / 16, d}, 1, part_rows, 256, tile, S);
          if (pf_qkv_few(M, cols / 16, 256)) printf("0 %d %d %d\n", n, 100 + (M + 15) / 16, 1);
          else printf("0 %d %d %d\n", n, tile, S);
        }
        pf_choose(PfProduct{RT, M, d / 32, 2 * F / 16, d}, 1, part_rows, 256, tile, S);
        printf("2 %d %d %d\n", n, tile, S);
        for (int K : {qd, F}) {
          pf_choose(PfProduct{RT, M, K / 32, d / 16, d}, PF_MAX_SPLIT, part_rows, 256, tile, S);
          printf("1 %d %d %d\n", n, tile, S);
        }
      }
    }
  }
  if (!strcmp(v[1], "few")) printf("%d\n", pf_qkv_few((int)num(2), (int)num(3), (int)num(4)) ? 1 : 0);
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(PROGRAM)
    exe = str(d / "plan")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, "-I", os.path.join(ROOT, "include"), str(d / "plan.cpp"), "-o", exe], check=True)
    return lambda *a: [[int(x) for x in line.split()] for line in
                       subprocess.run([exe, *map(str, a)], check=True, capture_output=True, text=True).stdout.splitlines()]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("rows", [128, 256, 512, 1024, 2048])
def test_buffers_hold_every_chunk_and_do_not_overlap(plan, shape, rows):
    d, qd, dh, F = SHAPES[shape]
    r, part_rows, *at, total = plan("layout", d, qd, dh, F, rows)[0]
    assert r == rows and part_rows >= rows
    sizes = [4 * rows * d, 4 * part_rows * d, 4 * rows * 32, 4 * rows * dh, 2 * rows * d, 2 * rows * qd, 2 * rows * qd, 2 * rows * F]
    for a, size, end in zip(at, sizes, at[1:] + [total]):
        assert a % 1024 == 0 and a + size <= end


def test_a_short_prompt_takes_a_short_prompts_buffers(plan):
    total = plan("layout", *SHAPES["7b"], 128)[0][-1]
    assert total <= 128 * (4096 * 38 + 14336 * 2 + 4096 * 4 + 4 * 32 + 4 * 128) + 8 * 1024
    assert total < 27e6 < 200e6 < plan("layout", *SHAPES["7b"], 2048)[0][-1]


def test_buffers_shrink_to_the_memory_that_is_left(plan):
    sizes = {rows: plan("layout", *SHAPES["7b"], rows)[0][-1] for rows in (128, 256, 512, 1024, 2048)}
    for rows, size in sizes.items():
        assert plan("fit", *SHAPES["7b"], size)[0][0] == rows
        assert plan("fit", *SHAPES["7b"], size - 1)[0][0] == (rows // 2 if rows > 128 else 0)
    # what a chunk of 1024 tokens once took (residual stream, operands, no slices' products) is enough for a prompt
    once = 1024 * (4096 * 8 + 14336 * 2 + 4096 * 4)
    assert plan("fit", *SHAPES["7b"], once)[0][0] >= 256


@pytest.mark.parametrize("rows,tiles,few", [
    (64, 384, 0), (65, 384, 1), (128, 384, 1), (129, 384, 0),             # 6144 columns
    (65, 512, 1), (128, 512, 1), (65, 513, 0), (65, 640, 0), (77, 768, 0),  # one round of 256 workgroups, and beyond it
    (100, 128, 1), (100, 1, 1),                                             # K and V of the last layer
])
def test_few_row_products_go_without_tiles_while_they_are_one_round(plan, rows, tiles, few):
    assert plan("few", rows, tiles, 256) == [[few]]


def test_the_gpu_sizes_reach_every_kernel_the_pass_picks_from(plan):
    """(product, tile or row tiles of the few-row kernel) and the numbers of slices, over all prompts of 65 to 2200 tokens of the
    shapes that the GPU test runs, against those at its sizes."""
    kernels, slices, have_kernels, have_slices = {}, {}, set(), set()
    for name, dtype, cases in SIZES:
        sh = shape_of(name, dtype)
        tested = {n for n, _ in cases}
        dims = (sh.d_model, sh.q_dim, sh.kv_dim, sh.d_ffn)
        for mode, n, tile, S in plan("routes", *dims, 65, 2200):
            kernels.setdefault((mode, tile), (name, n))
            slices.setdefault(S, (name, n))
            if n in tested:
                have_kernels.add((mode, tile))
                have_slices.add(S)
    assert {k: at for k, at in kernels.items() if k not in have_kernels} == {}
    assert {s: at for s, at in slices.items() if s not in have_slices} == {}
    assert len(kernels) >= 3 * 6 + 4  # all six tiles of the three kinds of product, four heights of the few-row kernel
