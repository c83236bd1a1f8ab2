"""The prompt pass's host decisions (la_prefill_plan.h, plain C++): a small program prints them, checked here without a GPU."""
import os
import subprocess

import pytest

from test_gpu_prefill_tiles import SIZES, shape_of
from test_prefill_rows import SIZES as ROW_SIZES

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
  if (!strcmp(v[1], "routes")) {  // product (QKV, O, gate/up, down, the last layer's K and V) by product: prompt lengths v[6] .. v[7]
    const int d = (int)num(2), qd = (int)num(3), kvd = (int)num(4), F = (int)num(5);
    for (int n = (int)num(6); n <= (int)num(7); ++n) {
      const int rows = n < PF_LONG ? PF_LONG : PF_ROWS, part_rows = pf_layout(PfDims{(size_t)d, (size_t)qd, 128, (size_t)F}, rows).part_rows;
      for (int done = 0; done < n; done += rows) {
        const int M = n - done < rows ? n - done : rows, RT = (M + 63) / 64 * 4;
        const struct { PfMode mode; int K, cols; } products[] = {{PF_QKV, d, qd + 2 * kvd}, {PF_PART, qd, d}, {PF_GATEUP, d, 2 * F}, {PF_PART, F, d}, {PF_QKV, d, 2 * kvd}};
        for (int i = 0; i < 5; ++i) {
          const PfRoute r = pf_route(products[i].mode, PfProduct{RT, M, products[i].K / 32, products[i].cols / 16, d}, part_rows, 256);
          printf("%d %d %d %d %d %d\n", i, n, products[i].mode, r.few ? 100 + r.few : r.rows ? 200 + r.rows : r.tile, r.S, r.S * M <= part_rows);
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
    """By the function that the launches ask: of each kind of product every kernel, and of O and of down every kernel with every number of slices, over all prompts
    of 65 to 2200 tokens of the shapes that the GPU tests run, against those at their sizes."""
    want, have = {}, set()
    for name, dtype, cases in SIZES + ROW_SIZES:
        sh = shape_of(name, dtype)
        tested = {n for n, _ in cases}
        for product, n, mode, kernel, S, fits in plan("routes", sh.d_model, sh.q_dim, sh.kv_dim, sh.d_ffn, 65, 2200):
            assert fits
            for key in ((mode, kernel), (product, kernel, S))[:2 if mode == 1 else 1]:
                want.setdefault(key, (name, n))
                if n in tested:
                    have.add(key)
    assert {k: at for k, at in want.items() if k not in have} == {}
    # all six tiles, the heights of the few-row kernel and of the cut tiles of the three kinds of product
    assert {k for k in want if len(k) == 2} == {(m, t) for m in range(3) for t in range(6)} | {(0, 100 + r) for r in range(5, 9)} | \
        {(0, 200 + r) for r in range(3, 9)} | {(1, 200 + r) for r in range(5, 9)} | {(2, 200 + r) for r in (5, 6, 7, 8, 10, 12)}
