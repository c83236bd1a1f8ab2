// The large-M prompt pass's decisions that need no GPU: sizes of its buffers, which kernel a product takes.  Plain C++, so that a program without HIP can
// include it.
#pragma once
#include <stddef.h>

#include <initializer_list>

#include "la.h"

namespace la {

// Rows of one prompt chunk (buffers are sized for it).  At 2048 rows a 4096-column matrix fills the chip with one slice
// of the contraction: 2048 tokens, four layers, 2.77 ms against 3.02 in chunks of 1024; 1100 tokens 1.89 against 2.05.  4096
// rows gain nothing more (3000 tokens at 1000: 5.4 ms against 4.5, two rounds of which the second is nearly empty).
constexpr int PF_ROWS = 2048;
// Shorter prompts are one block of the block kernel (64 rows of the 7B shape, eight layers: 1.14 ms); two blocks read the
// weights twice (77 tokens 1.92 ms, the products' 128-row tiles 1.24).  The line is drawn for the prompt: what 2048 tokens leave
// over is a chunk of its own however short it is (2049 tokens of eight layers 7.9 ms, as 2048 + 1 in two calls 7.4; 2048 + 64
// 8.0 and 7.8; chunks of 1024 with smaller tiles had taken 13.6).
constexpr int PF_MIN = LA_MAX_ROWS + 1;
constexpr int PF_CHUNKS = 32;       // partial sums of squares per row (column chunks of pf_norm_kernel)
constexpr int PF_PART_ROWS = 4096;  // rows of all slices' products together, at most
constexpr int PF_MAX_SPLIT = 8;     // most slices of a contraction

// Two sets of buffers: prompts shorter than PF_LONG run in one of PF_LONG rows (26 MB at the 7B shape), so that a program
// of short prompts does not hold a whole chunk's (212 MB); the first longer prompt gets a set of PF_ROWS rows, or of as many
// as the card has memory left for, halving down to PF_LONG.
constexpr int PF_LONG = 128;

struct PfDims {
  size_t d_model, qdim, head_dim, d_ffn;
};
struct PfLayout {
  int rows = 0, part_rows = 0;  // rows of a chunk; rows of the slices' products together
  size_t x = 0, part = 0, ss = 0, cs = 0, A = 0, Q = 0, attn = 0, act = 0, total = 0;  // byte offsets in the one allocation, its size
};

inline PfLayout pf_layout(const PfDims &d, int rows) {
  PfLayout l;
  l.rows = rows;
  l.part_rows = PF_MAX_SPLIT * rows < PF_PART_ROWS ? PF_MAX_SPLIT * rows : PF_PART_ROWS;
  const size_t R = (size_t)rows;
  auto place = [&](size_t bytes) {
    const size_t at = l.total;
    l.total += (bytes + 1023) / 1024 * 1024;
    return at;
  };
  l.x = place(R * d.d_model * 4);
  l.part = place((size_t)l.part_rows * d.d_model * 4);
  l.ss = place(R * PF_CHUNKS * 4);
  l.cs = place(R * d.head_dim * 4);
  l.A = place(R * d.d_model * 2);
  l.Q = place(R * d.qdim * 2);
  l.attn = place(R * d.qdim * 2);
  l.act = place(R * d.d_ffn * 2);
  return l;
}

// The largest set of `most` rows, halved down to `least`, that alloc(bytes) succeeds for; rows = 0: none.
template <typename Alloc>
inline PfLayout pf_fit(const PfDims &d, int most, int least, Alloc alloc) {
  for (int rows = most; rows >= least; rows /= 2) {
    const PfLayout l = pf_layout(d, rows);
    if (alloc(l.total)) return l;
  }
  return PfLayout{};
}

// The tiles pf_choose picks from (pf_launch_tile has their kernels), and what a k-tile of them costs: of the two smallest, two
// workgroups fit a CU.
struct PfTile {
  int rows, cols;         // in 16 x 16 tiles
  int per_cu;
  float t_full, t_single;  // us per k-tile of a round that fills the chip, and of one with a workgroup per CU at most
};
// (from the products of the 7B shape at 77 .. 1023 rows, launch overhead included, before a step's requests were dealt out between its products: a launch takes
// 5 to 20 % less now; what is chosen by them is measured below)
constexpr PfTile PF_TILES[] = {
    {16, 14, 1, 0.85f, 0.85f}, {16, 10, 1, 0.66f, 0.66f}, {16, 8, 1, 0.57f, 0.57f}, {8, 12, 1, 0.50f, 0.50f}, {8, 8, 2, 0.70f, 0.45f}, {8, 4, 2, 0.52f, 0.30f},
};
constexpr int PF_N_TILES = 6, PF_SMALLEST = 5;

enum PfMode { PF_QKV = 0, PF_PART = 1, PF_GATEUP = 2 };

struct PfProduct {
  int RT, M, KT, n_tiles, d;  // row tiles of the buffers, rows, k-tiles, column tiles wanted, row length of the products
};
// Tile and number of slices of the contraction by estimated time: whole rounds of the chip's CUs times the k-tiles of a
// slice, and the slices' products written and read once (8 bytes an element at about 4.5 TB/s).  (The tiles are dealt to the eight
// XCDs evenly, so that the chip counts as one pool of CUs.)  Only
// the projections that add to the residual stream are sliced: at 1023 rows a 4096-column matrix has 128 tiles of 256 x 128
// for 256 CUs (down in one slice 182 us, in two 111 + 3 us more in pf_norm), at 77 rows 32 of 128 x 128 (eight slices).
// Against every tile, cut or not, and number of slices, 64 lengths of 65 .. 2047 rows, 7B and 12B shapes: what a product takes (pf_route) is within 5 % of the
// best in 591 of 640; the others are O of at most 512 rows (up to 36 %: 21.9 us against 16.1), down of 129 to 160 (12 %) and the last layer's K and V of 1100
// to 1200 (32 %).
inline float pf_choose(const PfProduct &p, int max_split, int part_rows, int cus, int &tile, int &S) {
  auto up = [](int a, int b) { return (a + b - 1) / b; };
  float best = 0.f;
  tile = -1;
  for (int i = 0; i < PF_N_TILES; ++i)
    for (int k = 1; k <= max_split; ++k) {
      const PfTile &t = PF_TILES[i];
      if (k > 1 && (p.KT / k < 4 || (long long)k * p.M > part_rows)) break;
      const int n = up(p.RT, t.rows) * up(p.n_tiles, t.cols) * k, round = t.per_cu * cus, rest = n % round;
      float us = (float)(n / round) * t.t_full + (rest == 0 ? 0.f : rest <= cus ? t.t_single : t.t_full);
      us *= (float)up(p.KT, k);
      if (max_split > 1) us += (float)k * (float)p.M * (float)p.d * 8.f / 4.5e6f;
      if (tile < 0 || us < best) {
        best = us;
        tile = i;
        S = k;
      }
    }
  return best;
}

// Tiles that are cut to the prompt's rows, as row tiles of a workgroup (pf_launch_rows has their kernels); 0: pf_choose's.  What they save
// is a CU's intake: a KB takes a CU 16 ns (lines of its XCD's L2) to 35 ns (weights from memory), whatever the depth of the ring, the
// policy of the loads or lines requested ahead into L2, and a small product waits for nothing else.
// Up to 128 rows, of gate/up 7 columns and all rows a workgroup: 28672 columns in one round of 256 CUs, and no padding rows.  us, before (128 x 128
// tiles on 224 CUs) and now: 77 rows 56.3 -> 46.0, 128 rows 57.6 -> 54.0.  Where pf_choose takes its smallest tiles, which then are at most one
// to a CU, those are faster (4096 wide, smallest or 128 x 128 tiles / 7 columns: 8192 channels of gate 35.3 / 37.8 at 77 rows and 36.3 / 45.9 at 128, 8704 channels
// 45.8 / 36.9 and 46.9 / 45.3; 2048 wide, 8192 channels 16.2 / 17.2 and 16.7 / 22.9).
// Of O and down 8 columns and all rows, in as many slices as fill the chip (if that is more than half of it), but where pf_choose takes its smallest tiles:
// those are faster there, too.  us with what the slices cost pf_norm, tiles / cut: down of 4096 x 14336 77 rows 31.0 / 29.5, 128 rows 34.8 / 34.1; O of
// 4096 x 4096 77 rows 13.3 / 12.9, 96 rows 12.6 / 13.8, 128 rows 13.3 / 15.2; O of 5120 x 4096 97 rows 21.1 / 18.5, 112 rows 16.3 / 19.6; down of 3072 x 8192
// (192 workgroups) 70 rows 16.3 / 14.9, 96 rows 15.3 / 16.2.  Of 15 widths and 13 lengths none is more than 3 % slower than pf_choose's but O of 8192 x
// 8192 at 97 and 105 rows (7 %).
// Beyond five row tiles in seven slices at most: with eight, 256 workgroups, a launch takes 4 us more now and then, on some cards most of the time.  Down of
// 4096 x 14336, us in the mean of 100 on two cards, eight slices / seven / tiles: 80 rows 29.0, 29.2 / 29.0, 29.5 / 31.1, 31.2; 97 rows 32.4, 34.5 / 31.9, 32.5 /
// 32.6, 32.6; 112 rows 33.6, 36.7 / 33.0, 34.2 / 33.6, 33.7.
// Gate/up beyond 128 rows: 10 or 12 row tiles x 14 columns where whole rounds of them cost less than pf_choose's best, at 0.64 and 0.69 us per k-tile against
// PF_TILES' (the 16 row tiles of that width take 0.70 there, not 0.85, at 257 rows; the constants are kept because what they choose is right): 7B shape, 300
// rows 91 -> 82, 600 rows 164 -> 143, 700 rows 176 -> 160, 1600 rows 374 -> 354.  Over 15 widths up to 512 rows and nine up to 2047 they take a slower kernel
// only of 10240 channels at 257 and 288 rows (71 -> 75).
// QKV of 129 to 512 rows: a quarter of the rows and 6 columns a workgroup, while that is one round (7B and 12B shapes: 64 column groups).
// 150 rows 33 -> 29, 200 rows 36.6 -> 32.0, 300 rows 51 -> 38, 400 rows 56 -> 45, 500 rows 59 -> 52.
// Beyond 256 rows (five row tiles), where pf_choose takes its smallest tiles (fewer columns: the last layer's K and V, narrow models), only while the
// contraction is short.  Time over the tiles' at 3 / 4 / 5 / 6 / 7 / 8 row tiles, K and V: 512 wide .75 / .80 / .92 / .97 / 1.09 / 1.16, 1024 wide .73 / .82 / .91 /
// 1.00 / 1.12 / 1.21, 2048 wide .80 / .86 / .96 / 1.04 / 1.18 / 1.24, 3072 wide .87 / .87 / 1.04 / 1.03 / 1.26 / 1.23, 4096 wide .91 / .86 / 1.07 / 1.03 / 1.30 / 1.24,
// 8192 wide 1.02 / .89 / 1.17 / 1.03 / 1.39 / 1.24; 4096 x 6144, more than one round of those tiles: .92 / .88 / .68 / .69 / .84 / .85.
constexpr int PF_ROW_COLS_QKV = 6, PF_ROW_COLS_PART = 8, PF_ROW_COLS_GATEUP = 7;
inline int pf_up(int a, int b) { return (a + b - 1) / b; }
inline int pf_qkv_rows(const PfProduct &p, int cus) {
  const int rt = pf_up(p.M, 16), rows = pf_up(rt, 4);
  if (p.M <= 128 || p.M > 512 || pf_up(rt, rows) * pf_up(p.n_tiles, PF_ROW_COLS_QKV) > cus) return 0;
  int tile, S;
  pf_choose(p, 1, 0, cus, tile, S);
  return rows <= 4 || tile != PF_SMALLEST || p.KT <= 32 * (7 - rows) ? rows : 0;
}
inline int pf_part_rows(const PfProduct &p, int part_rows, int cus, int &S) {
  const int groups = pf_up(p.n_tiles, PF_ROW_COLS_PART), rt = pf_up(p.M, 16), most = rt > 5 ? PF_MAX_SPLIT - 1 : PF_MAX_SPLIT;
  int k = cus / groups < most ? cus / groups : most, tile, S_tile;
  while (k > 1 && (p.KT / k < 4 || (long long)k * p.M > part_rows)) --k;
  if (p.M <= LA_MAX_ROWS || p.M > 128 || k < 1 || 2 * groups * k <= cus) return 0;
  pf_choose(p, PF_MAX_SPLIT, part_rows, cus, tile, S_tile);
  if (tile == PF_SMALLEST) return 0;
  S = k;
  return rt;
}
inline int pf_gateup_rows(const PfProduct &p, int cus) {
  const int rt = pf_up(p.M, 16);
  int tile, S, rows = 0;
  float best = pf_choose(p, 1, 0, cus, tile, S);
  if (p.M <= 128) return p.M > LA_MAX_ROWS && pf_up(p.n_tiles, PF_ROW_COLS_GATEUP) <= cus && tile != PF_SMALLEST ? rt : 0;
  for (int r : {10, 12}) {
    const float us = (float)(pf_up(pf_up(rt, r) * pf_up(p.n_tiles, 14), cus) * p.KT) * (r == 10 ? 0.64f : 0.69f);
    if (us < best) {
      best = us;
      rows = r;
    }
  }
  return rows;
}

// The QKV product of M rows and n_tiles column tiles by the kernel without tiles (pf_qkv_few_kernel: two column tiles and all rows a
// workgroup): up to 128 rows, while its workgroups are one round of the chip.  us, without / with tiles, at 65 and 128 rows:
// 4096 x 6144 (192 workgroups) 27 / 39, 30 / 39; 4096 x 8192 (256) 29 / 38, 32 / 40; beyond one round every workgroup's own
// pass over the activations costs more than the tiles: 4096 x 12288 (384) 46 / 42, 52 / 43; 8192 x 10240 (320) 78 / 67, 93 / 67.
// The last layer's 2048 columns of K and V: 16 / 37, 21 / 38.
inline bool pf_qkv_few(int M, int n_tiles, int cus) { return M > LA_MAX_ROWS && M <= 128 && (n_tiles + 1) / 2 <= cus; }

// The kernel that a product takes.
struct PfRoute {
  int few = 0;    // row tiles, by the kernel without tiles; 0: not by it
  int rows = 0;   // row tiles of a tile that is cut to the prompt's rows; 0: not by one
  int tile = -1;  // else: of PF_TILES
  int S = 1;      // slices of the contraction
};
inline PfRoute pf_route(PfMode mode, const PfProduct &p, int part_rows, int cus) {
  PfRoute r;
  if (mode == PF_QKV && pf_qkv_few(p.M, p.n_tiles, cus)) r.few = pf_up(p.M, 16);
  else if (mode == PF_QKV) r.rows = pf_qkv_rows(p, cus);
  else if (mode == PF_PART) r.rows = pf_part_rows(p, part_rows, cus, r.S);
  else r.rows = pf_gateup_rows(p, cus);
  if (!r.few && !r.rows) pf_choose(p, mode == PF_PART ? PF_MAX_SPLIT : 1, part_rows, cus, r.tile, r.S);
  return r;
}

static_assert(PF_PART_ROWS >= PF_ROWS, "one slice of a whole chunk");
static_assert(PF_ROWS % PF_LONG == 0 && PF_MIN <= PF_LONG, "chunks halve down to the smaller set");

}  // namespace la
