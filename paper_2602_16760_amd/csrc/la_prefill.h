// Large-M prompt pass (Section 4.1 step 1, Section 6.3 "Prefill"; chunked prefill is the paper's named future work,
// Section 8): the whole prompt, up to PF_ROWS tokens at a time, goes through each layer as ONE matrix product per weight
// matrix, so the weights are read once per prompt chunk instead of once per 64 rows.  Included by la_mfma.hip (it needs
// the model's packed weight streams).
//
// Per layer: pf_norm (the residual stream takes in the down projection of the layer before; sums of squares and x * gain as
// half-precision MFMA operand fragments) -> pf_tile QKV (epilogue: row factor, RoPE, K and V rows into the cache, q as
// operand fragments) -> pf_attn (causal flash attention over the cache) -> pf_tile O (products of the contraction's
// slices) -> pf_norm -> pf_tile gate/up (epilogue: SwiGLU into operand fragments) -> pf_tile down.  The arithmetic is the
// block kernel's (half-precision operands, f32 accumulation, the cache's 16-bit type in the attention); only the order
// of the sums differs.
//
// Both operands of the products are MFMA fragments of 1 KB: the activations are stored as [k-tile][row tile][lane][8
// halves] by their producers, and a weight fragment is the 1 KB block of the per-CU streams the block kernel reads.
#pragma once
#include "la_prefill_plan.h"

namespace la {

constexpr int PF_KEYS = 64;     // keys of a block of the attention

struct PfGemm {
  const uint8_t *wstream;
  size_t cu_bytes;
  unsigned frag0;  // fragment index of the layer inside a CU's region
  int G, NW;       // workgroups and MFMA waves the streams were packed for
  int n_prev, prev_ntiles[3], prev_KT[3];
  int t_first, ntiles, KT;  // column tiles t_first .. ntiles - 1 are wanted
  int S;              // slices of the contraction (PART; else 1)
  const uint16_t *A;  // operand fragments [KT][RT][64][8]
  int RT, M;          // row tiles the buffers are laid out for, rows
  // epilogues
  float *part;        // PART: products of slice s [S][M][d]
  int d;
  const float *ss;    // QKV, GATEUP: partial sums of squares of the norm's input [M][PF_CHUNKS]
  float inv_d, eps;
  const float *cs;    // QKV: cos, sin [M][dh/2][2]
  uint16_t *Kc, *Vc;  // QKV: this layer's cache
  uint16_t *Q;        // QKV: q fragments [Hq][RT][dh/32][64][8]
  int L0, Hq, Hkv, dh, f16;
  uint16_t *act;      // GATEUP: operand fragments of the down projection [F/32][RT][64][8]
};

// The epilogue of a wave's tile.  The products are formed with the weight fragment as the MFMA's first operand, so
// a lane holds FOUR CONSECUTIVE COLUMNS of one row (NM row tiles x NTW column tiles): acc[m][j][i] is row 16 (r0 + m) + c16, column 4 q4 + i of column
// tile t0 + j.  Every store is then an 8- or 16-byte vector (the cache's V layout aside), and the partner of a RoPE
// pair or of a gate channel (8 columns further) sits 32 lanes further.
template <int MODE, int NM, int NTW>
__device__ __forceinline__ void pf_epilogue(const PfGemm &p, const f32x4 (&acc)[NM][NTW], int r0, int t0, int lane, int slice, LDS_AS const float *rf) {
  const int q4 = lane >> 4, c16 = lane & 15;
  float rsm[NM];  // row factors of the norm
#pragma unroll
  for (int m = 0; m < NM; ++m) rsm[m] = MODE == PF_PART ? 0.f : rf[16 * m + c16];
#pragma unroll
  for (int j = 0; j < NTW; ++j) {
    const int t = t0 + j;
    if (t >= p.ntiles) continue;
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const int row = 16 * (r0 + m) + c16;
      const f32x4 v = acc[m][j];
      if (MODE == PF_PART) {
        if (row < p.M) *reinterpret_cast<f32x4 *>(p.part + ((size_t)slice * p.M + row) * p.d + 16 * t + 4 * q4) = v;
      } else {
        const float rsf = rsm[m];
        f32x4 other;
#pragma unroll
        for (int i = 0; i < 4; ++i) other[i] = __shfl_xor(v[i], 32, 64);
        if (row >= p.M) continue;
        if (MODE == PF_GATEUP) {
          // tile columns: 8 gate channels (lanes q4 = 0, 1), then the same 8 channels of up (q4 = 2, 3)
          if (q4 < 2) {
            float y[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float g = v[i] * rsf, u = other[i] * rsf;
              y[i] = g / (1.0f + __expf(-g)) * u;
            }
            const int ch = 8 * t + 4 * q4;
            *(u32x2 *)((uint8_t *)p.act + frag_piece(ch & ~7, row, p.RT) + 8 * (q4 & 1)) = u32x2{pack_f16(y[0], y[1]), pack_f16(y[2], y[3])};
          }
        } else {
          // tile columns: channels 8 jj .. 8 jj + 7 (q4 = 0, 1) and dh/2 + 8 jj .. (q4 = 2, 3) of head hs: eight RoPE pairs
          const int spj = p.dh >> 4, half = p.dh >> 1;
          const int hs = t / spj, jj = t - hs * spj;
          const int pr = 8 * jj + 4 * (q4 & 1);  // first of this lane's four pairs
          const int ch = q4 < 2 ? pr : half + pr;
          const bool h16 = p.f16 != 0;
          float y[4];
          if (hs < p.Hq + p.Hkv) {
            const float qscale = hs < p.Hq ? 1.0f / sqrtf((float)p.dh) : 1.0f;
            const f32x4 *csp = reinterpret_cast<const f32x4 *>(p.cs + ((size_t)row * half + pr) * 2);
            const f32x4 cs0 = csp[0], cs1 = csp[1];  // (cos, sin) of pairs pr .. pr + 3
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float c = i < 2 ? cs0[2 * i] : cs1[2 * (i - 2)], sn = i < 2 ? cs0[2 * i + 1] : cs1[2 * (i - 2) + 1];
              const float mine = v[i] * rsf, oth = other[i] * rsf;
              y[i] = (q4 < 2 ? mine * c - oth * sn : mine * c + oth * sn) * qscale;
            }
          } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) y[i] = v[i] * rsf;
          }
          if (hs < p.Hq) {
            const int KTq = p.dh >> 5;
            const size_t frag = ((size_t)hs * p.RT + (row >> 4)) * KTq + (ch >> 5);
            *(u32x2 *)(p.Q + (frag * 64 + (row & 15) + 16 * ((ch & 31) >> 3)) * 8 + (ch & 7)) = u32x2{pack_kv(h16, y[0], y[1]), pack_kv(h16, y[2], y[3])};
          } else if (hs < p.Hq + p.Hkv) {
            *(u32x2 *)(p.Kc + ((size_t)(p.L0 + row) * p.Hkv + (hs - p.Hq)) * p.dh + ch) = u32x2{pack_kv(h16, y[0], y[1]), pack_kv(h16, y[2], y[3])};
          } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) p.Vc[v_index(true, p.L0 + row, hs - p.Hq - p.Hkv, ch + i, p.Hkv, p.dh)] = kv_bits(h16, y[i]);
          }
        }
      }
    }
  }
}

template <int N>
__device__ __forceinline__ void pf_wait_lds_reads() {  // at most N LDS operations of this wave outstanding
  asm volatile("s_waitcnt lgkmcnt(%0)" : : "n"(N) : "memory");
}

// Row factor of the norm from the partial sums of squares.
__device__ __forceinline__ float pf_row_factor(const PfGemm &p, int row) {
  if (row >= p.M) return 0.f;
  f32x4 a = {0.f, 0.f, 0.f, 0.f};
  const f32x4 *sp = reinterpret_cast<const f32x4 *>(p.ss + (size_t)row * PF_CHUNKS);
#pragma unroll
  for (int i = 0; i < PF_CHUNKS / 4; ++i) a += sp[i];
  return 1.0f / sqrtf(((a[0] + a[1]) + (a[2] + a[3])) * p.inv_d + p.eps);
}

// One product.  A workgroup computes a tile of 16 NM WM rows x 16 WN NTW columns, a wave 16 NM rows x 16 NTW columns of it (NM is 4 but in tiles
// that are cut to the prompt's rows); the
// fragments of a k-tile (32 deep) come in once per workgroup with direct-to-LDS loads, into a ring of NS stages.
// Bound: the matrix cores, if the operands get there: a wave reads NM + NTW fragments of LDS for NM NTW products (16 cycles
// each, four waves' reads sharing 128 bytes a cycle), so small tiles are LDS-bound, and a workgroup takes NM WM + WN NTW KB
// a k-tile through its CU's 64 bytes a cycle.  256 rows x 224 columns (8 waves, one workgroup per CU) needs 79 % of the
// LDS cycles and 54 % of the load cycles that its products take, and cuts the 28672 columns of the 7B shape's gate/up
// into whole rounds of 256 CUs; smaller tiles are for the narrower matrices and fewer rows (pf_choose).  One workgroup
// barrier per k-tile: past it every wave's part of the next stage is in, and nobody reads the stage any more that the
// next requests overwrite (its fragments are in registers, one k-tile ahead of the products).
// A step's requests and fragment reads are dealt out between its products, and the offsets of the requests only ever grow by a constant
// (but for the ends of the walk's runs): with all requests behind the barrier and their offsets multiplied out, the products waited for some
// fifty scalar instructions and for the load unit to take 30 KB (a k-tile's other instructions: 79 -> 37 beside 28 products).
// 1023 rows, 7B shape, us a product, before and after: gate/up 222 -> 202 (1190 TFLOP/s; a large library product reaches 1219 on this
// card), QKV 66 -> 61, O 44 -> 41, down 123 -> 110; 2048 rows: 428 -> 395, 110 -> 102, 72 -> 66, 223 -> 205.  What is left is paid in clock:
// with the same operands over and over gate/up takes 131 us, with constant fragments through LDS 176.  Four waves of 128 x 112 or 64 x 128
// read a third less LDS and are no faster (214, and 106 for down): one wave a SIMD has nothing to do at the barrier.
template <int MODE, int WM, int WN, int NTW, int NS, int NM>
__device__ __forceinline__ void pf_tile_body(const PfGemm &p, LDS_AS uint8_t *pf_lds) {
  constexpr int NWV = WM * WN;                  // waves
  constexpr int RTB = NM * WM, CTB = WN * NTW;  // row and column tiles of the workgroup
  constexpr int F = RTB + CTB;                 // fragments of a k-tile
  constexpr int LPW = (F + NWV - 1) / NWV;     // ... a wave brings (the last one several times if they do not divide)
  static_assert((NS - 1) * LPW <= 63, "load counter");
  const int wave = uni((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int wm = wave % WM, wn = wave / WM;
  const int n_cg = (p.ntiles - p.t_first + CTB - 1) / CTB, RB = ((p.M + 15) / 16 + RTB - 1) / RTB;
  // An XCD takes a run of the tiles, row blocks first (they share the weights in its L2), and all XCDs as many, to one: with whole
  // column groups dealt to them, some had a round of workgroups more than the chip needs (7B shape, 700 rows: down
  // 166 -> 91 us, O 61 -> 36; 1300 rows: 298 -> 160, 101 -> 57; 1600 rows: gate/up 452 -> 390; 12B shape, 300 rows: down 121 -> 67).
  const int tiles = RB * p.S * n_cg, per_xcd = (tiles + 7) / 8, turn = (int)blockIdx.x / 8, tile = ((int)blockIdx.x % 8) * per_xcd + turn;
  if (tile >= tiles) return;  // (the whole workgroup; the grid is eight times per_xcd)
  const int rb = tile % RB, slice = tile / RB % p.S, cg = tile / (RB * p.S);
  const int row0 = p.KT * slice / p.S, row1 = p.KT * (slice + 1) / p.S, n_kt = row1 - row0;
  const unsigned lds0 = (unsigned)(uintptr_t)pf_lds;
  const unsigned voff = (unsigned)lane * 16u;
  // The k-tiles go in the order the weights are stored: row r of a tile's stream is k-tile kt, kt = w, w + NW, ... for w = 0, 1, ...
  int nx_kt = row0, nx_w = 0;
  while (nx_kt >= (p.KT - nx_w + p.NW - 1) / p.NW) {
    nx_kt -= (p.KT - nx_w + p.NW - 1) / p.NW;
    ++nx_w;
  }
  nx_kt = nx_w + p.NW * nx_kt;
  // what this wave brings of a k-tile: fragments wave * LPW ..; 0 .. RTB - 1 are the activations' row tiles
  __amdgpu_buffer_rsrc_t rs[LPW];
  unsigned of[LPW], inc[LPW], dst[LPW];
  int n_act = 0;
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    int f = wave * LPW + i;
    if (f >= F) f = F - 1;
    dst[i] = uni(lds0 + (unsigned)f * 1024u);
    if (f < RTB) {
      const int r = rb * RTB + f;
      rs[i] = rsrc_of(p.A);
      of[i] = uni((unsigned)((r < p.RT ? r : p.RT - 1) + nx_kt * p.RT) * 1024u);
      inc[i] = uni((unsigned)(p.NW * p.RT) * 1024u);
      n_act = i + 1;
    } else {
      const int tj = p.t_first + cg * CTB + f - RTB;
      const int t = tj < p.ntiles ? tj : p.ntiles - 1;  // (a group past the last tile repeats it; its result is dropped)
      const int c = uni(t % p.G), lt = uni(t / p.G);
      unsigned off = p.frag0;
      for (int q = 0; q < p.n_prev; ++q) off += (unsigned)((p.prev_ntiles[q] > c ? (p.prev_ntiles[q] - c + p.G - 1) / p.G : 0) * p.prev_KT[q]);
      const unsigned nt = (unsigned)((p.ntiles - c + p.G - 1) / p.G);
      rs[i] = rsrc_of(p.wstream + (size_t)c * p.cu_bytes);
      of[i] = uni((off + (unsigned)lt + (unsigned)row0 * nt) * 1024u);
      inc[i] = uni(nt * 1024u);
    }
  }
  // requests until the walk leaves the line of its offsets: the end of a run of k-tiles, where the activations' go back, or the last k-tile,
  // which is requested again from then on and never used
  int left = uni(row1 - row0 - 1), run = uni((p.KT - 1 - nx_kt) / p.NW);
  unsigned nx_slot = 0;
  auto advance = [&]() {
    if (left > 0) {
#pragma unroll
      for (int i = 0; i < LPW; ++i) of[i] += inc[i];
      if (run == 0) {  // from the last k-tile of run w to k-tile w + 1
        ++nx_w;
        const int last = nx_w - 1 + (p.KT - nx_w) / p.NW * p.NW;
#pragma unroll
        for (int i = 0; i < LPW; ++i)
          if (i < n_act) of[i] = uni(of[i] - inc[i] - (unsigned)((last - nx_w) * p.RT) * 1024u);
        run = uni((p.KT - 1 - nx_w) / p.NW + 1);
      }
      --run;
      --left;
    }
    nx_slot = nx_slot + F * 1024u == NS * F * 1024u ? 0u : nx_slot + F * 1024u;
  };
  auto request_one = [&](int i) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs[i], (LDS_AS void *)(uintptr_t)(dst[i] + nx_slot), 16, voff, of[i], 0, 0);
  };
  u32x4 fa[2][NM], fb[2][NTW];
  unsigned rd_slot = 0;
  const unsigned rd_a = lds0 + voff + (unsigned)(NM * wm) * 1024u, rd_b = lds0 + voff + (unsigned)(RTB + wn * NTW) * 1024u;
  f32x4 acc[NM][NTW];
#pragma unroll
  for (int m = 0; m < NM; ++m)
#pragma unroll
    for (int j = 0; j < NTW; ++j) acc[m][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto product = [&](int s, int n) {
    const int j = n / NM, m = n % NM;
    acc[m][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, fb[s][j]), __builtin_bit_cast(f16x8, fa[s][m]), acc[m][j], 0, 0, 0);
  };
  auto read_one = [&](int s, int f, unsigned a, unsigned b) {
    if (f < NTW) fb[s][f < NTW ? f : 0] = *(LDS_AS const u32x4 *)(uintptr_t)(b + (unsigned)f * 1024u);
    else fa[s][f < NTW ? 0 : f - NTW] = *(LDS_AS const u32x4 *)(uintptr_t)(a + (unsigned)(f - NTW) * 1024u);
  };
  auto turn_over = [&]() {  // everybody's next stage is in, and everybody has read the stage that the next request overwrites
    wait_vmcnt<(NS - 2) * LPW>();
    pf_wait_lds_reads<0>();
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_barrier();
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
  };
  // a step: the products of the k-tile in registers, the fragments of the next one and the requests of one further on between them
  auto step = [&](int s) {
    constexpr int P = NM * NTW, R = NM + NTW;
    turn_over();
    const unsigned a = rd_a + rd_slot, b = rd_b + rd_slot;
#pragma unroll
    for (int n = 0; n < P; ++n) {
      // read f goes in front of product f P / R, request i in front of product (2 i + 1) P / (2 LPW)
#pragma unroll
      for (int f = 0; f < R; ++f)
        if (f * P / R == n) read_one(s ^ 1, f, a, b);
#pragma unroll
      for (int i = 0; i < LPW; ++i)
        if ((2 * i + 1) * P / (2 * LPW) == n) request_one(i);
      product(s, n);
      __builtin_amdgcn_sched_barrier(0);
      if (n == (2 * LPW - 1) * P / (2 * LPW)) {  // (the last request is out)
        advance();
        rd_slot = rd_slot + F * 1024u == NS * F * 1024u ? 0u : rd_slot + F * 1024u;
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
#pragma unroll
  for (int s = 0; s < NS; ++s) {
#pragma unroll
    for (int i = 0; i < LPW; ++i) request_one(i);
    advance();
  }
  // row factors of the norm into LDS, while the first stages are on their way
  LDS_AS float *rf = (LDS_AS float *)(uintptr_t)(lds0 + NS * F * 1024u);
  if (MODE != PF_PART && (int)threadIdx.x < 16 * RTB) rf[threadIdx.x] = pf_row_factor(p, 16 * rb * RTB + (int)threadIdx.x);
  wait_vmcnt<(NS - 1) * LPW>();
  pf_wait_lds_reads<0>();
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_s_barrier();
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
#pragma unroll
  for (int f = 0; f < NM + NTW; ++f) read_one(0, f, rd_a, rd_b);
  rd_slot = F * 1024u;
  int r = 0;
  for (; r + 2 <= n_kt; r += 2) {
    step(0);
    step(1);
  }
  if (r < n_kt) {
#pragma unroll
    for (int n = 0; n < NM * NTW; ++n) product(0, n);
  }
  wait_vmcnt<0>();  // (the requests past the last k-tile land before the LDS is given back)
  const int r0 = rb * RTB + NM * wm;
  if (r0 < p.RT) pf_epilogue<MODE, NM, NTW>(p, acc, r0, p.t_first + cg * CTB + wn * NTW, lane, slice, rf + 16 * NM * wm);
}

template <int MODE, int WM, int WN, int NTW, int NS, int NM>
__global__ __launch_bounds__(64 * WM * WN, 2) void pf_tile_kernel(PfGemm p) {
  extern __shared__ __attribute__((aligned(1024))) uint8_t pf_lds[];
  pf_tile_body<MODE, WM, WN, NTW, NS, NM>(p, (LDS_AS uint8_t *)pf_lds);
}

// The QKV product for 65 to 128 rows where it has few columns (pf_qkv_few; 96 of the smallest tiles for 256 CUs at the 7B shape)
// and an epilogue that cannot take slices of the contraction: a workgroup takes two column tiles and all rows, and its four waves share the contraction (wave w the
// k-tiles w, w + 4, ..., which is how the weights lie); each streams its fragments into registers, NS k-tiles ahead, with
// no barrier until the four sums are added.  MT: row tiles that hold rows (padding is neither loaded nor multiplied).  Bound by
// the activations' way in, which every workgroup repeats: 77 rows of the 7B shape 37.5 -> 23.8 us, 120 rows 38.7 -> 28.0; the
// gate/up product is faster in tiles (77 rows 57.8 us, this way 75.7).
template <int MT, int NS>
__device__ __forceinline__ void pf_qkv_few_body(const PfGemm &p, LDS_AS uint8_t *lds) {
  constexpr int CT = 2;
  const int wave = uni((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int t0 = p.t_first + (int)blockIdx.x * CT;
  const unsigned lds0 = (unsigned)(uintptr_t)lds;
  LDS_AS float *rf = (LDS_AS float *)(uintptr_t)(lds0 + 4u * MT * CT * 1024u);
  if ((int)threadIdx.x < 16 * MT) rf[threadIdx.x] = pf_row_factor(p, (int)threadIdx.x);
  // this wave's k-tiles: wave + 4 i, i < nk; fragment (before + i) of a tile's stream
  const int nk = p.KT > wave ? (p.KT - wave + 3) / 4 : 0;
  int before = 0;
  for (int w = 0; w < wave; ++w) before += p.KT > w ? (p.KT - w + 3) / 4 : 0;
  const uint8_t *wb[CT];
  unsigned wstep[CT];
#pragma unroll
  for (int j = 0; j < CT; ++j) {
    const int t = t0 + j < p.ntiles ? t0 + j : p.ntiles - 1;  // (a group past the last tile repeats it; its result is dropped)
    const int c = uni(t % p.G), lt = uni(t / p.G);
    unsigned off = p.frag0;
    for (int q = 0; q < p.n_prev; ++q) off += (unsigned)((p.prev_ntiles[q] > c ? (p.prev_ntiles[q] - c + p.G - 1) / p.G : 0) * p.prev_KT[q]);
    const unsigned nt = uni((unsigned)((p.ntiles - c + p.G - 1) / p.G));
    wstep[j] = nt * 1024u;
    wb[j] = p.wstream + (size_t)c * p.cu_bytes + ((size_t)off + (unsigned)lt + (size_t)before * nt) * 1024u + (unsigned)lane * 16u;
  }
  const uint8_t *ab = (const uint8_t *)p.A + (size_t)lane * 16u;
  const size_t a_kt = (size_t)p.RT * 1024u;
  auto load = [&](int i, u32x4 (&a)[MT], u32x4 (&b)[CT]) {
    const uint8_t *ap = ab + (size_t)(wave + 4 * i) * a_kt;
#pragma unroll
    for (int j = 0; j < CT; ++j) b[j] = *(const u32x4 *)(wb[j] + (size_t)i * wstep[j]);
#pragma unroll
    for (int m = 0; m < MT; ++m) a[m] = *(const u32x4 *)(ap + (unsigned)m * 1024u);
  };
  f32x4 acc[MT][CT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int j = 0; j < CT; ++j) acc[m][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto mul = [&](const u32x4 (&a)[MT], const u32x4 (&b)[CT]) {
#pragma unroll
    for (int j = 0; j < CT; ++j)
#pragma unroll
      for (int m = 0; m < MT; ++m)
        acc[m][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, b[j]), __builtin_bit_cast(f16x8, a[m]), acc[m][j], 0, 0, 0);
  };
  // A window of NS k-tiles.  The loop has no branch around a load (requests past the last k-tile repeat it and are never
  // used), so that the compiler counts the loads on their way instead of waiting for all of them.
  if (nk > 0) {
    u32x4 sa[NS][MT], sb[NS][CT];
#pragma unroll
    for (int s = 0; s < NS - 1; ++s) load(s < nk ? s : nk - 1, sa[s], sb[s]);
    int i = 0;
    for (; i + NS <= nk; i += NS) {
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int nx = i + s + NS - 1;
        load(nx < nk ? nx : nk - 1, sa[(s + NS - 1) % NS], sb[(s + NS - 1) % NS]);
        __builtin_amdgcn_sched_barrier(0);
        mul(sa[s], sb[s]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
      if (i + s < nk) mul(sa[s], sb[s]);
  }
  LDS_AS f32x4 *part = (LDS_AS f32x4 *)(uintptr_t)lds0 + lane;
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int j = 0; j < CT; ++j) part[((wave * MT + m) * CT + j) * 64] = acc[m][j];
  __syncthreads();
  for (int m = wave; m < MT; m += 4) {  // a wave finishes every fourth row tile
    f32x4 sum[1][CT];
#pragma unroll
    for (int j = 0; j < CT; ++j) {
      sum[0][j] = part[(m * CT + j) * 64];
#pragma unroll
      for (int w = 1; w < 4; ++w) sum[0][j] += part[((w * MT + m) * CT + j) * 64];
    }
    pf_epilogue<PF_QKV, 1, CT>(p, sum, m, t0, lane, 0, rf + 16 * m);
  }
}

template <int MT, int NS>
__global__ __launch_bounds__(256, 2) void pf_qkv_few_kernel(PfGemm p) {
  extern __shared__ __attribute__((aligned(1024))) uint8_t pf_lds[];
  pf_qkv_few_body<MT, NS>(p, (LDS_AS uint8_t *)pf_lds);
}

// The residual stream takes in the products of the projection before (x += the slices' products, added in slice order),
// and the operand fragments of x * gain and the sums of squares for the next projection's row factors are formed in the
// same pass: a workgroup takes 16 rows x one of PF_CHUNKS column chunks, a wave whole fragments of 16 rows x 32 columns.
// S = 0: x as it is.  Rows M .. 16 RT - 1 of the fragments are written as zeros (the products read whole row blocks).
template <int S>
__global__ __launch_bounds__(256) void pf_norm_kernel(float *x, const float *part, const float *gain, int M, int d, int RT, float *ss, uint16_t *A) {
  const int rt = blockIdx.x, chunk = blockIdx.y, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, q4 = lane >> 4, c16 = lane & 15;
  const int KT = d >> 5, per = (KT + PF_CHUNKS - 1) / PF_CHUNKS, k1 = (chunk + 1) * per < KT ? (chunk + 1) * per : KT;
  const int row = 16 * rt + c16;
  __shared__ float red[4][16];
  float sq = 0.f;
  for (int kt = chunk * per + wave; kt < k1; kt += 4) {
    const int col = 32 * kt + 8 * q4;
    u32x4 out = {0u, 0u, 0u, 0u};
    if (row < M) {
      f32x4 *xp = reinterpret_cast<f32x4 *>(x + (size_t)row * d + col);
      f32x4 x0 = xp[0], x1 = xp[1];
      if (S > 0) {
        f32x4 y0 = {0.f, 0.f, 0.f, 0.f}, y1 = y0;
#pragma unroll
        for (int s = 0; s < S; ++s) {
          const f32x4 *pp = reinterpret_cast<const f32x4 *>(part + ((size_t)s * M + row) * d + col);
          y0 += pp[0];
          y1 += pp[1];
        }
        x0 += y0;
        x1 += y1;
        xp[0] = x0;
        xp[1] = x1;
      }
      const f32x4 *gp = reinterpret_cast<const f32x4 *>(gain + col);
      const f32x4 g0 = gp[0], g1 = gp[1];
#pragma unroll
      for (int i = 0; i < 4; ++i) sq += x0[i] * x0[i] + x1[i] * x1[i];
      out = u32x4{pack_f16(x0[0] * g0[0], x0[1] * g0[1]), pack_f16(x0[2] * g0[2], x0[3] * g0[3]),
                  pack_f16(x1[0] * g1[0], x1[1] * g1[1]), pack_f16(x1[2] * g1[2], x1[3] * g1[3])};
    }
    *(u32x4 *)((uint8_t *)A + (((size_t)kt * RT + rt) * 64 + lane) * 16) = out;
  }
  sq += __shfl_xor(sq, 16, 64);
  sq += __shfl_xor(sq, 32, 64);
  if (q4 == 0) red[wave][c16] = sq;
  __syncthreads();
  if (threadIdx.x < 16 && 16 * rt + (int)threadIdx.x < M)
    ss[(size_t)(16 * rt + threadIdx.x) * PF_CHUNKS + chunk] = (red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x]);
}

// Causal attention over cache rows 0 .. L0 + row (Section 4.4's plain causal mask).  A workgroup takes four consecutive
// (row tile, q head) pairs of one kv head (the heads of a row tile are neighbours), a wave one of them; blocks of 64 keys of
// K and V go through LDS once for all four.  The products and the running softmax are the block kernel's.  Output: operand
// fragments of the O projection.
// Bound: the vector instructions of the softmax beside the products (about 600 cycles of the former, 512 of the latter
// per wave and 64 keys).  Four waves share a K/V block because a wave of its own took 16 KB from L2 for 32 keys and 16
// rows, four times what its products take at 64 bytes a cycle; 64 keys at a time halve the maxima, the barriers and the
// branches of 32 (26 -> 23 us and 70 -> 62 us at the two sizes below); a wave takes one tile and not two (36 us): two
// tiles leave one workgroup per CU and the longest rows last.  The running maximum's lanes are compared without LDS
// (v_permlane swaps), the sums stay per lane until the end, and the output is rescaled only when a maximum moved.
// Measured per layer (7B shape): 1023 rows at 0 69 -> 23 us, 1024 rows at 1000 .. 3000 231 -> 62 us (mean).
template <int DH, bool F16>
__device__ __forceinline__ void pf_attn_body(LDS_AS uint8_t *lds, const uint16_t *Q, const uint16_t *Kc, const uint16_t *Vc, uint16_t *out, int M, int RT, int RTr,
                                             int L0, int Hq, int Hkv) {  // RT: row tiles the fragment buffers are laid out for; RTr: tiles that hold rows
  constexpr int KT = DH / 32, DT = DH / 16;
  constexpr int NB = PF_KEYS / 32;                                  // the cache's 32-key blocks of a stage
  constexpr int ROWB = DH * 2, HALF = PF_KEYS * ROWB, STAGE = 2 * HALF;  // a stage: K rows, then V blocks
  constexpr int LPW = HALF / 1024 / 4;                              // requests of a wave per half stage
  using v8 = std::conditional_t<F16, f16x8, bf16x8>;
  auto mma = [](v8 x, v8 y, f32x4 c) {
    if constexpr (F16) return __builtin_amdgcn_mfma_f32_16x16x32_f16(x, y, c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, y, c, 0, 0, 0);
  };
  const int wave = uni((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63, q4 = lane >> 4, c16 = lane & 15;
  const int g = Hq / Hkv, n_tile = g * RTr, n_task = (n_tile + 3) / 4;
  const int kvh = uni((int)blockIdx.x % Hkv), w0 = uni((n_task - 1 - (int)blockIdx.x / Hkv) * 4);  // (the longest rows first)
  const unsigned lds0 = (unsigned)(uintptr_t)lds;
  const int last_row = L0 + M - 1, last_tile = n_tile - 1;
  auto last_key = [&](int rt) { return L0 + 16 * rt + 15 < last_row ? L0 + 16 * rt + 15 : last_row; };  // last one that a row of the tile sees
  auto blocks_of = [&](int rt) { return last_key(rt) / PF_KEYS + 1; };                                  // blocks that hold a visible key
  const int nkb = uni(blocks_of((w0 + 3 < last_tile ? w0 + 3 : last_tile) / g));
  // K half: row-major [key][DH], the 16-byte pieces of a row permuted by the key so that sixteen keys' equal pieces lie in
  // different banks; V half: the cache's own blocks.  The last block may reach past the cache's last 32-key block: those
  // requests repeat it (no row of it is visible).
  auto swz = [](int key) { return DH == 128 ? key & 15 : (key >> 1) & 7; };
  __amdgpu_buffer_rsrc_t rk = rsrc_of(Kc), rv = rsrc_of(Vc);
  constexpr int KPI = 1024 / ROWB, PPR = ROWB / 16;  // keys a K request brings, pieces per key
  constexpr int RPB = 32 * ROWB / 1024;              // requests per 32-key block
  const int top_block = last_row >> 5;
  const unsigned k_lane = (unsigned)((lane / PPR) * Hkv * ROWB), v_lane = (unsigned)(c16 * 64 + q4 * 16);
  int nx_kb = 0;
  unsigned nx_slot = 0;
  auto request = [&]() {
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
      const int n = wave * LPW + i;  // request of the half stage: part n % RPB of its 32-key block n / RPB
      int blk = nx_kb * NB + n / RPB;
      blk = blk < top_block ? blk : top_block;
      const int key0 = (n % RPB) * KPI;
      const unsigned k_off = k_lane + (unsigned)(((lane % PPR) ^ swz(key0 + lane / PPR)) * 16);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rk, (LDS_AS void *)(uintptr_t)(lds0 + nx_slot + (unsigned)n * 1024u), 16, k_off,
                                               uni((unsigned)((blk * 32 + key0) * Hkv + kvh) * (unsigned)ROWB), 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rv, (LDS_AS void *)(uintptr_t)(lds0 + nx_slot + (unsigned)HALF + (unsigned)n * 1024u), 16, v_lane,
                                               uni((unsigned)(blk * Hkv + kvh) * (unsigned)(32 * ROWB) + (unsigned)(n % RPB) * 1024u), 0, 0);
    }
    nx_slot = nx_slot ? 0u : (unsigned)STAGE;
    if (nx_kb + 1 < nkb) ++nx_kb;  // (past the end the last one is requested again and never used)
  };
  const int t0 = w0 + wave, t = t0 < last_tile ? t0 : last_tile;  // (a wave without a tile repeats the last one and drops it)
  const int rt = t / g, h = kvh * g + t % g;
  const int row = 16 * rt + c16, last = L0 + (row < M ? row : M - 1);  // this lane's query row (as a column of the scores), its last visible key
  v8 q[KT];
#pragma unroll
  for (int kt = 0; kt < KT; ++kt) q[kt] = *(const v8 *)(Q + ((((size_t)h * RT + rt) * KT + kt) * 64 + lane) * 8);
  request();
  const int last_t = uni(last_key(rt)), nkb_w = uni(blocks_of(rt)), full = uni((L0 + 16 * rt + 1) / PF_KEYS);  // blocks 0 .. full - 1 are visible to every row of the tile
  f32x4 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -1e30f, l_run = 0.f;
  for (int kb = 0; kb < nkb; ++kb) {
    wait_vmcnt<0>();
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_barrier();  // everybody's part of the stage is in, and nobody reads the stage before any more
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    request();
    if (kb < nkb_w) {
      const unsigned base = lds0 + (unsigned)((kb & 1) * STAGE);
      f32x4 sc[2 * NB];
#pragma unroll
      for (int n = 0; n < 2 * NB; ++n) sc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int n = 0; n < 2 * NB; ++n) {
          const v8 kf = __builtin_bit_cast(v8, *(LDS_AS const u32x4 *)(uintptr_t)(base + (unsigned)((16 * n + c16) * ROWB + ((4 * kt + q4) ^ swz(c16)) * 16)));
          sc[n] = mma(kf, q[kt], sc[n]);
        }
      if (kb >= full) {
#pragma unroll
        for (int n = 0; n < 2 * NB; ++n)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (kb * PF_KEYS + 16 * n + 4 * q4 + i > last) sc[n][i] = -INFINITY;
      }
      float mx = sc[0][0];
#pragma unroll
      for (int n = 0; n < 2 * NB; ++n)
#pragma unroll
        for (int i = 0; i < 4; ++i) mx = fmaxf(mx, sc[n][i]);
      mx = max_q4(mx);
      if (__any(mx > m_run)) {  // (otherwise the factor is one in every lane)
        const float m_new = fmaxf(m_run, mx);
        const float corr = __builtin_amdgcn_exp2f((m_run - m_new) * LOG2E);
        m_run = m_new;
        l_run *= corr;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[dt] *= corr;
      }
      const float mb = m_run * LOG2E;
      v8 pb[NB];
#pragma unroll
      for (int n = 0; n < NB; ++n) {
        float pr[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          pr[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[2 * n + (i >> 2)][i & 3], LOG2E, -mb));
          l_run += pr[i];  // (this lane's keys; added over the lanes at the end)
        }
        pb[n] = __builtin_bit_cast(v8, u32x4{pack_p<F16>(pr[0], pr[1]), pack_p<F16>(pr[2], pr[3]), pack_p<F16>(pr[4], pr[5]), pack_p<F16>(pr[6], pr[7])});
      }
#pragma unroll
      for (int n = 0; n < NB; ++n) {
        if (n > 0 && kb * PF_KEYS + 32 * n > last_t) break;  // (no row sees these keys, and what they hold need not be finite)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          const v8 vf = __builtin_bit_cast(v8, *(LDS_AS const u32x4 *)(uintptr_t)(base + (unsigned)(HALF + (n * DT + dt) * 1024) + (unsigned)lane * 16u));
          o[dt] = mma(vf, pb[n], o[dt]);
        }
      }
    }
  }
  wait_vmcnt<0>();  // (the request past the last block lands before the LDS is given back)
  l_run = sum_q4(l_run);
  if (t0 <= last_tile && row < M) {
    const float inv = 1.0f / l_run;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const int col = h * DH + 16 * dt + 8 * (q4 >> 1);
      *(u32x2 *)((uint8_t *)out + frag_piece(col, row, RT) + 8 * (q4 & 1)) =
          u32x2{pack_f16(o[dt][0] * inv, o[dt][1] * inv), pack_f16(o[dt][2] * inv, o[dt][3] * inv)};
    }
  }
}

template <int DH, bool F16>
__global__ __launch_bounds__(256, 2) void pf_attn_kernel(const uint16_t *Q, const uint16_t *Kc, const uint16_t *Vc, uint16_t *out, int M, int RT, int RTr,
                                                         int L0, int Hq, int Hkv) {
  __shared__ __attribute__((aligned(1024))) uint8_t pf_kv[4 * PF_KEYS * DH * 2];
  pf_attn_body<DH, F16>((LDS_AS uint8_t *)pf_kv, Q, Kc, Vc, out, M, RT, RTr, L0, Hq, Hkv);
}

// The length that the chunk starts at, x[row] = E[tok[row]] (eight elements per thread at a time), and cos, sin of position L0 + row for every RoPE pair (double
// precision angles, as the block kernel's table); one workgroup per row.
__global__ __launch_bounds__(256) void pf_embed_kernel(const uint16_t *E, const int32_t *tok, int V, int d, int f16, float *x, float *cs, int half, int L0,
                                                       double theta, int32_t *L_dev) {
  const int row = blockIdx.x;
  if (row == 0 && threadIdx.x == 0) *L_dev = L0;
  int t = tok[row];
  t = t < 0 ? 0 : (t >= V ? V - 1 : t);
  for (int i = threadIdx.x * 8; i < d; i += 256 * 8) {
    const u32x4 e = *(const u32x4 *)(E + (size_t)t * d + i);
    f32x4 y[2];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const uint16_t b = (uint16_t)(e[k >> 1] >> (16 * (k & 1)));
      y[k >> 2][k & 3] = f16 ? (float)__builtin_bit_cast(_Float16, b) : __uint_as_float((uint32_t)b << 16);
    }
    f32x4 *xp = reinterpret_cast<f32x4 *>(x + (size_t)row * d + i);
    xp[0] = y[0];
    xp[1] = y[1];
  }
  for (int i = threadIdx.x; i < half; i += 256) {
    const double inv = exp2(-(double)i / (double)half * log2(theta));
    double s, c;
    sincos((double)(L0 + row) * inv, &s, &c);
    cs[((size_t)row * half + i) * 2] = (float)c;
    cs[((size_t)row * half + i) * 2 + 1] = (float)s;
  }
}

// ---- host side ----------------------------------------------------------------------------------------
template <int MODE, int WM, int WN, int NTW, int NS, int NM = 4>
static int pf_launch_tile(const PfGemm &p, hipStream_t s, bool prepare) {
  constexpr int bytes = NS * (NM * WM + WN * NTW) * 1024 + NM * WM * 64;
  static_assert(bytes <= 160 * 1024, "LDS of one CU");
  if (prepare) {
    LA_HIP(hipFuncSetAttribute((const void *)pf_tile_kernel<MODE, WM, WN, NTW, NS, NM>, hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
    return LA_OK;
  }
  const int n_cg = ceil_div(p.ntiles - p.t_first, WN * NTW), RB = ceil_div(ceil_div(p.M, 16), NM * WM);
  pf_tile_kernel<MODE, WM, WN, NTW, NS, NM><<<(RB * p.S * n_cg + 7) / 8 * 8, 64 * WM * WN, bytes, s>>>(p);
  LA_HIP(hipGetLastError());
  return LA_OK;
}
template <int MODE>
static int pf_launch_tile(int tile, const PfGemm &p, hipStream_t s, bool prepare) {
  switch (tile) {
  case 0: return pf_launch_tile<MODE, 4, 2, 7, 5>(p, s, prepare);
  case 1: return pf_launch_tile<MODE, 4, 2, 5, 6>(p, s, prepare);
  case 2: return pf_launch_tile<MODE, 4, 2, 4, 6>(p, s, prepare);
  case 3: return pf_launch_tile<MODE, 2, 4, 3, 6>(p, s, prepare);
  case 4: return pf_launch_tile<MODE, 2, 2, 4, 4>(p, s, prepare);
  default: return pf_launch_tile<MODE, 2, 2, 2, 6>(p, s, prepare);
  }
}

// The tiles that are cut to the prompt's rows (pf_qkv_rows, pf_part_rows, pf_gateup_rows): `rows` row tiles x 6, 8 or 7 columns with a wave per
// column tile, or 10 and 12 x 14.  The narrow ones take as many stages as let two workgroups into a CU's LDS: more change nothing.
constexpr int pf_stages(int frags) { return 78 / frags; }
template <int MODE, int ROWS>
static int pf_launch_rows(const PfGemm &p, hipStream_t s, bool prepare) {
  if constexpr (MODE == PF_QKV) return pf_launch_tile<MODE, 1, 6, 1, pf_stages(ROWS + 6), ROWS>(p, s, prepare);
  else if constexpr (MODE == PF_PART) return pf_launch_tile<MODE, 1, 8, 1, pf_stages(ROWS + 8), ROWS>(p, s, prepare);
  else if constexpr (ROWS == 10) return pf_launch_tile<MODE, 2, 2, 7, 6, 5>(p, s, prepare);
  else if constexpr (ROWS == 12) return pf_launch_tile<MODE, 4, 2, 7, 6, 3>(p, s, prepare);
  else return pf_launch_tile<MODE, 1, 7, 1, pf_stages(ROWS + 7), ROWS>(p, s, prepare);
}
template <int MODE>
static int pf_launch_rows(const PfGemm &p, int rows, hipStream_t s, bool prepare) {
  if constexpr (MODE == PF_QKV) {
    if (rows == 3) return pf_launch_rows<MODE, 3>(p, s, prepare);
    if (rows == 4) return pf_launch_rows<MODE, 4>(p, s, prepare);
  }
  if constexpr (MODE == PF_GATEUP) {
    if (rows == 10) return pf_launch_rows<MODE, 10>(p, s, prepare);
    if (rows == 12) return pf_launch_rows<MODE, 12>(p, s, prepare);
  }
  switch (rows) {
  case 5: return pf_launch_rows<MODE, 5>(p, s, prepare);
  case 6: return pf_launch_rows<MODE, 6>(p, s, prepare);
  case 7: return pf_launch_rows<MODE, 7>(p, s, prepare);
  default: return pf_launch_rows<MODE, 8>(p, s, prepare);
  }
}

template <int MT, int NS>
static int pf_launch_qkv_few(const PfGemm &p, hipStream_t s, bool prepare) {
  constexpr int bytes = 4 * MT * 2 * 1024 + MT * 64;
  if (prepare) {
    LA_HIP(hipFuncSetAttribute((const void *)pf_qkv_few_kernel<MT, NS>, hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
    return LA_OK;
  }
  pf_qkv_few_kernel<MT, NS><<<ceil_div(p.ntiles - p.t_first, 2), 256, bytes, s>>>(p);
  LA_HIP(hipGetLastError());
  return LA_OK;
}
static int pf_launch_qkv_few(const PfGemm &p, int row_tiles, hipStream_t s, bool prepare) {
  switch (row_tiles) {
  case 5: return pf_launch_qkv_few<5, 4>(p, s, prepare);
  case 6: return pf_launch_qkv_few<6, 4>(p, s, prepare);
  case 7: return pf_launch_qkv_few<7, 3>(p, s, prepare);
  default: return pf_launch_qkv_few<8, 3>(p, s, prepare);
  }
}

template <int MODE>
static int pf_launch_gemm(PfGemm p, hipStream_t s, const char *name, int cus, int part_rows = 0, int *S = nullptr) {
  ProfScope ps(name, s);
  static_assert(R_NW == 4, "pf_qkv_few_kernel's waves take the k-tiles as they lie for four MFMA waves");
  const PfRoute r = pf_route((PfMode)MODE, PfProduct{p.RT, p.M, p.KT, p.ntiles - p.t_first, p.d}, part_rows, cus);
  p.S = r.S;
  if (S) *S = r.S;
  if (MODE == PF_QKV && r.few) return pf_launch_qkv_few(p, r.few, s, false);
  if (r.rows) return pf_launch_rows<MODE>(p, r.rows, s, false);
  return pf_launch_tile<MODE>(r.tile, p, s, false);
}

static int pf_launch_norm(int S, float *x, const float *part, const float *gain, int M, int d, int RT, float *ss, uint16_t *A, hipStream_t s) {
  ProfScope ps("pf_norm", s);
  const dim3 grid(RT, PF_CHUNKS);
  switch (S) {
  case 0: pf_norm_kernel<0><<<grid, 256, 0, s>>>(x, part, gain, M, d, RT, ss, A); break;
  case 1: pf_norm_kernel<1><<<grid, 256, 0, s>>>(x, part, gain, M, d, RT, ss, A); break;
  case 2: pf_norm_kernel<2><<<grid, 256, 0, s>>>(x, part, gain, M, d, RT, ss, A); break;
  case 3: pf_norm_kernel<3><<<grid, 256, 0, s>>>(x, part, gain, M, d, RT, ss, A); break;
  case 4: pf_norm_kernel<4><<<grid, 256, 0, s>>>(x, part, gain, M, d, RT, ss, A); break;
  case 5: pf_norm_kernel<5><<<grid, 256, 0, s>>>(x, part, gain, M, d, RT, ss, A); break;
  case 6: pf_norm_kernel<6><<<grid, 256, 0, s>>>(x, part, gain, M, d, RT, ss, A); break;
  case 7: pf_norm_kernel<7><<<grid, 256, 0, s>>>(x, part, gain, M, d, RT, ss, A); break;
  default: pf_norm_kernel<8><<<grid, 256, 0, s>>>(x, part, gain, M, d, RT, ss, A); break;
  }
  LA_HIP(hipGetLastError());
  return LA_OK;
}

template <int DH, bool F16>
static int pf_launch_attn(const PfBuffers &b, const PfGemm &p, int M, int RT, int RTr, hipStream_t s) {
  ProfScope ps("pf_attn", s);
  pf_attn_kernel<DH, F16><<<p.Hkv * ceil_div(p.Hq / p.Hkv * RTr, 4), 256, 0, s>>>(b.Q, p.Kc, p.Vc, b.attn, M, RT, RTr, p.L0, p.Hq, p.Hkv);
  LA_HIP(hipGetLastError());
  return LA_OK;
}

// One allocation for all buffers of a set (eight took 0.4 ms of the first prompt).  They need no clearing: what the products
// read of rows past the prompt's end only reaches rows past its end.  The thread's capture mode is relaxed meanwhile, so that
// a first prompt may be captured into a graph (its buffers are the model's, not the graph's) and does not end a capture of
// another thread.  No memory: b stays empty, and that is no error.
static int pf_alloc(la_model *m, int most, int least, PfBuffers &b) {
  const la_model_desc &d = m->d;
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  const bool relaxed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
  int rc = LA_OK;
  for (int i = 0; !rc && i < PF_N_TILES; ++i) {
    rc = pf_launch_tile<PF_QKV>(i, PfGemm{}, nullptr, true);
    if (!rc) rc = pf_launch_tile<PF_PART>(i, PfGemm{}, nullptr, true);
    if (!rc) rc = pf_launch_tile<PF_GATEUP>(i, PfGemm{}, nullptr, true);
  }
  for (int i = 5; !rc && i <= 8; ++i) rc = pf_launch_qkv_few(PfGemm{}, i, nullptr, true);
  for (int i = 3; !rc && i <= 8; ++i) rc = pf_launch_rows<PF_QKV>(PfGemm{}, i, nullptr, true);
  for (int i = 5; !rc && i <= 8; ++i) rc = pf_launch_rows<PF_PART>(PfGemm{}, i, nullptr, true);
  for (int i : {5, 6, 7, 8, 10, 12})
    if (!rc) rc = pf_launch_rows<PF_GATEUP>(PfGemm{}, i, nullptr, true);
  uint8_t *p = nullptr;
  if (!rc) {
    const PfLayout l = pf_fit(PfDims{(size_t)d.d_model, (size_t)m->qdim(), (size_t)d.head_dim, (size_t)d.d_ffn}, most, least,
                              [&](size_t bytes) { return (p = (uint8_t *)dalloc(bytes)) != nullptr; });
    if (p)
      b = PfBuffers{p, l.rows, l.part_rows, (float *)(p + l.x), (float *)(p + l.part), (float *)(p + l.ss), (float *)(p + l.cs),
                    (uint16_t *)(p + l.A), (uint16_t *)(p + l.Q), (uint16_t *)(p + l.attn), (uint16_t *)(p + l.act)};
  }
  if (!rc && !p) (void)hipGetLastError();  // (the next launch's check would report the failed allocation)
  if (relaxed) (void)hipThreadExchangeStreamCaptureMode(&mode);
  return rc;
}

static PfBuffers &pf_buffers(MfmaModel *f) { return f->pf.base ? f->pf : f->pf_few; }

// *rows: of a chunk of a prompt of n tokens, its buffers allocated; 0: the prompt goes through the block kernel (it is short,
// the model has no large-M path, or the card has no memory left for the buffers).
int mfma_prefill_rows(la_model *m, int n, int *rows) {
  MfmaModel *f = m->mf;
  *rows = 0;
  if (!f || !f->use_r || !m->embed || n < PF_MIN) return LA_OK;
  for (int l = 0; l < m->d.n_layers; ++l) LA_REQUIRE(m->layers[l].set, LA_EINVAL, "layer %d has no weights", l);
  int rc = LA_OK;
  if (!f->pf.base && n >= PF_LONG) rc = pf_alloc(m, PF_ROWS, f->pf_few.base ? 2 * PF_LONG : PF_LONG, f->pf);
  if (!rc && !f->pf.base && !f->pf_few.base) rc = pf_alloc(m, PF_LONG, PF_LONG, f->pf_few);
  *rows = rc ? 0 : pf_buffers(f).rows;
  return rc;
}

// One prompt chunk of M tokens (as many as mfma_prefill_rows says at most) at positions L0 .. L0 + M - 1 through every layer (the caller sets the cache
// length afterwards).
int mfma_prefill_chunk(la_model *m, la_kv *kv, const int32_t *tok, int M, int L0, hipStream_t s) {
  MfmaModel *f = m->mf;
  const la_model_desc &d = m->d;
  LA_REQUIRE(f->use_r, LA_EINVAL, "the large-M prompt pass reads the register-streaming kernel's weight layout");
  PfBuffers &b = pf_buffers(f);
  LA_REQUIRE(M <= b.rows, LA_EINVAL, "%d rows in buffers of %d", M, b.rows);
  const int RT = (M + 63) / 64 * 4, RTr = (M + 15) / 16, half = d.head_dim / 2, f16 = d.dtype == LA_F16;
  {
    ProfScope ps("pf_embed", s);
    pf_embed_kernel<<<M, 256, 0, s>>>((const uint16_t *)m->embed, tok, d.vocab, d.d_model, f16, b.x, b.cs, half, L0, (double)d.rope_theta, kv->L_dev);
  }
  LA_HIP(hipGetLastError());
  const GemmPlan *plans[4] = {&f->p_qkv, &f->p_o, &f->p_gu, &f->p_down};
  int S_down = 0;  // slices of the products that x has not taken in yet
  for (int l = 0; l < d.n_layers; ++l) {
    auto gemm_args = [&](int gi, const uint16_t *A) {
      PfGemm p{};
      p.wstream = f->wstream;
      p.cu_bytes = f->cu_bytes;
      p.frag0 = (unsigned)l * f->seg_frags;
      p.G = f->n_wgs;
      p.NW = R_NW;
      p.n_prev = gi;
      for (int i = 0; i < gi; ++i) {
        p.prev_ntiles[i] = plans[i]->ntiles;
        p.prev_KT[i] = plans[i]->KT;
      }
      p.ntiles = plans[gi]->ntiles;
      p.KT = plans[gi]->KT;
      p.A = A;
      p.S = 1;
      p.RT = RT;
      p.M = M;
      p.part = b.part;
      p.d = d.d_model;
      p.ss = b.ss;
      p.inv_d = 1.0f / (float)d.d_model;
      p.eps = d.rms_eps;
      p.cs = b.cs;
      p.Kc = (uint16_t *)kv->K + (size_t)l * kv->layer_elems();
      p.Vc = (uint16_t *)kv->V + (size_t)l * kv->layer_elems();
      p.Q = b.Q;
      p.L0 = L0;
      p.Hq = d.n_q_heads;
      p.Hkv = d.n_kv_heads;
      p.dh = d.head_dim;
      p.f16 = f16;
      p.act = b.act;
      return p;
    };
    const bool last = l + 1 == d.n_layers;  // its K and V rows are all that anybody reads: the pass ends with them
    int rc, S_o = 0;
    if ((rc = pf_launch_norm(S_down, b.x, b.part, m->layers[l].g_attn, M, d.d_model, RT, b.ss, b.A, s))) return rc;
    PfGemm p = gemm_args(0, b.A);
    if (last) p.t_first = m->qdim() / 16;
    if ((rc = pf_launch_gemm<PF_QKV>(p, s, "pf_gemm_qkv", f->n_wgs))) return rc;
    if (last) break;
    if (d.head_dim == 128) rc = f16 ? pf_launch_attn<128, true>(b, p, M, RT, RTr, s) : pf_launch_attn<128, false>(b, p, M, RT, RTr, s);
    else rc = f16 ? pf_launch_attn<64, true>(b, p, M, RT, RTr, s) : pf_launch_attn<64, false>(b, p, M, RT, RTr, s);
    if (rc) return rc;
    if ((rc = pf_launch_gemm<PF_PART>(gemm_args(1, b.attn), s, "pf_gemm_o", f->n_wgs, b.part_rows, &S_o))) return rc;
    if ((rc = pf_launch_norm(S_o, b.x, b.part, m->layers[l].g_mlp, M, d.d_model, RT, b.ss, b.A, s))) return rc;
    if ((rc = pf_launch_gemm<PF_GATEUP>(gemm_args(2, b.A), s, "pf_gemm_gateup", f->n_wgs))) return rc;
    if ((rc = pf_launch_gemm<PF_PART>(gemm_args(3, b.act), s, "pf_gemm_down", f->n_wgs, b.part_rows, &S_down))) return rc;
  }
  LA_HIP(hipGetLastError());
  return LA_OK;
}

}  // namespace la
