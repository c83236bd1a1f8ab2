// The plain kernels of small layers (fp32 arithmetic; included by la_generic.hip): five launches a layer, each of which requests
// everything it reads before it waits for any of it.  Such a launch is a chain of memory latencies around next to no arithmetic:
// its loads in turns, and rotation and cache rows as a launch of their own, were half of a step of the tiny shape.
#pragma once
#include "la_device.h"
#include "la_internal.h"

namespace la {

constexpr int PL_WAVES = 8, PL_THREADS = 64 * PL_WAVES;
typedef float pl_f4 __attribute__((ext_vector_type(4)));
typedef unsigned pl_u4 __attribute__((ext_vector_type(4)));
constexpr unsigned PL_OOB = 0x80000000u;

// Buffer loads: what lies past a matrix's end comes back as zero, and offsets are 32 bits.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t pl_rsrc(const void *p, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}
template <typename T>
__device__ __forceinline__ float pl_load(__amdgpu_buffer_rsrc_t r, unsigned i) {  // element i
  if constexpr (sizeof(T) == 4) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, i * 4u, 0, 0));
  } else {
    const T v = __builtin_bit_cast(T, (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, i * 2u, 0, 0));
    return load_as_float<T>(&v);
  }
}
// Elements as they are stored, 16 bytes of them or one: turned into floats where they are used.  (Turned behind their load, a load under a condition is
// waited for where the condition ends.)
template <typename T>
__device__ __forceinline__ float pl_value(unsigned bits) {
  if constexpr (sizeof(T) == 4) {
    return __uint_as_float(bits);
  } else {
    const T h = __builtin_bit_cast(T, (uint16_t)bits);
    return load_as_float<T>(&h);
  }
}
template <typename T>
__device__ __forceinline__ float pl_element(const pl_u4 *raw, int i) {
  if constexpr (sizeof(T) == 4) return pl_value<T>(raw[i >> 2][i & 3]);
  else return pl_value<T>(raw[i >> 3][(i >> 1) & 3] >> (16 * (i & 1)));
}
// A rotated channel (lower: of the lower half of its head); products and sum are rounded one by one wherever this is inlined.
__device__ __forceinline__ float rotated(bool lower, float mine, float other, float c, float s) {
#pragma clang fp contract(off)
  const float a = mine * c, b = other * s;
  return lower ? a - b : a + b;
}

enum PlKind { PL_QKV = 0, PL_RESID = 1, PL_GLU = 2, PL_STORE = 3, PL_QKV_FIRST = 4 };

struct PlProduct {
  const float *A;     // [M][lda]
  int lda, M, K;
  const float *gain;  // of the norm: A is x * gain, and the sums are multiplied by its row factor (RESID: none, A as it is)
  float eps;
  const void *W;      // [K][ldw]
  int ldw, N;         // N: columns of the result (GLU: of gate, and as many of up behind them)
  float *out;         // RESID: added to; GLU: the SwiGLU; QKV: q
  int ldo;
  // a block that does not fit the cache behind its length is skipped as a whole: QKV reports it, RESID leaves `out` as it is
  const int32_t *L_dev;
  int max_len;
  int32_t *err, *err_map;
  // QKV: rotation table [row][pair][2], this layer's cache, where the block's rows go
  float *cs;
  void *Kc, *Vc;
  int Hq, Hkv, dh;
  // QKV_FIRST: the table is made, from these
  const int32_t *pos;  // (NULL: the rows follow the length)
  double theta;
};

// cos, sin of pos theta^(-2 i / head_dim), evaluated in double so that the float results are correctly rounded for every position the cache can hold.
__device__ __forceinline__ void rotation(int pos, int i, int half, double theta, float *c, float *s) {
  const double inv = exp2(-(double)i / (double)half * log2(theta));
  double ds, dc;
  sincos((double)pos * inv, &ds, &dc);
  *c = (float)dc;
  *s = (float)ds;
}

// One product.  A workgroup takes 16 columns and all rows of a block (64 rows of a prompt); its eight waves share the contraction, 16 deep at a time (the same
// order as gemm_generic_kernel's), NP slices of it on their way at once, and their sums are added in gemm_generic_kernel's order, an element per thread (but
// where sixteen waves share a contraction, below).
//   QKV: eight channels of the lower half of a head and their rotation partners; rotates, and writes K and V to the cache.
//   GLU: eight channels of gate and the same of up.
//   STORE: the columns as they are (the unembedding).
//   QKV_FIRST: QKV of the first layer of a call, where more waves make the rotation table meanwhile, each workgroup the pairs of its own tile
//   (those of head 0 leave them for the layers behind it): a launch in front of the layers cost 2.9 us, the same work in front of the product 1.5.
//   RESID: a contraction of more than 256 is shared by sixteen waves, three slices each on their way; the upper half's sums are added to the lower half's first.
// Bound: a launch, the weights' way from memory (each is read by one wave) and the sums' through LDS.  Step of the tiny shape (256
// wide, 2 layers, 17 rows): 76.0 -> 62.6 us with these and the attention below; -> 57.9 with the table, the unembedding and the arg-max in
// products of this kind, what an epilogue adds to or rotates by requested with the operands, and K and V of the attention's first piece with q.
// Eight waves / sixteen for RESID, a captured step of two fp32 layers, us at 17 and 64 rows: 688 channels of gate 52.1 / 52.1 and 73.8 / 74.2 (error against 64
// bits 2.5e-7 / 2.4e-7), 512 wide and 2048 channels 85.5 / 83.8 and 136.7 / 131.8, 256 wide and 4096 channels 96.6 / 93.1 and 154.1 / 147.5.  That a product
// has a norm is known when it is compiled: a test at run time cost registers (the sixteen waves' four row tiles 129 of 128, and scratch memory for the last)
// and 3 to 7 % of these steps.  A's rows are loaded 16 bytes at a time wherever they begin (word by word where a row was not a multiple of 16 bytes, or A not
// aligned to them, the unembedding 1024 x 4096 of 64 rows took 39.8 us, 19.3 so, 22.5 with the general product; 254 x 777 11.9, 8.3 and 10.1).
constexpr int pl_waves(int kind, int np) { return kind == PL_RESID && np > 2 ? 2 * PL_WAVES : PL_WAVES; }
template <typename T, int MT, int KIND0, int NP0>
__global__ __launch_bounds__(64 * pl_waves(KIND0, NP0) + (KIND0 == PL_QKV_FIRST ? 64 * MT : 0)) void plain_product_kernel(PlProduct p) {
  constexpr bool FIRST = KIND0 == PL_QKV_FIRST;
  constexpr int KIND = FIRST ? (int)PL_QKV : KIND0, PER = (MT + 1) / 2;  // elements of the result a thread finishes
  constexpr int WV = pl_waves(KIND0, NP0);
  constexpr bool NORM = KIND != PL_RESID;
  constexpr int NP = WV > PL_WAVES ? NP0 / 2 : FIRST && MT > 2 && NP0 > 4 ? 4 : NP0;  // (QKV_FIRST: three waves on a SIMD, 168 registers)
  __shared__ __attribute__((aligned(16))) float part[PL_WAVES * MT * 256];  // [wave][row tile][lane][4]
  __shared__ float sqs[PL_WAVES * 64];
  __shared__ float rot[FIRST ? MT * 16 * 16 : 1];  // [row][pair of the tile][2]
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63, q4 = lane >> 4, c16 = lane & 15;
  const int row0 = 64 * blockIdx.y, t = blockIdx.x, K = p.K, M = p.M - row0 < 64 ? p.M - row0 : 64, per = p.dh >> 4, head = KIND == PL_QKV ? t / per : 0, jj = t - head * per, half = p.dh >> 1;
  // source column (columns past the end read the last one, their results are dropped)
  int col;
  if (KIND == PL_QKV) col = head * p.dh + (c16 < 8 ? 8 * jj + c16 : half + 8 * jj + c16 - 8);
  else if (KIND == PL_GLU) col = (8 * t + (c16 & 7) < p.N ? 8 * t + (c16 & 7) : p.N - 1) + (c16 < 8 ? 0 : p.N);
  else col = 16 * t + c16 < p.N ? 16 * t + c16 : p.N - 1;
  if (FIRST && wave >= PL_WAVES) {
    for (int e = (int)threadIdx.x - PL_THREADS; e < 8 * M; e += 64 * MT) {
      const int row = e >> 3, pair = 8 * jj + (e & 7);
      float c, s;
      rotation(p.pos ? p.pos[row] : *p.L_dev + row0 + row, pair, half, p.theta, &c, &s);
      rot[2 * e] = c;
      rot[2 * e + 1] = s;
      if (head == 0) {
        p.cs[((size_t)(row0 + row) * half + pair) * 2] = c;
        p.cs[((size_t)(row0 + row) * half + pair) * 2 + 1] = s;
      }
    }
    __syncthreads();
    return;
  }
  const __amdgpu_buffer_rsrc_t rw = pl_rsrc(p.W, (size_t)K * p.ldw * sizeof(T)), ra = pl_rsrc(p.A + (size_t)row0 * p.lda, (size_t)M * p.lda * 4), rg = pl_rsrc(p.gain, (size_t)K * 4);
  const bool quads = K % 4 == 0;
  constexpr bool LEN = KIND == PL_QKV || KIND == PL_RESID;
  int L = 0;
  if (LEN) L = *p.L_dev;
  // what the end adds to or rotates by: behind the sums it was a trip to memory of its own
  float was[PER][2];
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int it = (int)threadIdx.x + PL_THREADS * u, row = 16 * (it >> 8) + ((it >> 4) & 15), c = it & 15;
    was[u][0] = was[u][1] = 0.f;
    if (KIND == PL_RESID && threadIdx.x < PL_THREADS && row < M && 16 * t + c < p.N) was[u][0] = p.out[(size_t)(row0 + row) * p.ldo + 16 * t + c];
    if (KIND == PL_QKV && !FIRST && row < M && head < p.Hq + p.Hkv) {
      const float *cs = p.cs + ((size_t)(row0 + row) * half + 8 * jj + (c & 7)) * 2;
      was[u][0] = cs[0];
      was[u][1] = cs[1];
    }
  }
  pl_f4 acc[MT];
  float sq[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    acc[mt] = pl_f4{0.f, 0.f, 0.f, 0.f};
    sq[mt] = 0.f;
  }
  for (int k0 = 16 * wave; k0 < K; k0 += 16 * WV * NP) {
    pl_f4 b[NP], g[NP], x[NP][MT];
#pragma unroll
    for (int n = 0; n < NP; ++n) {
      const int k = k0 + 16 * WV * n + 4 * q4;
      if (k0 + 16 * WV * n >= K) continue;
#pragma unroll
      for (int j = 0; j < 4; ++j) b[n][j] = pl_load<T>(rw, (unsigned)((k + j) * p.ldw + col));
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const unsigned o = (unsigned)((16 * mt + c16) * p.lda + k) * 4u;  // (rows past the end: zeros)
        if (quads || k0 + 16 * WV * n + 16 <= K) {  // (16 bytes from any element on: such loads want addresses in whole words)
          x[n][mt] = __builtin_bit_cast(pl_f4, __builtin_amdgcn_raw_buffer_load_b128(ra, k < K ? o : PL_OOB, 0, 0));
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) x[n][mt][j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ra, k + j < K ? o + 4u * j : PL_OOB, 0, 0));
        }
      }
      if (NORM) {
#pragma unroll
        for (int j = 0; j < 4; ++j) g[n][j] = pl_load<float>(rg, (unsigned)(k + j));
      }
    }
#pragma unroll
    for (int n = 0; n < NP; ++n) {
      if (k0 + 16 * WV * n >= K) continue;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float v = x[n][mt][j];
          if (NORM) sq[mt] = fmaf(v, v, sq[mt]);
          acc[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(NORM ? v * g[n][j] : v, b[n][j], acc[mt], 0, 0, 0);
        }
    }
  }
  if constexpr (WV > PL_WAVES) {  // the upper half's sums go to the lower half first
    pl_f4 *pp = reinterpret_cast<pl_f4 *>(part) + (size_t)(wave % PL_WAVES) * MT * 64 + lane;
    if (wave >= PL_WAVES)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) pp[mt * 64] = acc[mt];
    __syncthreads();
    if (wave >= PL_WAVES) {
      __syncthreads();
      return;
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] += pp[mt * 64];
  }
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    reinterpret_cast<pl_f4 *>(part)[(wave * MT + mt) * 64 + lane] = acc[mt];
    if (NORM) {
      sq[mt] += __shfl_xor(sq[mt], 16, 64);
      sq[mt] += __shfl_xor(sq[mt], 32, 64);
      if (q4 == 0) sqs[wave * 64 + 16 * mt + c16] = sq[mt];
    }
  }
  __syncthreads();
  if (LEN && (L < 0 || L + p.M > p.max_len)) {
    if (KIND == PL_QKV && t == 0 && row0 == 0 && threadIdx.x == 0) {  // the device word, and the host's mapped word (read without synchronising)
      *p.err = 1;
      __hip_atomic_store(p.err_map, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    return;
  }
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int it = (int)threadIdx.x + PL_THREADS * u;
    if (it >= 256 * MT) break;
    const int mt = it >> 8, r16 = (it >> 4) & 15, row = 16 * mt + r16, c = it & 15;
    const float *pp = part + (size_t)(mt * 64 + 16 * (r16 >> 2) + c) * 4 + (r16 & 3);
    constexpr int HALF = PL_WAVES / 2, WS = MT * 256;
    float v = pp[HALF * WS] + pp[0];
#pragma unroll
    for (int w = 1; w < HALF; ++w) v += pp[(w + HALF) * WS] + pp[w * WS];
    if (NORM) {
      float q = sqs[row];
#pragma unroll
      for (int w = 1; w < PL_WAVES; ++w) q += sqs[w * 64 + row];
      v *= 1.0f / sqrtf(q / (float)K + p.eps);
    }
    const float other = KIND == PL_RESID || KIND == PL_STORE ? 0.f : __shfl_xor(v, 8, 64);
    if (row >= M) continue;
    if (KIND == PL_QKV) {
      const int ch = c < 8 ? 8 * jj + c : half + 8 * jj + c - 8;
      float y = v;
      if (head < p.Hq + p.Hkv) {
        const float cs = FIRST ? rot[(8 * row + (c & 7)) * 2] : was[u][0], sn = FIRST ? rot[(8 * row + (c & 7)) * 2 + 1] : was[u][1];
        y = rotated(c < 8, v, other, cs, sn);
      }
      if (head < p.Hq) p.out[(size_t)(row0 + row) * p.ldo + head * p.dh + ch] = y;
      else if (head < p.Hq + p.Hkv) store_from_float<T>((T *)p.Kc + ((size_t)(L + row0 + row) * p.Hkv + head - p.Hq) * p.dh + ch, y);
      else store_from_float<T>((T *)p.Vc + ((size_t)(L + row0 + row) * p.Hkv + head - p.Hq - p.Hkv) * p.dh + ch, y);
    } else if (KIND == PL_GLU) {
      if (c < 8 && 8 * t + c < p.N) p.out[(size_t)(row0 + row) * p.ldo + 8 * t + c] = v / (1.0f + expf(-v)) * other;
    } else if (16 * t + c < p.N) {
      p.out[(size_t)(row0 + row) * p.ldo + 16 * t + c] = KIND == PL_STORE ? v : was[u][0] + v;
    }
  }
}

__device__ __forceinline__ float pl_wave_max(float v) {
#pragma unroll
  for (int w = 32; w > 0; w >>= 1) v = fmaxf(v, __shfl_xor(v, w, 64));
  return v;
}
__device__ __forceinline__ float pl_wave_sum(float v) {
#pragma unroll
  for (int w = 32; w > 0; w >>= 1) v += __shfl_xor(v, w, 64);
  return v;
}

// Attention: one workgroup per (row b, query head, 64 channels of the output; larger heads form their scores once per 64 channels).
// The keys go in pieces of 64 to eight shares, piece k to share k % 8, and a wave takes a share: a key per lane for the scores and
// a channel per lane for the output, with the running maximum and sum; the shares are added in order.  A piece's V is requested
// before its scores are formed, the share's next K behind them.  A workgroup has eight waves, or as many as the host's bound on the
// length allows pieces if those are fewer.  That is a matter of time only: accepts that a replayed graph makes leave the bound
// behind the length, and waves then take more than one share each, so that the sums depend on the length alone.
// Bound: a launch and two memory latencies for short contexts, a latency per 512 keys for long ones.
// 17 rows, 4 heads of 64, us a layer (256 threads a workgroup, a key each, 256 keys in turn before): L = 47 6.7 -> 5.0, L = 1000
// 28 -> 12, L = 4000 108 -> 41.
// EARLY: K and V of a wave's first piece are requested beside q and the length (V waited for both before): L = 47 5.7 -> 5.0.  Only where every wave has a
// piece: a captured launch has eight whatever the length, a long prompt's first rows see less than its last, and what such waves request costs
// as much as what is used (captured steps of two layers 256 wide, L = 47: 4 heads, 17 rows 54 us, 64 with all eight pieces requested, 32 heads, 64 rows 168 and 230).
template <typename T, bool EARLY>
__global__ __launch_bounds__(PL_THREADS) void plain_attention_kernel(const float *q, int ldq, int Hq, int Hkv, int dh, const T *Kc, const T *Vc, const int32_t *L_dev,
                                                                     int max_len, int Bp, const uint64_t *vis, float *out) {
  __shared__ __attribute__((aligned(16))) float qs[256], ps[PL_WAVES][64], os[PL_WAVES][64 + 2];
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int n_waves = (int)blockDim.x >> 6, b = blockIdx.x, hq = blockIdx.y, u0 = 64 * blockIdx.z;
  const int kvh = hq / (Hq / Hkv), nkv = Hkv * dh;
  // (rows behind the length are masked whatever they hold, rows behind the cache read as zeros: the first piece needs no length)
  const __amdgpu_buffer_rsrc_t rk = pl_rsrc(Kc, (size_t)max_len * nkv * sizeof(T)), rv = pl_rsrc(Vc, (size_t)max_len * nkv * sizeof(T));
  const int L_mem = *L_dev;
  const uint64_t vb = vis ? vis[b] : 0ull;
  const float scale = 1.0f / sqrtf((float)dh);
  constexpr int PER = 16 / sizeof(T);
  pl_u4 kr[64 / PER];
  unsigned vr[64];
  auto load_k = [&](int ck, int c0) {  // channels c0 .. c0 + 63 of this lane's key
    const unsigned at = (unsigned)((64 * ck + lane) * nkv + kvh * dh + c0);
#pragma unroll
    for (int c = 0; c < 64; c += 16)
      if (c0 + c < dh) {  // (head_dim is a multiple of 16)
#pragma unroll
        for (int n = c / PER; n < (c + 16) / PER; ++n)
          kr[n] = __builtin_bit_cast(pl_u4, __builtin_amdgcn_raw_buffer_load_b128(rk, (at + (unsigned)(n * PER)) * (unsigned)sizeof(T), 0, 0));
      }
  };
  auto load_v = [&](int ck) {  // this lane's channel of the 64 keys
    unsigned at = (unsigned)(64 * ck * nkv + kvh * dh + (u0 + lane < dh ? u0 + lane : 0)) * (unsigned)sizeof(T);
#pragma unroll
    for (int j = 0; j < 64; ++j) {
      if constexpr (sizeof(T) == 4) vr[j] = __builtin_amdgcn_raw_buffer_load_b32(rv, at, 0, 0);
      else vr[j] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rv, at, 0, 0);
      at += (unsigned)nkv * (unsigned)sizeof(T);
      asm volatile("" : "+v"(at));  // (one register, not 64 offsets kept ahead)
    }
  };
  // q first: loads come back in order
  float q_in[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) q_in[u] = (int)(threadIdx.x + u * blockDim.x) < dh ? q[(size_t)b * ldq + hq * dh + threadIdx.x + u * blockDim.x] : 0.f;
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (EARLY) {
    load_k(wave, 0);
    __builtin_amdgcn_sched_barrier(0);
    load_v(wave);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if ((int)(threadIdx.x + u * blockDim.x) < dh) qs[threadIdx.x + u * blockDim.x] = q_in[u];
  const int L = __builtin_amdgcn_readfirstlane(L_mem);
  if (L < 0 || L + Bp > max_len) return;
  // a prompt (vis = NULL) is causal, and what is behind a row is not looked at: a piece that it sees nothing of adds nothing
  const int total = vis ? L + Bp : L + b + 1, seen = vis ? L : total, n_chunks = (total + 63) >> 6, n_shares = n_chunks < PL_WAVES ? n_chunks : PL_WAVES;
  if (!EARLY && wave < n_shares) load_k(wave, 0);
  __syncthreads();
  for (int share = wave; share < n_shares; share += n_waves) {
    float m = -INFINITY, l = 0.f;
    pl_f4 o = {0.f, 0.f, 0.f, 0.f};  // (every fourth key each)
    if (share != wave) load_k(share, 0);
    for (int ck = share; ck < n_chunks; ck += PL_WAVES) {
      const int key = 64 * ck + lane;
      if (!EARLY || ck != wave) load_v(ck);
      float s0 = 0.f, s1 = 0.f;
      for (int c0 = 0; c0 < dh; c0 += 64) {
        if (c0 > 0) load_k(ck, c0);
#pragma unroll
        for (int c = 0; c < 64; c += 16)
          if (c0 + c < dh) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int e = 0; e < 16; e += 4) {
              const pl_f4 qv = *reinterpret_cast<const pl_f4 *>(qs + c0 + c + e);
              s0 = fmaf(qv[0], pl_element<T>(kr, c + e), s0);
              s1 = fmaf(qv[1], pl_element<T>(kr, c + e + 1), s1);
              s0 = fmaf(qv[2], pl_element<T>(kr, c + e + 2), s0);
              s1 = fmaf(qv[3], pl_element<T>(kr, c + e + 3), s1);
            }
          }
      }
      __builtin_amdgcn_sched_barrier(0);
      if (ck + PL_WAVES < n_chunks) load_k(ck + PL_WAVES, 0);
      const bool ok = key < total && (key < seen || ((vb >> (key - L)) & 1ull));
      const float v = ok ? (s0 + s1) * scale : -INFINITY;
      const float m_new = fmaxf(m, pl_wave_max(v));
      const float corr = m == -INFINITY ? 0.f : expf(m - m_new);
      const float p = ok ? expf(v - m_new) : 0.f;
      l = l * corr + pl_wave_sum(p);
      m = m_new;
      o *= corr;
      ps[wave][lane] = p;
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      __builtin_amdgcn_wave_barrier();
      // A probability of zero leaves its V row out: what a row does not see need not be finite.
#pragma unroll
      for (int j = 0; j < 64; j += 4) {
        if (j % 16 == 0) __builtin_amdgcn_sched_barrier(0);
        const pl_f4 pj = *reinterpret_cast<const pl_f4 *>(&ps[wave][j]);
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = fmaf(pj[e], pj[e] != 0.f ? pl_value<T>(vr[j + e]) : 0.f, o[e]);
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    os[share][lane] = ((o[0] + o[1]) + o[2]) + o[3];
    if (lane == 0) {
      os[share][64] = m;
      os[share][65] = l;
    }
  }
  __syncthreads();
  if (wave != 0 || u0 + lane >= dh) return;
  float mm = -INFINITY, ll = 0.f, acc = 0.f;
  for (int w = 0; w < n_shares; ++w) mm = fmaxf(mm, os[w][64]);
  for (int w = 0; w < n_shares; ++w) {
    const float f = os[w][64] == -INFINITY ? 0.f : expf(os[w][64] - mm);
    ll = fmaf(os[w][65], f, ll);
    acc = fmaf(os[w][lane], f, acc);
  }
  out[(size_t)b * (Hq * dh) + hq * dh + u0 + lane] = acc / ll;
}

// ---- host side --------------------------------------------------------------------------------------
template <typename T>
static int plain_attention(const float *q, int ldq, const la_model_desc &d, const T *Kc, const T *Vc, const la_kv *kv, int Bp, const uint64_t *vis, float *out,
                           hipStream_t s) {
  ProfScope ps("plain_attention", s);
  // (a captured launch serves the lengths of its replays, and has every wave)
  const bool captured = stream_captures(s);
  const int pieces = ceil_div(kv->L_bound + Bp, 64), waves = pieces < PL_WAVES && !captured ? pieces : PL_WAVES;
  auto run = [&](auto kernel) {
    kernel<<<dim3(Bp, d.n_q_heads, ceil_div(d.head_dim, 64)), 64 * waves, 0, s>>>(q, ldq, d.n_q_heads, d.n_kv_heads, d.head_dim, Kc, Vc, kv->L_dev, kv->max_len, Bp, vis, out);
  };
  if (!captured && Bp <= LA_MAX_ROWS) run(plain_attention_kernel<T, true>);
  else run(plain_attention_kernel<T, false>);
  LA_HIP(hipGetLastError());
  return LA_OK;
}

template <typename T, int KIND, int NP>
static int plain_product_np(const PlProduct &p, int n_tiles, hipStream_t s) {
  const int MT = p.M < 64 ? ceil_div(p.M, 16) : 4, threads = 64 * pl_waves(KIND, NP) + (KIND == PL_QKV_FIRST ? 64 * MT : 0);
  switch (MT) {
  case 1: plain_product_kernel<T, 1, KIND, NP><<<n_tiles, threads, 0, s>>>(p); break;
  case 2: plain_product_kernel<T, 2, KIND, NP><<<n_tiles, threads, 0, s>>>(p); break;
  case 3: plain_product_kernel<T, 3, KIND, NP><<<n_tiles, threads, 0, s>>>(p); break;
  default: plain_product_kernel<T, 4, KIND, NP><<<dim3(n_tiles, ceil_div(p.M, 64)), threads, 0, s>>>(p); break;
  }
  LA_HIP(hipGetLastError());
  return LA_OK;
}
// (contractions of at most 256 need two slices a wave, and fewer registers)
template <typename T, int KIND>
static int plain_product(const char *name, const PlProduct &p, int n_tiles, hipStream_t s) {
  ProfScope ps(name, s);
  return p.K <= 2 * 16 * PL_WAVES ? plain_product_np<T, KIND, 2>(p, n_tiles, s) : plain_product_np<T, KIND, 6>(p, n_tiles, s);
}

}  // namespace la
