// Any-shape kernels in fp32 arithmetic: the LA_F32 model's compute path, and the path of
// LA_BF16 models whose shape the MFMA kernels do not cover.  These shapes are small (the tiny
// decoder of the test configuration), so what counts is launches: the norms and SwiGLU are part
// of the products, six launches a layer; five (la_plain.h) where layers and heads allow it.
#include <type_traits>

#include "la_device.h"
#include "la_internal.h"
#include "la_plain.h"

namespace la {

__global__ void rope_table_kernel(const int32_t *pos, int Bp, int half, double theta, float *cs) {
  int b = blockIdx.x;
  for (int i = threadIdx.x; i < half; i += blockDim.x)
    rotation(pos[b], i, half, theta, &cs[((size_t)b * half + i) * 2], &cs[((size_t)b * half + i) * 2 + 1]);
}

__device__ __forceinline__ float block_sum(float v, float *red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  float t = 0.f;
  for (int i = 0; i < nw; ++i) t += red[i];
  return t;
}

__device__ __forceinline__ float block_max(float v, float *red) {
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  float t = red[0];
  for (int i = 1; i < nw; ++i) t = fmaxf(t, red[i]);
  return t;
}

// C[M, N] (=|+=) A[M, K] W[K, N] with the fp32 matrix instruction (fp32 operands, products and sums), M <= 64.  A workgroup
// takes 16 columns (WIDE: 64, GLU: 16 of the gate and the same 16 of up) and all rows; its eight waves share the
// contraction, 16 deep at a time, and their sums are added in wave order.  Bound: the latency of the loads; these matrices
// are small, so the columns are cut finely and the contraction is split where one thread per column walked it alone
// (2 layers of the tiny shape, 17 rows: 256 x 512 28 us, 688 x 256 70 us; now 4 - 6 us a launch).
//   gain != NULL: A is x * gain and the sums are multiplied by the row factor 1 / sqrt(mean x^2 + eps) of the norm.
//   GLU: C[M, F] = silu(gate) * up.
//   ADD: C is added to; it stays as it is where M rows behind the length *L_dev do not fit the cache (the block is skipped as a whole).
//   The length is requested behind the contraction, while the waves' sums come together (in front of it it held up the first operands: a
//   forward of two fp32 layers 1280 wide, 17 rows, 150 us against 146, 146 without the look at it).
// A lane's four contraction indices of a turn are consecutive: the k-th matrix instruction of the turn takes the k-th of
// them from every lane, in both operands alike.
enum GemmKind { GEMM_16 = 0, GEMM_WIDE = 1, GEMM_GLU = 2 };
typedef float f4 __attribute__((ext_vector_type(4)));
constexpr int GEMM_WAVES = 8;

template <typename T, int MT, int KIND, bool ADD>
__global__ __launch_bounds__(64 * GEMM_WAVES) void gemm_generic_kernel(const float *A, int lda, const float *gain, float eps, const T *W, int ldw,
                                                                       float *C, int ldc, int M, int K, int N, int vec, const int32_t *L_dev, int max_len) {
  constexpr int CT = KIND == GEMM_WIDE ? 4 : KIND == GEMM_GLU ? 2 : 1, HALF = GEMM_WAVES / 2;
  extern __shared__ __attribute__((aligned(16))) float gemm_lds[];
  f4 *part = reinterpret_cast<f4 *>(gemm_lds);                     // [wave of the lower half][MT][CT][lane]
  float *sqs = gemm_lds + HALF * MT * CT * 64 * 4;           // [wave][16 MT] sums of squares
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, q4 = lane >> 4, c16 = lane & 15;
  const int c0 = blockIdx.x * (KIND == GEMM_WIDE ? 64 : 16);
  // (columns past the end read the last one; their results are dropped)
  int col[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    const int c = KIND == GEMM_WIDE ? c0 + 4 * c16 + ct : c0 + c16;
    col[ct] = (c < N ? c : N - 1) + (KIND == GEMM_GLU && ct == 1 ? N : 0);
  }
  f4 acc[MT][CT];
  float sq[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    sq[mt] = 0.f;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) acc[mt][ct] = f4{0.f, 0.f, 0.f, 0.f};
  }
  const float *ar[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) ar[mt] = A + (size_t)(16 * mt + c16 < M ? 16 * mt + c16 : M - 1) * lda;  // (rows past the end repeat the last)
  for (int k0 = wave * 16; k0 < K; k0 += 16 * GEMM_WAVES) {
    const int k = k0 + 4 * q4;
    f4 a[MT], b[CT];
    float g[4];
    if (k0 + 16 <= K) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const T *w = W + (size_t)(k + j) * ldw;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) b[ct][j] = load_as_float<T>(w + col[ct]);
        g[j] = gain ? gain[k + j] : 1.f;
      }
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        if (vec) {
          a[mt] = *reinterpret_cast<const f4 *>(ar[mt] + k);
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) a[mt][j] = ar[mt][k + j];
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bool in = k + j < K;
        const int kk = in ? k + j : K - 1;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) b[ct][j] = in ? load_as_float<T>(W + (size_t)kk * ldw + col[ct]) : 0.f;
        g[j] = gain ? gain[kk] : 1.f;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) a[mt][j] = in ? ar[mt][kk] : 0.f;
      }
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (gain) sq[mt] = fmaf(a[mt][j], a[mt][j], sq[mt]);
        const float x = gain ? a[mt][j] * g[j] : a[mt][j];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[mt][ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, b[ct][j], acc[mt][ct], 0, 0, 0);
      }
  }
  int L = 0;
  if constexpr (ADD) L = (int)__builtin_amdgcn_raw_buffer_load_b32(pl_rsrc(L_dev, 4), 0, 0, 0);
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
    if (gain) {
      sq[mt] += __shfl_xor(sq[mt], 16, 64);
      sq[mt] += __shfl_xor(sq[mt], 32, 64);
      if (q4 == 0) sqs[wave * 16 * MT + 16 * mt + c16] = sq[mt];
    }
  // the upper half's sums go to the lower half first: four waves' sums fit the 64 KB a launch may ask for
  f4 *mine = part + (size_t)(wave % HALF) * MT * CT * 64 + lane;
  if (wave >= HALF)
#pragma unroll
    for (int n = 0; n < MT * CT; ++n) mine[n * 64] = acc[n / CT][n % CT];
  __syncthreads();
  if (wave < HALF)
#pragma unroll
    for (int n = 0; n < MT * CT; ++n) mine[n * 64] = acc[n / CT][n % CT] + mine[n * 64];
  __syncthreads();
  if (ADD && (L < 0 || L + M > max_len)) return;
  // a wave finishes a row tile's columns: the same lane layout as the products (column c16, rows 4 q4 + i)
  for (int it = wave; it < MT * (KIND == GEMM_GLU ? 1 : CT); it += GEMM_WAVES) {
    const int mt = KIND == GEMM_GLU ? it : it / CT, ct = KIND == GEMM_GLU ? 0 : it % CT;
    f4 s = {0.f, 0.f, 0.f, 0.f}, u = s;
#pragma unroll
    for (int w = 0; w < HALF; ++w) {
      s += part[((w * MT + mt) * CT + ct) * 64 + lane];
      if (KIND == GEMM_GLU) u += part[((w * MT + mt) * CT + 1) * 64 + lane];
    }
    const int c = KIND == GEMM_WIDE ? c0 + 4 * c16 + ct : c0 + c16;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = 16 * mt + 4 * q4 + i;
      if (row >= M || c >= N) continue;
      float r = 1.f;
      if (gain) {
        float t = 0.f;
#pragma unroll
        for (int w = 0; w < GEMM_WAVES; ++w) t += sqs[w * 16 * MT + row];
        r = 1.0f / sqrtf(t / (float)K + eps);
      }
      float v = s[i] * r;
      if (KIND == GEMM_GLU) v = v / (1.0f + expf(-v)) * (u[i] * r);
      float *cp = C + (size_t)row * ldc + c;
      *cp = ADD ? *cp + v : v;
    }
  }
}

// Rotates q (in place) and k by the row's position and writes k, v to cache rows L+b.
template <typename T>
__global__ void rope_kvwrite_kernel(float *qkv, int Hq, int Hkv, int dh, const float *cs, T *Kc, T *Vc,
                                    const int32_t *L_dev, int max_len, int Bp, int32_t *err, int32_t *err_map) {
  int b = blockIdx.x;
  int L = *L_dev;
  if (L < 0 || L + Bp > max_len) {
    if (threadIdx.x == 0) {  // the device word, and the host's mapped word (read without synchronising)
      *err = 1;
      __hip_atomic_store(err_map, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    return;
  }
  int half = dh / 2;
  int nq = Hq * dh, nkv = Hkv * dh;
  float *row = qkv + (size_t)b * (nq + 2 * nkv);
  for (int e = threadIdx.x; e < (Hq + Hkv) * half; e += blockDim.x) {
    int hd = e / half, i = e % half;
    float c = cs[((size_t)b * half + i) * 2], s = cs[((size_t)b * half + i) * 2 + 1];
    float *u = row + hd * dh;  // q heads then k heads are contiguous
    float x0 = u[i], x1 = u[i + half];
    float y0 = x0 * c - x1 * s, y1 = x1 * c + x0 * s;
    if (hd < Hq) {
      u[i] = y0;
      u[i + half] = y1;
    } else {
      int h = hd - Hq;
      size_t o = ((size_t)(L + b) * Hkv + h) * dh;
      store_from_float<T>(Kc + o + i, y0);
      store_from_float<T>(Kc + o + i + half, y1);
    }
  }
  for (int e = threadIdx.x; e < nkv; e += blockDim.x)
    store_from_float<T>(Vc + (size_t)(L + b) * nkv + e, row[nq + nkv + e]);
}

// One workgroup per (row b, query head): online softmax over the visible keys in chunks of blockDim.x keys, a key per
// thread for the scores; for the output the threads form blockDim.x / dh groups of a channel each, which share the chunk's
// keys and are added at the end in group order.  Scores and probabilities in float.  (With one thread per channel and the
// rest idle, one key after the other, 64 keys of 64 channels took 22 us.)
template <typename T>
__global__ __launch_bounds__(256) void attention_generic_kernel(const float *qkv, int Hq, int Hkv, int dh, const T *Kc, const T *Vc,
                                                                const int32_t *L_dev, int max_len, int Bp, const uint64_t *vis,
                                                                float *out) {
  __shared__ float qs[256], ps[256], red[8];
  int b = blockIdx.x, hq = blockIdx.y;
  int L = *L_dev;
  if (L < 0 || L + Bp > max_len) return;
  int kvh = hq / (Hq / Hkv);
  int nq = Hq * dh, nkv = Hkv * dh;
  const float *q = qkv + (size_t)b * (nq + 2 * nkv) + hq * dh;
  for (int i = threadIdx.x; i < dh; i += blockDim.x) qs[i] = q[i];
  __syncthreads();
  uint64_t vb = vis[b];
  float scale = 1.0f / sqrtf((float)dh);
  const int groups = (int)blockDim.x / dh, gi = (int)threadIdx.x / dh, ch = (int)threadIdx.x - gi * dh;
  float m_run = -INFINITY, l_run = 0.f, acc = 0.f;  // acc: output channel ch over this group's keys
  int total = L + Bp;
  for (int k0 = 0; k0 < total; k0 += blockDim.x) {
    int key = k0 + threadIdx.x;
    bool ok = key < total && (key < L || ((vb >> (key - L)) & 1ull));
    float s = -INFINITY;
    if (ok) {
      const T *kr = Kc + ((size_t)key * Hkv + kvh) * dh;
      float d0 = 0.f, d1 = 0.f;
      int i = 0;
      for (; i + 8 <= dh; i += 8) {
        float kv[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) kv[j] = load_as_float<T>(kr + i + j);
#pragma unroll
        for (int j = 0; j < 8; j += 2) {
          d0 = fmaf(qs[i + j], kv[j], d0);
          d1 = fmaf(qs[i + j + 1], kv[j + 1], d1);
        }
      }
      for (; i < dh; ++i) d0 = fmaf(qs[i], load_as_float<T>(kr + i), d0);
      s = (d0 + d1) * scale;
    }
    float m_new = fmaxf(m_run, block_max(s, red));
    float p = ok ? expf(s - m_new) : 0.f;
    float corr = (m_run == -INFINITY) ? 0.f : expf(m_run - m_new);
    __syncthreads();
    ps[threadIdx.x] = p;
    float psum = block_sum(p, red);  // contains the barriers that publish ps
    l_run = l_run * corr + psum;
    m_run = m_new;
    if (gi < groups) {
      acc *= corr;
      int kmax = min((int)blockDim.x, total - k0);
      const T *vp = Vc + ((size_t)k0 * Hkv + kvh) * dh + ch;
      int j = gi;
      for (; j + 7 * groups < kmax; j += 8 * groups) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = load_as_float<T>(vp + (size_t)(j + u * groups) * nkv);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const float pj = ps[j + u * groups];
          if (pj != 0.f) acc = fmaf(pj, v[u], acc);
        }
      }
      for (; j < kmax; j += groups) {
        const float pj = ps[j];
        if (pj != 0.f) acc = fmaf(pj, load_as_float<T>(vp + (size_t)j * nkv), acc);
      }
    }
    __syncthreads();
  }
  ps[threadIdx.x] = gi < groups ? acc : 0.f;
  __syncthreads();
  if ((int)threadIdx.x < dh) {
    float t = 0.f;
    for (int u = 0; u < groups; ++u) t += ps[u * dh + threadIdx.x];
    out[(size_t)b * nq + hq * dh + threadIdx.x] = t / l_run;
  }
}

// Greedy choice per row with ties to the lowest index, plus the two largest values.
struct Top {
  float v1;
  int i1;
  float v2;
};
__device__ __forceinline__ Top top_merge(Top a, Top b) {
  bool b_wins = (b.v1 > a.v1) || (b.v1 == a.v1 && b.i1 < a.i1);
  Top r;
  if (b_wins) {
    r.v1 = b.v1; r.i1 = b.i1; r.v2 = fmaxf(a.v1, fmaxf(a.v2, b.v2));
  } else {
    r.v1 = a.v1; r.i1 = a.i1; r.v2 = fmaxf(b.v1, fmaxf(a.v2, b.v2));
  }
  return r;
}

// A workgroup per row.  Bound by a trip to memory: eight values are on their way per thread (one at a time, each was waited for before the
// next was requested: 17 rows of 1024 4.4 -> 3.2 us).
__global__ __launch_bounds__(256) void argmax_rows_kernel(const float *logits, int V, int32_t *ids, float *top2) {
  __shared__ Top red[4];
  const float *r = logits + (size_t)blockIdx.x * V;
  Top t{-INFINITY, 0x7fffffff, -INFINITY};
  for (int i0 = threadIdx.x; i0 < V; i0 += 8 * 256) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = r[i0 + 256 * u < V ? i0 + 256 * u : i0];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (i0 + 256 * u >= V) continue;
      if (v[u] > t.v1) { t.v2 = t.v1; t.v1 = v[u]; t.i1 = i0 + 256 * u; }
      else if (v[u] > t.v2) t.v2 = v[u];
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) t = top_merge(t, Top{__shfl_xor(t.v1, o, 64), __shfl_xor(t.i1, o, 64), __shfl_xor(t.v2, o, 64)});
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = t;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) t = top_merge(t, red[w]);
    ids[blockIdx.x] = t.i1;
    if (top2) { top2[blockIdx.x * 2] = t.v1; top2[blockIdx.x * 2 + 1] = t.v2; }
  }
}

int launch_rope_table(la_model *m, const int32_t *pos, int Bp, hipStream_t s) {
  ProfScope p("rope_table", s);
  rope_table_kernel<<<Bp, 64, 0, s>>>(pos, Bp, m->d.head_dim / 2, (double)m->d.rope_theta, m->rope_cs);
  LA_HIP(hipGetLastError());
  return LA_OK;
}

int launch_argmax_rows(const float *logits, int Bp, int V, int32_t *ids, float *top2, hipStream_t s) {
  ProfScope p("argmax_rows", s);
  argmax_rows_kernel<<<Bp, 256, 0, s>>>(logits, V, ids, top2);
  LA_HIP(hipGetLastError());
  return LA_OK;
}

template <typename T, int KIND, bool ADD>
static int gemm_kind(int MT, dim3 grid, hipStream_t s, const float *A, int lda, const float *gain, float eps, const T *W, int ldw, float *C, int ldc, int M,
                     int K, int N, int vec, const int32_t *L_dev, int max_len) {
  constexpr int CT = KIND == GEMM_WIDE ? 4 : KIND == GEMM_GLU ? 2 : 1;
  const size_t lds = (size_t)GEMM_WAVES * MT * (CT * 32 * 4 + 16) * sizeof(float);
  switch (MT) {
  case 1: gemm_generic_kernel<T, 1, KIND, ADD><<<grid, 64 * GEMM_WAVES, lds, s>>>(A, lda, gain, eps, W, ldw, C, ldc, M, K, N, vec, L_dev, max_len); break;
  case 2: gemm_generic_kernel<T, 2, KIND, ADD><<<grid, 64 * GEMM_WAVES, lds, s>>>(A, lda, gain, eps, W, ldw, C, ldc, M, K, N, vec, L_dev, max_len); break;
  default:
    if constexpr (KIND != GEMM_WIDE) {  // (two row tiles at most)
      if (MT == 3) gemm_generic_kernel<T, 3, KIND, ADD><<<grid, 64 * GEMM_WAVES, lds, s>>>(A, lda, gain, eps, W, ldw, C, ldc, M, K, N, vec, L_dev, max_len);
      else gemm_generic_kernel<T, 4, KIND, ADD><<<grid, 64 * GEMM_WAVES, lds, s>>>(A, lda, gain, eps, W, ldw, C, ldc, M, K, N, vec, L_dev, max_len);
    }
  }
  LA_HIP(hipGetLastError());
  return LA_OK;
}

// N: columns of C (GLU: half the columns of W).  into: C is added to, unless the block does not fit this cache.
// 64 columns per workgroup once that alone gives each of 256 CUs some, up to two
// row tiles (16 columns / 64, us): 4096 x 32768 179 / 144 at one row, 253 / 158 at 32; 1024 x 16384 25 / 21 and 29 / 26;
// 1024 x 8192 14 / 21 and 18 / 26.
template <typename T>
static int gemm(const char *name, const float *A, int lda, const float *gain, float eps, const void *W, int ldw, float *C, int ldc, int M, int K,
                int N, const la_kv *into, bool glu, hipStream_t s) {
  ProfScope p(name, s);
  const int MT = ceil_div(M, 16), vec = ((uintptr_t)A | (size_t)lda * 4) % 16 == 0;
  auto run = [&](auto kind, auto add, int wgs) {
    return gemm_kind<T, decltype(kind)::value, decltype(add)::value>(MT, wgs, s, A, lda, gain, eps, (const T *)W, ldw, C, ldc, M, K, N, vec,
                                                                     into ? into->L_dev : nullptr, into ? into->max_len : 0);
  };
  using std::bool_constant;
  using std::integral_constant;
  if (glu) return run(integral_constant<int, GEMM_GLU>{}, bool_constant<false>{}, ceil_div(N, 16));
  if (N >= 64 * 256 && MT <= 2)
    return into ? run(integral_constant<int, GEMM_WIDE>{}, bool_constant<true>{}, ceil_div(N, 64)) : run(integral_constant<int, GEMM_WIDE>{}, bool_constant<false>{}, ceil_div(N, 64));
  return into ? run(integral_constant<int, GEMM_16>{}, bool_constant<true>{}, ceil_div(N, 16)) : run(integral_constant<int, GEMM_16>{}, bool_constant<false>{}, ceil_div(N, 16));
}

// la_plain.h's attention takes heads that are whole groups of 16 channels and a layer's cache within 32-bit offsets; beside the
// general products it runs where its workgroups (a row, a head and 64 channels each) are a few rounds of the chip for the fullest
// block: two bf16 layers 1024 wide, 16 heads of 64, L = 47, 17 / 64 rows 125 / 174 us against 126 / 180, L = 3000, 64 rows 371 / 408. Twice the
// workgroups (2048 wide, 16 heads of 128): L = 47, 17 / 64 rows 287 / 420 against 290 / 405, L = 3000, 17 rows 577 / 633; four times (4096
// wide, 32 heads), L = 3000, 17 rows 1156 / 1074.  Not by the rows of a block: a row must not depend on the block it is in, and the two
// kernels sum in different orders.
static bool plain_heads(const la_model *m, const la_kv *kv) { return m->d.head_dim % 16 == 0 && kv->layer_elems() * m->esize < (size_t)1 << 31; }
static bool plain_attention_pays(const la_model *m, const la_kv *kv) {
  return plain_heads(m, kv) && m->d.n_q_heads * ceil_div(m->d.head_dim, 64) <= 16;
}
// Its products take layers that also fit 32-bit offsets, of up to 16 M weights, whose products are one round of the chip each: a workgroup of eight waves with
// six slices of its operands on their way (sixteen with three into the residual stream) has a CU to itself, with two slices (contractions of at most 256) there
// is room for two.  A second round reads all activations again and waits as long as the first.  Both sides of the lines, a forward of two layers at 1 / 17 / 48
// / 64 rows, L = 47, heads of 64 channels, fp32 (bf16 the same or up to 7 % less, 13 % at one row), us, these products (the general ones):
//   512 wide, 2048 of gate: 61 / 73 / 95 / 111 (74 / 92 / 111 / 125); 2064: 62 / 79 / 103 / 122 (77 / 94 / 111 / 123)
//   256 wide, 4096 of gate: 66 / 81 / 110 / 130 (85 / 106 / 125 / 141); 8192: 87 / 114 / 165 / 202 (119 / 150 / 187 / 214)
//   768 wide, 2064 of gate: 67 / 89 / 120 / 143 (81 / 99 / 123 / 138)
//   1024 wide, 2752 of gate: 85 / 110 / 155 / 187 (100 / 124 / 154 / 176)
//   1536 wide, 2048 of gate (16.5 M): 103 / 120 / 159 / 190 (113 / 144 / 181 / 207); 2064: 105 / 132 / 181 / 218 (113 / 143 / 180 / 205)
//   2048 wide, 2048 of gate (25 M): 131 / 150 / 194 / 234 (131 / 167 / 211 / 250)
// (The lines were drawn when these products took up to 15 % longer: a second round still loses at 64 rows where the activations are wide, but not 256 wide, and
// layers of 25 M weights would gain.)
// The rule does not ask for the rows: the two kinds of products round differently, and a row must not depend on the block it is in.
constexpr size_t PL_LAYER_WEIGHTS = (size_t)1 << 24;
static bool plain_round(int K, int workgroups) { return workgroups <= (K <= 2 * 16 * PL_WAVES ? 2 : 1) * 256; }
static bool plain_layers(const la_model *m, const la_kv *kv) {
  const la_model_desc &d = m->d;
  const size_t qd = m->qdim(), dm = d.d_model, F = d.d_ffn, pad = 16 * PL_WAVES * 6;
  for (size_t n : {(dm + pad) * m->nqkv(), (qd + pad) * dm, (dm + pad) * 2 * F, (F + pad) * dm, (LA_MAX_ROWS + 1) * (dm + qd + F) + pad})
    if (n * 4 >= (size_t)1 << 31) return false;
  return plain_heads(m, kv) && dm * (m->nqkv() + qd) + 3 * dm * F <= PL_LAYER_WEIGHTS && plain_round(dm, m->nqkv() / 16) && plain_round(dm, ceil_div(F, 8)) &&
         plain_round(qd, ceil_div(dm, 16)) && plain_round(F, ceil_div(dm, 16));
}

// The unembedding takes the same products by the same rule (it sums in the general product's order, bit for bit).  Unembedding and arg-max, fp32,
// 1 / 17 / 64 rows, us (with the general product, which waits for each turn's loads before it asks for the next): 256 x 1024 5.5 / 6.8 / 9.1 (6.6 / 8.7 /
// 10.3), 256 x 8192 8.3 / 10.5 / 14.4 (15.7 / 18.2 / 21.6), 1024 x 4096 9.3 / 13.1 / 19.7 (14.4 / 18.0 / 22.5).
static bool plain_head(const la_model_desc &d) {
  const size_t dm = d.d_model, V = d.vocab, pad = 16 * PL_WAVES * 6;
  return (dm + pad) * V * 4 < (size_t)1 << 31 && ((LA_MAX_ROWS + 1) * dm + pad) * 4 < (size_t)1 << 31 && dm * V <= PL_LAYER_WEIGHTS && plain_round(dm, ceil_div(V, 16));
}

struct PlainScratch {
  float *q, *attn, *act, *cs;
};
// pos, vis NULL: the rows of a prompt, behind the length.
template <typename T>
static int plain_forward_t(la_model *m, int lb, int le, float *hidden, int Bp, const int32_t *pos, const uint64_t *vis, la_kv *kv, const PlainScratch &b, hipStream_t s) {
  const la_model_desc &d = m->d;
  const int nqkv = m->nqkv(), qd = m->qdim(), F = d.d_ffn, dm = d.d_model;
  int rc = LA_OK;
  for (int l = lb; l < le; ++l) {
    const GenericLayer &w = m->layers[l];
    LA_REQUIRE(w.set, LA_EINVAL, "layer %d has no weights", l);
    T *Kc = (T *)kv->K + (size_t)l * kv->layer_elems(), *Vc = (T *)kv->V + (size_t)l * kv->layer_elems();
    auto product = [&](const float *A, int K, const float *gain, const void *W, int ldw, int N, float *out, int ldo) {
      PlProduct p{};
      p.A = A; p.lda = K; p.M = Bp; p.K = K; p.gain = gain; p.eps = d.rms_eps; p.W = W; p.ldw = ldw; p.N = N; p.out = out; p.ldo = ldo;
      p.cs = b.cs; p.Kc = Kc; p.Vc = Vc; p.Hq = d.n_q_heads; p.Hkv = d.n_kv_heads; p.dh = d.head_dim; p.max_len = kv->max_len;
      p.L_dev = kv->L_dev; p.err = kv->err_dev; p.err_map = m->err_map; p.pos = pos; p.theta = d.rope_theta;
      return p;
    };
    const PlProduct qkv = product(hidden, dm, w.g_attn, w.wqkv, nqkv, nqkv, b.q, qd);
    if ((rc = l == lb ? plain_product<T, PL_QKV_FIRST>("plain_qkv", qkv, nqkv / 16, s) : plain_product<T, PL_QKV>("plain_qkv", qkv, nqkv / 16, s))) return rc;
    if (!vis && l + 1 == d.n_layers) break;  // (of a prompt's last layer nobody reads more than the K and V rows)
    if ((rc = plain_attention<T>(b.q, qd, d, Kc, Vc, kv, Bp, vis, b.attn, s))) return rc;
    if ((rc = plain_product<T, PL_RESID>("plain_o", product(b.attn, qd, nullptr, w.wo, dm, dm, hidden, dm), ceil_div(dm, 16), s))) return rc;
    if ((rc = plain_product<T, PL_GLU>("plain_gateup", product(hidden, dm, w.g_mlp, w.wgu, 2 * F, F, b.act, F), ceil_div(F, 8), s))) return rc;
    if ((rc = plain_product<T, PL_RESID>("plain_down", product(b.act, F, nullptr, w.wdown, dm, dm, hidden, dm), ceil_div(dm, 16), s))) return rc;
  }
  return LA_OK;
}

template <typename T>
static int forward_t(la_model *m, int lb, int le, float *hidden, int Bp, const int32_t *pos, const uint64_t *vis,
                     la_kv *kv, hipStream_t s) {
  if (plain_layers(m, kv)) return plain_forward_t<T>(m, lb, le, hidden, Bp, pos, vis, kv, PlainScratch{m->qkv, m->attn, m->act, m->rope_cs}, s);
  const la_model_desc &d = m->d;
  int nqkv = m->nqkv(), qd = m->qdim(), F = d.d_ffn, dm = d.d_model;
  int rc = launch_rope_table(m, pos, Bp, s);
  if (rc) return rc;
  for (int l = lb; l < le; ++l) {
    const GenericLayer &w = m->layers[l];
    LA_REQUIRE(w.set, LA_EINVAL, "layer %d has no weights", l);
    T *Kc = (T *)kv->K + (size_t)l * kv->layer_elems();
    T *Vc = (T *)kv->V + (size_t)l * kv->layer_elems();
    if ((rc = gemm<T>("gemm_qkv", hidden, dm, w.g_attn, d.rms_eps, w.wqkv, nqkv, m->qkv, nqkv, Bp, dm, nqkv, nullptr, false, s))) return rc;
    {
      ProfScope p("rope_kvwrite", s);
      rope_kvwrite_kernel<T><<<Bp, 256, 0, s>>>(m->qkv, d.n_q_heads, d.n_kv_heads, d.head_dim, m->rope_cs, Kc, Vc,
                                                 kv->L_dev, kv->max_len, Bp, kv->err_dev, m->err_map);
    }
    if (plain_attention_pays(m, kv)) {
      if ((rc = plain_attention<T>(m->qkv, nqkv, d, Kc, Vc, kv, Bp, vis, m->attn, s))) return rc;
    } else {
      ProfScope p("attention", s);
      attention_generic_kernel<T><<<dim3(Bp, d.n_q_heads), 256, 0, s>>>(
          m->qkv, d.n_q_heads, d.n_kv_heads, d.head_dim, Kc, Vc, kv->L_dev, kv->max_len, Bp, vis, m->attn);
    }
    if ((rc = gemm<T>("gemm_o", m->attn, qd, nullptr, 0.f, w.wo, dm, hidden, dm, Bp, qd, dm, kv, false, s))) return rc;
    if ((rc = gemm<T>("gemm_gateup", hidden, dm, w.g_mlp, d.rms_eps, w.wgu, 2 * F, m->act, F, Bp, dm, F, nullptr, true, s))) return rc;
    if ((rc = gemm<T>("gemm_down", m->act, F, nullptr, 0.f, w.wdown, dm, hidden, dm, Bp, F, dm, kv, false, s))) return rc;
    LA_HIP(hipGetLastError());
  }
  return LA_OK;
}

int generic_forward(la_model *m, int lb, int le, float *hidden, int Bp, const int32_t *pos, const uint64_t *vis,
                    la_kv *kv, hipStream_t s) {
  if (m->d.dtype == LA_F32) return forward_t<float>(m, lb, le, hidden, Bp, pos, vis, kv, s);
  if (m->d.dtype == LA_F16) return forward_t<_Float16>(m, lb, le, hidden, Bp, pos, vis, kv, s);
  return forward_t<uint16_t>(m, lb, le, hidden, Bp, pos, vis, kv, s);
}

// A prompt through the small layers' launches, PL_PROMPT rows at a time: every row is summed as it is in a block, in one launch instead of one for each 64
// rows, which leave most of the chip idle, and nothing of the last layer but its K and V.  Two fp32 layers 256 wide, us: 65 tokens 129 -> 53, 300 tokens
// 402 -> 80, 1000 tokens 1414 -> 215, 3000 tokens 5108 -> 1045.
// Scratch for the rows (6 MB for these layers, some tens at most: plain_layers) comes with the first prompt of more than one block and stays with the model;
// without memory for it, and for short prompts, the rows go 64 at a time through a block's.  The thread's capture mode is relaxed meanwhile, so that a first prompt may be captured.
constexpr int PL_PROMPT = 1024;
int generic_prefill_rows(la_model *m, const la_kv *kv, int n, int *rows) {
  *rows = 0;
  if (m->use_mfma || !m->embed || !plain_layers(m, kv)) return LA_OK;
  for (int l = 0; l < m->d.n_layers; ++l) LA_REQUIRE(m->layers[l].set, LA_EINVAL, "layer %d has no weights", l);
  if (n > LA_MAX_ROWS && !m->prompt) {
    const size_t per_row = (size_t)m->d.d_model + 2 * (size_t)m->qdim() + m->d.d_ffn + m->d.head_dim;
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    const bool relaxed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
    if (hipMalloc((void **)&m->prompt, PL_PROMPT * per_row * 4) != hipSuccess) {
      m->prompt = nullptr;
      (void)hipGetLastError();  // (the next launch's check would report it)
    }
    if (relaxed) (void)hipThreadExchangeStreamCaptureMode(&mode);
  }
  *rows = n > LA_MAX_ROWS && m->prompt ? PL_PROMPT : LA_MAX_ROWS;
  return LA_OK;
}

// M tokens at L0, L0 + 1, ... through every layer (the caller sets the cache length afterwards).
int generic_prefill_chunk(la_model *m, la_kv *kv, const int32_t *tok, int M, int L0, hipStream_t s) {
  const la_model_desc &d = m->d;
  const size_t R = PL_PROMPT;
  float *x = m->pf_hidden;
  PlainScratch b{m->qkv, m->attn, m->act, m->rope_cs};
  if (M > LA_MAX_ROWS) {
    x = m->prompt;
    b.q = x + R * d.d_model;
    b.attn = b.q + R * m->qdim();
    b.act = b.attn + R * m->qdim();
    b.cs = b.act + R * d.d_ffn;
  }
  const int rc = launch_embed(m, tok, M, x, kv->L_dev, L0, s);
  if (rc) return rc;
  if (d.dtype == LA_F32) return plain_forward_t<float>(m, 0, d.n_layers, x, M, nullptr, nullptr, kv, b, s);
  if (d.dtype == LA_F16) return plain_forward_t<_Float16>(m, 0, d.n_layers, x, M, nullptr, nullptr, kv, b, s);
  return plain_forward_t<uint16_t>(m, 0, d.n_layers, x, M, nullptr, nullptr, kv, b, s);
}

int generic_unembed_argmax(la_model *m, const float *hidden, int Bp, int32_t *ids, float *top2, hipStream_t s) {
  const la_model_desc &d = m->d;
  int rc;
  auto head = [&](auto t) {
    using T = decltype(t);
    if (plain_head(d)) {
      PlProduct p{};
      p.A = hidden; p.lda = p.K = d.d_model; p.M = Bp; p.gain = m->g_final; p.eps = d.rms_eps; p.W = m->unembed; p.ldw = p.N = p.ldo = d.vocab; p.out = m->logits;
      return plain_product<T, PL_STORE>("gemm_unembed", p, ceil_div(d.vocab, 16), s);
    }
    return gemm<T>("gemm_unembed", hidden, d.d_model, m->g_final, d.rms_eps, m->unembed, d.vocab, m->logits, d.vocab, Bp, d.d_model, d.vocab, nullptr, false, s);
  };
  rc = d.dtype == LA_F32 ? head(float{}) : d.dtype == LA_F16 ? head(_Float16{}) : head(uint16_t{});
  if (rc) return rc;
  return launch_argmax_rows(m->logits, Bp, d.vocab, ids, top2, s);
}

}  // namespace la
