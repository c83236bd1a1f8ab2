// Lookahead controller on the device (Section 4.3 of the paper; Section 3.3 for the cache
// crop / relocation): block layout, n-gram pool, verification, acceptance, KV commit.
// All integer work.  A step never needs the host: one launch verifies, moves the cache rows of
// accepted verification rows (a workgroup per layer and row) and, in the workgroup that is
// through last, updates the pool and lays out the next block with one wave.
#include "la_device.h"
#include "la_internal.h"

namespace la {

struct PoolView {
  uint32_t *stamp;
  int32_t *toks;
  uint32_t *counter;
  int vocab, N, G;
};

__host__ __device__ inline int la_row_index(int W, int r, int c) { return 1 + r * W + c; }
__host__ __device__ inline int v_row_index(int W, int N, int k, int j) { return 1 + W * (N - 1) + k * (N - 1) + (j - 1); }

// Token-free part of the block: position and visibility of every row.  Row 0 is the real
// next-token row at position t.  Window entry (r, c) sits at t+1+c+r and sees row 0, the
// level-0 entries of columns <= c and the entries above it in its own column.  Verification
// row (k, j) sits at t+j and sees row 0 and the earlier tokens of candidate k.  Rows that
// carry nothing (candidates absent, padding) sit at t and see only themselves.
__host__ __device__ inline void block_layout(int W, int N, int G, int n_cand, int t, int Bp, int32_t *pos,
                                             uint64_t *vis) {
  for (int i = 0; i < Bp; ++i) {
    pos[i] = t;
    vis[i] = 1ull << i;
  }
  for (int r = 0; r < N - 1; ++r)
    for (int c = 0; c < W; ++c) {
      int i = la_row_index(W, r, c);
      uint64_t m = 1ull;
      for (int c2 = 0; c2 <= c; ++c2) m |= 1ull << la_row_index(W, 0, c2);
      for (int r2 = 1; r2 <= r; ++r2) m |= 1ull << la_row_index(W, r2, c);
      pos[i] = t + 1 + c + r;
      vis[i] = m;
    }
  for (int k = 0; k < n_cand && k < G; ++k)
    for (int j = 1; j <= N - 1; ++j) {
      int i = v_row_index(W, N, k, j);
      uint64_t m = 1ull;
      for (int j2 = 1; j2 <= j; ++j2) m |= 1ull << v_row_index(W, N, k, j2);
      pos[i] = t + j;
      vis[i] = m;
    }
}

// The next block into *st, one row per lane (lane < 64): tokens from the window and the candidates in LDS.
__device__ __forceinline__ void build_block(la_step_state *st, int W, int N, int n_cand, int t, int Bp, int c0, const int32_t *win, const int32_t *cand, int i) {
  if (i >= Bp) return;
  const int n1 = N - 1;
  int pos = t, tok = c0;
  uint64_t vis = 1ull << i;
  const int w = i - 1, v = w - W * n1;  // index among the window rows, among the verification rows
  if (i > 0 && v < 0) {
    const int r = w / W, c = w - r * W;
    uint64_t m = 1ull | (((2ull << c) - 1ull) << la_row_index(W, 0, 0));
    for (int r2 = 1; r2 <= r; ++r2) m |= 1ull << la_row_index(W, r2, c);
    pos = t + 1 + c + r;
    vis = m;
    tok = win[w];
  } else if (i > 0 && v < n_cand * n1) {
    const int k = v / n1, j = v - k * n1 + 1;
    vis = 1ull | (((1ull << j) - 1ull) << v_row_index(W, N, k, 1));
    pos = t + j;
    tok = cand[v];
  }
  st->pos[i] = pos;
  st->vis[i] = vis;
  st->tok[i] = tok;
}

// A slot on its way from the pool: its stamp and its tuple's first words (all requested before any is waited for: with one after
// the other each cost a trip to memory), the rest of a longer tuple when it is put into LDS.
struct SlotIn {
  const int32_t *src;  // NULL: no slot in this lane
  uint32_t stamp;
  int32_t t[4];
};
__device__ __forceinline__ SlotIn slot_request(const PoolView &p, bool in, size_t slot) {
  const int n1 = p.N - 1;
  SlotIn r{};
  if (!in) return r;
  r.src = p.toks + slot * n1;
  r.stamp = p.stamp[slot];
#pragma unroll
  for (int u = 0; u < 4; ++u) r.t[u] = r.src[u < n1 ? u : n1 - 1];
  return r;
}
__device__ __forceinline__ void slot_put(const SlotIn &r, int32_t *dst, int n1) {
  if (r.src == nullptr) return;
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (u < n1) dst[u] = r.t[u];
  for (int j = 4; j < n1; ++j) dst[j] = r.src[j];
}
// The slots of `key`, slot s in lane s.
__device__ __forceinline__ SlotIn key_request(const PoolView &p, int key, int lane) {
  const bool in = lane < p.G && key >= 0 && key < p.vocab;
  return slot_request(p, in, in ? (size_t)key * p.G + lane : 0);
}

// Candidates from a key's slots (stamp of slot s in lane s, its tuple in tok[s (N-1)]), most recently inserted first, into
// cand[k*(N-1)+j] (LDS and, where it is kept, the state); returns the count.  Stamps are distinct, so a slot's place is the number
// of later ones.
__device__ __forceinline__ int pool_order(const PoolView &p, uint32_t sv, const int32_t *tok, int32_t *cand, int32_t *state_cand, int lane) {
  const int n1 = p.N - 1;
  int place = 0;
  for (int s = 0; s < p.G; ++s) place += (uint32_t)__builtin_amdgcn_readlane((int)sv, s) > sv ? 1 : 0;
  if (sv != 0u)
    for (int j = 0; j < n1; ++j) {
      const int32_t t = tok[lane * n1 + j];
      cand[place * n1 + j] = t;
      state_cand[place * n1 + j] = t;
    }
  return __popcll(__ballot(sv != 0u));
}

// LDS words written by one lane of the (single remaining) wave are read by others: a wave's LDS operations are in order.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Inserts (win[c] -> tuple of column c) for c = 0 .. W - 1 in that order: a tuple that is present gets a new stamp, else a
// free slot is taken, else the one with the smallest stamp.  Keys do not meet, so a wave takes as many of them at once as it has
// lanes for their slots (lane: slot s of a key), and each key's columns in order, its slots in registers and LDS meanwhile: a
// column that shares its key with others costs no trip to memory.  (One by one through memory, 31 columns of one key with 32
// slots made an accept 101 us, one thread had taken 52; now 19.  15 columns, 15
// slots, five keys: 10 us, one thread 43.)
// In two steps: the first keys' slots come in while the accept's other work is on its way (harvest_load, which writes nothing but
// LDS), the rest follows when every workgroup has read what it needs.
struct HarvestLds {
  int32_t lead[LA_MAX_ROWS], next[LA_MAX_ROWS];  // first column of the k-th key; the next column with the same key
  int32_t tok[256];                              // tuples of the slots at hand (224 words at most: W = 7, N = 5, G = 8)
};
struct HarvestAt {
  int n_keys, c;  // keys; this lane's first column (W: none)
  size_t slot;
  SlotIn in;
};
__device__ __forceinline__ void harvest_slots(const PoolView &p, const int32_t *win, int W, HarvestLds &h, int lane, int k0, HarvestAt &at) {
  const int G = p.G, per = 64 / G, g = lane / G, s = lane - g * G;
  const bool in = g < per && k0 + g < at.n_keys;
  at.c = in ? h.lead[k0 + g] : W;
  at.slot = in ? (size_t)win[at.c] * G + s : 0;
  at.in = slot_request(p, in, at.slot);
}
__device__ __forceinline__ void harvest_load(const PoolView &p, const int32_t *win, int W, HarvestLds &h, int lane, HarvestAt &at) {
  at.n_keys = 0;
  at.c = W;
  at.slot = 0;
  at.in = SlotIn{};
  if (p.G == 0) return;
  const int my_key = lane < W ? win[lane] : -1;
  bool first = my_key >= 0 && my_key < p.vocab;
  int next = W;
  for (int c = W - 1; c >= 0; --c) {
    const bool same = __builtin_amdgcn_readlane(my_key, c) == my_key;
    if (same && c < lane) first = false;
    if (same && c > lane) next = c;
  }
  h.next[lane] = next;
  const uint64_t firsts = __ballot(first);
  if (first) h.lead[__popcll(firsts & ((1ull << lane) - 1ull))] = lane;
  at.n_keys = __popcll(firsts);
  wave_sync();
  harvest_slots(p, win, W, h, lane, 0, at);
}
__device__ __forceinline__ void pool_harvest(const PoolView &p, const int32_t *win, const int32_t *newest, int W, HarvestLds &h, int lane, HarvestAt &at,
                                             uint32_t now) {
  const int G = p.G, n1 = p.N - 1;
  if (lane == 0) *p.counter = now + (uint32_t)W;
  if (G == 0) return;
  const int per = 64 / G, g = lane / G, s = lane - g * G;
  const uint64_t mine = ((1ull << G) - 1ull) << (g * G < 64 ? g * G : 0);  // (G < 64)
  for (int k0 = 0; k0 < at.n_keys; k0 += per) {
    int32_t *tok = h.tok + (at.c < W ? lane * n1 : 0);
    if (k0 > 0) {
      harvest_slots(p, win, W, h, lane, k0, at);
      tok = h.tok + (at.c < W ? lane * n1 : 0);
      slot_put(at.in, tok, n1);
    }
    int c = at.c;
    uint32_t sv = at.in.stamp;
    bool replaced = false;
    while (__any(c < W)) {
      const bool on = c < W;
      bool same = on && sv != 0u;
      if (on)
        for (int j = 0; j < n1; ++j) same = (tok[j] == (j + 1 < n1 ? win[(j + 1) * W + c] : newest[c])) && same;
      const uint64_t hit = __ballot(same) & mine, empty = __ballot(on && sv == 0u) & mine;
      bool oldest = true;
      if (__any(on && !hit && !empty))
        for (int i = 0; i < G; ++i) {
          const uint32_t o = (uint32_t)__shfl((int)sv, g * G + i < 64 ? g * G + i : 63, 64);
          oldest = oldest && (i == s || o > sv);
        }
      if (on && (hit ? same : empty ? lane == __ffsll((long long)empty) - 1 : oldest)) {
        sv = now + (uint32_t)c + 1u;
        if (!hit) {
          for (int j = 0; j < n1; ++j) tok[j] = j + 1 < n1 ? win[(j + 1) * W + c] : newest[c];
          replaced = true;
        }
      }
      if (on) c = h.next[c];
    }
    if (sv != at.in.stamp) p.stamp[at.slot] = sv;
    if (replaced)
      for (int j = 0; j < n1; ++j) p.toks[at.slot * n1 + j] = tok[j];
  }
}

__global__ void fill_u32_kernel(uint32_t *p, size_t n, uint32_t v) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}

// Every N-gram of the prompt into the (empty) pool, as if inserted in order: a key ends up with its last G distinct tuples,
// each with the stamp of its last insertion.  One wave per position; the last position of each key does the work: it walks
// back over the prompt, 256 positions at a time, and collects tuples it has not seen until it has G.  (One thread inserting
// one N-gram after the other waited for the pool's memory twice per token: 2.7 ms for 2048 tokens of text and seven slots, now
// 9 us.  Occurrences of a key are compared one by one, about 0.3 us each, so a prompt that repeats few tuples is slower than
// text, though not than one thread: 2048 times the same token 0.65 ms, one thread 1.4.)
__global__ __launch_bounds__(256) void pool_seed_kernel(PoolView p, const int32_t *prompt, int n) {  // n = P - N + 1 N-grams
  const int lane = threadIdx.x & 63, i = (int)(blockIdx.x * 4 + (threadIdx.x >> 6)), n1 = p.N - 1;
  if (i >= n) return;
  const int key = prompt[i];
  if (key < 0 || key >= p.vocab) return;
  for (int j0 = i + 1; j0 < n; j0 += 256) {  // a later position with this key?
    bool found = false;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = j0 + 64 * u + lane;
      found = found || (j < n && prompt[j] == key);
    }
    if (__any(found)) return;
  }
  int got = i, count = 1;  // lane s: position of the s-th tuple found
  for (int j0 = i - 1; j0 >= 0 && count < p.G; j0 -= 256) {  // positions j0, j0 - 1, ...
    bool at[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = j0 - 64 * u - lane;
      at[u] = j >= 0 && prompt[j < 0 ? 0 : j] == key;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      uint64_t m = __ballot(at[u]);
      while (m != 0 && count < p.G) {
        const int j = j0 - 64 * u - (__ffsll((long long)m) - 1);
        m &= m - 1;
        bool same = lane < count;
        for (int t = 1; t <= n1; ++t) same = (prompt[got + t] == prompt[j + t]) && same;
        if (!__any(same)) {
          if (lane == count) got = j;
          ++count;
        }
      }
    }
  }
  if (lane < count) {
    const size_t slot = (size_t)key * p.G + lane;
    p.stamp[slot] = (uint32_t)got + 1u;
    for (int t = 0; t < n1; ++t) p.toks[slot * n1 + t] = prompt[got + 1 + t];
  }
}

__global__ __launch_bounds__(64) void state_init_kernel(PoolView p, la_step_state *st, const int32_t *prompt, int P, int W, int N, int G,
                                                        int Bp, uint32_t inserted, int32_t *kv_L) {
  __shared__ int32_t win[LA_MAX_ROWS], cand[LA_MAX_ROWS], slots[LA_MAX_ROWS];
  const int lane = threadIdx.x, c0 = prompt[P - 1];
  if (lane < W * (N - 1)) {
    const int r = lane / W, c = lane - r * W;
    win[lane] = st->win[lane] = prompt[(r + c) % P];
  }
  int n_cand = 0;
  if (N >= 2) {
    const SlotIn in = key_request(p, c0, lane);
    slot_put(in, slots + (in.src ? lane * (N - 1) : 0), N - 1);
    n_cand = pool_order(p, in.stamp, slots, cand, st->cand, lane);
  }
  __syncthreads();
  build_block(st, W, N, n_cand, P - 1, Bp, c0, win, cand, lane);
  if (lane == 0) {
    *p.counter = inserted;
    st->L = P - 1;
    st->c0 = c0;
    st->Bp = Bp;
    st->steps = st->matched_steps = st->n_emitted = st->last_emitted = st->last_k = st->last_m = 0;
    st->error = st->reserved = 0;
    st->n_cand = n_cand;
    *kv_L = P - 1;
  }
}

// The accept phase in one launch: a workgroup per layer and verification row.  Every workgroup verifies for itself (a candidate
// per lane), those whose row is accepted move it in their layer (cache relocation: the rows of candidate best_k go from block
// rows v(k, j) to cache rows L0 + j, j = 1 .. e - 1), and the one that is through last -- all others have read the state by
// then; nobody waits -- does the rest with one wave: harvest with a pool slot per lane, the next block with a row per lane.
// The workgroups are counted in st->reserved (zero between launches): a word of the state and not of the pool, which several
// generations may share, and cleared by the init kernels on the stream that the accepts follow on.
// Bound by the trips to memory that depend on each other: the state; with it known, the pool's slots (of the window's keys and of
// the last accepted token) beside the moving rows and the count; the next block out.  (One thread doing all of it took 23 us, most
// of it waiting for one word after the other; the relocation as a launch of its own cost 16 accepts 40 us; slots asked for after
// the count, a tuple's words and a moved row's elements one after the other: 7.4 us an accept at W = 7, N = 4, G = 7 where
// nothing is accepted, now 6.3; 40 tokens in all, so that rows move in 2 layers 9.4 -> 8.2, in 32 layers 10.3 -> 8.8.)
template <typename T>
__global__ __launch_bounds__(256) void accept_kernel(PoolView p, la_step_state *st, const int32_t *ids, int32_t *emitted, int max_total, int W, int N, int G,
                                                     int32_t *kv_L, const int32_t *err, T *K, T *V, size_t layer_elems, int Hkv, int dh, int v_blocked,
                                                     int max_len) {
  __shared__ int32_t id[LA_MAX_ROWS], win[LA_MAX_ROWS], cand[LA_MAX_ROWS], newest[LA_MAX_ROWS], slots[LA_MAX_ROWS];
  __shared__ HarvestLds harvest;
  __shared__ int is_last;
  const int lane = threadIdx.x & 63, n1 = N - 1, rows = 1 + (W + G) * n1;
  if (threadIdx.x < 64) {
    if (lane < rows) id[lane] = ids[lane];
    win[lane] = lane < W * n1 ? st->win[lane] : 0;
    cand[lane] = st->cand[lane];
  }
  const int emitted_before = st->n_emitted, n_cand = st->n_cand, L0 = st->L, Bp = st->Bp;
  const int error = *err;  // what the launches before this one on the model raised (0: nothing)
  const int steps = st->steps, matched = st->matched_steps;
  __syncthreads();
  const int remaining = max_total - emitted_before;
  // candidate `lane` matches m tokens; the longest match wins, the lowest candidate of equal ones
  int m = 0;
  if (lane < n_cand && cand[lane * n1] == id[0]) {
    m = 1;
    while (m < n1 && cand[lane * n1 + m] == id[v_row_index(W, N, lane, m)]) ++m;
  }
  int best = m * 64 + (63 - lane);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const int other = __shfl_xor(best, o, 64);
    best = other > best ? other : best;
  }
  const int best_m = best >> 6, best_k = best_m > 0 ? 63 - (best & 63) : 0;
  const int e = best_m + 1 < remaining ? best_m + 1 : remaining;
  const int last = e <= 1 ? id[0] : id[v_row_index(W, N, best_k, e - 1)];
  // the pool's slots that the serial part will need, while the rows move and the workgroups are counted (nothing of the pool is
  // written before the last one is through here)
  HarvestAt at;
  uint32_t sv = 0u, now = 0u;
  if (N >= 2 && threadIdx.x < 64) {
    now = *p.counter;
    const SlotIn in = key_request(p, last, lane);
    harvest_load(p, win, W, harvest, lane, at);
    sv = in.stamp;
    slot_put(in, slots + (in.src ? lane * n1 : 0), n1);
    slot_put(at.in, harvest.tok + (at.in.src ? lane * n1 : 0), n1);
  }
  const int row = (int)blockIdx.y + 1, src = L0 + v_row_index(W, N, best_k, row), dst = L0 + row;
  if (row < e && src < max_len && dst < max_len && L0 >= 0) {
    T *Kl = K + (size_t)blockIdx.x * layer_elems;
    T *Vl = V + (size_t)blockIdx.x * layer_elems;
    const int n = Hkv * dh;
    for (int i0 = threadIdx.x; i0 < n; i0 += 4 * 256) {  // (all loads of a turn before its first store)
      T k[4], v[4];
      auto at_v = [&](int row, int i) {
        const int h = i / dh;
        return v_index(v_blocked, row, h, i - h * dh, Hkv, dh);
      };
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = i0 + 256 * u < n ? i0 + 256 * u : i0;
        k[u] = Kl[(size_t)src * n + i];
        v[u] = Vl[at_v(src, i)];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = i0 + 256 * u;
        if (i >= n) continue;
        Kl[(size_t)dst * n + i] = k[u];
        Vl[at_v(dst, i)] = v[u];
      }
    }
  }
  __syncthreads();  // (every wave has what it needs of the state)
  if (threadIdx.x == 0) {
    is_last = atomicAdd(&st->reserved, 1) + 1 == (int)(gridDim.x * gridDim.y);
    if (is_last) st->reserved = 0;
  }
  __syncthreads();
  if (!is_last || threadIdx.x >= 64) return;
  if (remaining <= 0) {  // budget spent: the step is a no-op
    if (lane == 0) {
      st->error = error;
      st->last_emitted = 0;
    }
    return;
  }
  if (lane < e) emitted[emitted_before + lane] = lane == 0 ? id[0] : id[v_row_index(W, N, best_k, lane)];
  // harvest: each window column yields one n-gram ending in the model's newest guess; then the columns move up
  int n_next = 0;
  if (N >= 2) {
    if (lane < W) newest[lane] = id[la_row_index(W, N - 2, lane)];
    wave_sync();
    pool_harvest(p, win, newest, W, harvest, lane, at, now);
    if (__any(lane < W && win[lane] == last)) {  // a column has just been inserted under the key that is looked up
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
      const SlotIn in = key_request(p, last, lane);
      sv = in.stamp;
      slot_put(in, slots + (in.src ? lane * n1 : 0), n1);
    }
    const int up = lane + W < W * n1 ? win[lane + W] : lane < W * n1 ? newest[lane - W * (n1 - 1)] : 0;
    wave_sync();
    if (lane < W * n1) win[lane] = st->win[lane] = up;
    n_next = pool_order(p, sv, slots, cand, st->cand, lane);
    wave_sync();
  }
  build_block(st, W, N, n_next, L0 + e, Bp, last, win, cand, lane);
  if (lane == 0) {
    st->error = error;
    st->n_emitted = emitted_before + e;
    st->last_emitted = e;
    st->last_k = best_k;
    st->last_m = best_m;
    st->steps = steps + 1;
    st->matched_steps = matched + (best_m >= 1 ? 1 : 0);
    st->L = L0 + e;
    *kv_L = L0 + e;
    st->c0 = last;
    st->n_cand = n_next;
  }
}

// ---- Jacobi decoding (Section 4.2) --------------------------------------------------------------
// The block's rows: row 0 = c0 at position L, row i = guess y_i at L + i (i < k) under the plain
// causal mask; rows k.. carry nothing.  The guesses live in st->cand[0..k-1].
__device__ __forceinline__ void jacobi_build(la_step_state *st, int k, int t, int Bp, int c0, const int32_t *guess, int i) {
  if (i >= Bp) return;
  st->tok[i] = i >= k ? 0 : i == 0 ? c0 : guess[i - 1];
  st->pos[i] = i < k ? t + i : t + k - 1;
  st->vis[i] = i < k ? (2ull << i) - 1ull : 1ull << i;
}

__global__ __launch_bounds__(64) void jacobi_init_kernel(la_step_state *st, const int32_t *prompt, int P, int k, int Bp, int32_t *kv_L) {
  __shared__ int32_t guess[LA_MAX_ROWS];
  const int lane = threadIdx.x, c0 = prompt[P - 1];
  guess[lane] = c0;  // every position starts from the last committed token
  if (lane < k) st->cand[lane] = c0;
  __syncthreads();
  jacobi_build(st, k, P - 1, Bp, c0, guess, lane);
  if (lane == 0) {
    st->L = P - 1;
    st->c0 = c0;
    st->Bp = Bp;
    st->n_cand = k;
    st->steps = st->matched_steps = st->n_emitted = st->last_emitted = st->last_k = st->last_m = 0;
    st->error = st->reserved = 0;
    *kv_L = P - 1;
  }
}

// One pass's greedy ids become the new guesses (ids[i] is the prediction for position L + i + 1).  The block has
// converged when the pass returned its own input, and after k passes at the latest (pass j fixes guess j for good);
// it then commits: the pass's cache rows L.. were computed from the final tokens, so they stay and L advances.
// One wave, a guess per lane.
__global__ __launch_bounds__(64) void jacobi_accept_kernel(la_step_state *st, const int32_t *ids, int32_t *emitted, int max_total, int k,
                                                           int32_t *kv_L, const int32_t *err) {
  __shared__ int32_t guess[LA_MAX_ROWS];
  const int lane = threadIdx.x;
  const int id = lane < k ? ids[lane] : 0, old = lane < k ? st->cand[lane] : 0;
  const int before = st->n_emitted, passes = st->last_k + 1, steps = st->steps, matched = st->matched_steps, L0 = st->L, Bp = st->Bp, c0 = st->c0;
  const int error = *err;
  const int remaining = max_total - before;
  __syncthreads();
  if (lane == 0) st->error = error;
  if (remaining <= 0) {
    if (lane == 0) st->last_emitted = 0;
    return;
  }
  const bool commit = !__any(id != old) || passes >= k;
  const int e = k < remaining ? k : remaining;
  const int last = __shfl(id, e - 1, 64);
  guess[lane] = commit ? last : id;
  if (lane < k) st->cand[lane] = guess[lane];
  if (commit && lane < e) emitted[before + lane] = id;
  __syncthreads();
  jacobi_build(st, k, commit ? L0 + e : L0, Bp, commit ? last : c0, guess, lane);
  if (lane != 0) return;
  st->steps = steps + 1;
  st->last_emitted = commit ? e : 0;
  st->last_k = commit ? 0 : passes;
  if (!commit) return;
  st->n_emitted = before + e;
  st->last_m = passes;
  st->matched_steps = matched + 1;
  st->L = L0 + e;
  *kv_L = L0 + e;
  st->c0 = last;
}

}  // namespace la

using namespace la;

static int check_la(const la_lookahead_desc *d, int Bp) {
  LA_REQUIRE(d != nullptr, LA_EINVAL, "lookahead desc is NULL");
  LA_REQUIRE(d->N >= 1 && d->W >= 0 && d->G >= 0, LA_EINVAL, "bad lookahead parameters W=%d N=%d G=%d", d->W, d->N, d->G);
  LA_REQUIRE(d->N >= 2 || (d->G == 0), LA_EINVAL, "N=1 (sequential decoding) needs G=0");
  int rows = 1 + (d->W + d->G) * (d->N - 1);
  LA_REQUIRE(rows <= LA_MAX_ROWS, LA_EINVAL, "block of %d rows exceeds %d", rows, LA_MAX_ROWS);
  LA_REQUIRE(Bp >= rows && Bp <= LA_MAX_ROWS, LA_EINVAL, "Bp=%d must be in [%d, %d]", Bp, rows, LA_MAX_ROWS);
  return LA_OK;
}

extern "C" int la_lookahead_layout(const la_lookahead_desc *d, int t, int n_cand, int Bp, int32_t *pos_host,
                                   uint64_t *vis_host) {
  int rc = check_la(d, Bp);
  if (rc) return rc;
  LA_REQUIRE(pos_host && vis_host, LA_EINVAL, "NULL output");
  LA_REQUIRE(n_cand >= 0 && n_cand <= d->G, LA_EINVAL, "n_cand=%d outside [0, G=%d]", n_cand, d->G);
  block_layout(d->W, d->N, d->G, n_cand, t, Bp, pos_host, vis_host);
  return LA_OK;
}

extern "C" int la_pool_alloc(int vocab, int N, int G, la_pool **out) {
  LA_REQUIRE(out != nullptr, LA_EINVAL, "out is NULL");
  *out = nullptr;
  LA_REQUIRE(vocab > 0 && N >= 1 && G >= 0 && N <= LA_MAX_ROWS, LA_EINVAL, "bad pool shape vocab=%d N=%d G=%d", vocab, N, G);
  la_pool *p = new (std::nothrow) la_pool();
  LA_REQUIRE(p != nullptr, LA_ENOMEM, "out of host memory");
  p->vocab = vocab; p->N = N; p->G = G;
  size_t slots = (size_t)vocab * (G > 0 ? G : 1);
  size_t n1 = N > 1 ? N - 1 : 1;
  if (hipMalloc(&p->stamp, slots * sizeof(uint32_t)) != hipSuccess ||
      hipMalloc(&p->toks, slots * n1 * sizeof(int32_t)) != hipSuccess ||
      hipMalloc(&p->counter, sizeof(uint32_t)) != hipSuccess) {
    la_free_pool(p);
    set_error("pool allocation failed");
    return LA_ENOMEM;
  }
  *out = p;
  return LA_OK;
}

extern "C" void la_free_pool(la_pool *p) {
  if (!p) return;
  if (p->stamp) (void)hipFree(p->stamp);
  if (p->toks) (void)hipFree(p->toks);
  if (p->counter) (void)hipFree(p->counter);
  delete p;
}

static PoolView view(la_pool *p) { return PoolView{p->stamp, p->toks, p->counter, p->vocab, p->N, p->G}; }

extern "C" int la_state_init(la_pool *p, la_kv *kv, const la_lookahead_desc *d, const int32_t *prompt, int P, int Bp,
                             int seed_pool, la_step_state *state, void *stream) {
  LA_REQUIRE(p && kv && prompt && state, LA_EINVAL, "NULL argument");
  LA_PENDING(kv->m);
  int rc = check_la(d, Bp);
  if (rc) return rc;
  LA_REQUIRE(P >= 1, LA_EINVAL, "prompt must have at least one token");
  LA_REQUIRE(p->N == d->N && p->G == d->G, LA_EINVAL, "pool was allocated for N=%d G=%d", p->N, p->G);
  LA_REQUIRE(P - 1 + Bp <= kv->max_len, LA_ERANGE, "prompt of %d tokens + block of %d rows exceeds max_len %d", P, Bp, kv->max_len);
  hipStream_t s = (hipStream_t)stream;
  size_t slots = (size_t)p->vocab * (p->G > 0 ? p->G : 1);
  {
    ProfScope ps("pool_clear", s);
    fill_u32_kernel<<<1024, 256, 0, s>>>(p->stamp, slots, 0u);
  }
  const int grams = seed_pool && P >= d->N ? P - d->N + 1 : 0;
  if (grams > 0 && d->G > 0) {
    ProfScope ps("pool_seed", s);
    pool_seed_kernel<<<ceil_div(grams, 4), 256, 0, s>>>(view(p), prompt, grams);
  }
  {
    ProfScope ps("state_init", s);
    state_init_kernel<<<1, 64, 0, s>>>(view(p), state, prompt, P, d->W, d->N, d->G, Bp, (uint32_t)grams, kv->L_dev);
  }
  LA_HIP(hipGetLastError());
  kv->L_bound = P - 1;
  return LA_OK;
}

extern "C" int la_ngram_accept(la_pool *p, la_kv *kv, const la_lookahead_desc *d, const int32_t *ids,
                               la_step_state *state, int32_t *emitted, int max_total, void *stream) {
  LA_REQUIRE(p && kv && ids && state && emitted, LA_EINVAL, "NULL argument");
  LA_PENDING(kv->m);
  int rc = check_la(d, 1 + (d ? (d->W + d->G) * (d->N - 1) : 0));
  if (rc) return rc;
  LA_REQUIRE(p->N == d->N && p->G == d->G, LA_EINVAL, "pool was allocated for N=%d G=%d", p->N, p->G);
  LA_REQUIRE(max_total >= 0, LA_EINVAL, "max_total < 0");
  hipStream_t s = (hipStream_t)stream;
  {
    ProfScope ps("ngram_accept", s);
    const la_model_desc &md = kv->m->d;
    const dim3 grid(d->N >= 2 ? kv->n_layers : 1, d->N >= 2 ? d->N - 1 : 1);
    if (md.dtype == LA_F32)
      accept_kernel<float><<<grid, 256, 0, s>>>(view(p), state, ids, emitted, max_total, d->W, d->N, d->G, kv->L_dev, kv->err_dev, (float *)kv->K,
                                                (float *)kv->V, kv->layer_elems(), md.n_kv_heads, md.head_dim, kv->v_blocked, kv->max_len);
    else
      accept_kernel<uint16_t><<<grid, 256, 0, s>>>(view(p), state, ids, emitted, max_total, d->W, d->N, d->G, kv->L_dev, kv->err_dev, (uint16_t *)kv->K,
                                                   (uint16_t *)kv->V, kv->layer_elems(), md.n_kv_heads, md.head_dim, kv->v_blocked, kv->max_len);
  }
  LA_HIP(hipGetLastError());
  kv->L_bound += d->N;
  return LA_OK;
}

extern "C" int la_jacobi_init(la_kv *kv, int k, const int32_t *prompt, int P, int Bp, la_step_state *state, void *stream) {
  LA_REQUIRE(kv && prompt && state, LA_EINVAL, "NULL argument");
  LA_PENDING(kv->m);
  LA_REQUIRE(k >= 1 && k <= Bp && Bp <= LA_MAX_ROWS, LA_EINVAL, "need 1 <= k=%d <= Bp=%d <= %d", k, Bp, LA_MAX_ROWS);
  LA_REQUIRE(P >= 1, LA_EINVAL, "prompt must have at least one token");
  LA_REQUIRE(P - 1 + Bp <= kv->max_len, LA_ERANGE, "prompt of %d tokens + block of %d rows exceeds max_len %d", P, Bp, kv->max_len);
  hipStream_t s = (hipStream_t)stream;
  {
    ProfScope ps("jacobi_init", s);
    jacobi_init_kernel<<<1, 64, 0, s>>>(state, prompt, P, k, Bp, kv->L_dev);
  }
  LA_HIP(hipGetLastError());
  kv->L_bound = P - 1;
  return LA_OK;
}

extern "C" int la_jacobi_accept(la_kv *kv, int k, const int32_t *ids, la_step_state *state, int32_t *emitted, int max_total,
                                void *stream) {
  LA_REQUIRE(kv && ids && state && emitted, LA_EINVAL, "NULL argument");
  LA_PENDING(kv->m);
  LA_REQUIRE(k >= 1 && k <= LA_MAX_ROWS, LA_EINVAL, "k=%d outside [1, %d]", k, LA_MAX_ROWS);
  LA_REQUIRE(max_total >= 0, LA_EINVAL, "max_total < 0");
  hipStream_t s = (hipStream_t)stream;
  {
    ProfScope ps("jacobi_accept", s);
    jacobi_accept_kernel<<<1, 64, 0, s>>>(state, ids, emitted, max_total, k, kv->L_dev, kv->err_dev);
  }
  LA_HIP(hipGetLastError());
  kv->L_bound += k;
  return LA_OK;
}
