// Non-contraction kernels of the RNNLM step: stream indexing, token checks, embedding gather,
// softmax statistics merge, fused softmax-gradient pass, split-K reduction, sort/segment helpers
// and the segmented embedding update.
#pragma once
#include "common.h"

namespace rnnlm_dev {

// ---- a0: data-offset stream indexing (Sec. 4.2) ------------------------------------------------
__global__ void stream_chunk_kernel(const int32_t *__restrict__ tok, long L, long k, int T, int B,
                                    int32_t *__restrict__ x, int32_t *__restrict__ y) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= T * B) return;
  const int t = i / B, s = i % B;
  const long p = (long)s * L + k * T + t;
  x[i] = tok[p];
  y[i] = tok[p + 1];
}

// First kernel of a window, two kinds of workgroups:
// blockIdx.x < prep_blocks: token check + re-layout into the padded window: xp/yp[t*Bp + s]; padding rows
//   get -1.  Ids outside [0, V) are clamped and raise flags[0].  Also marks padded positions with
//   lse = +inf so that the softmax-gradient pass produces exact zeros there, copies the carried state into
//   slot 0 of the hidden-state buffer (compute type, padded with zeros) and clears the barrier / ticket
//   counters of the persistent recurrent kernel that follows (slot / counters == nullptr: tokens only).  Also
//   gives the exchange buffers of the persistent recurrent kernels (ring[0] forward, ring[1] backward; nullptr: none)
//   their first contents: UNWRITTEN, and the carried state, in operand order, as the forward step before the first.
//   prep_blocks covers max(Mp, Bp*Hp, ring pieces of 16 bytes, SYNC_WORDS) threads.
// blockIdx.x >= prep_blocks (present when X or Xc != nullptr), padded row r = blockIdx.x - prep_blocks:
//   - a1, embedding gather (r < T*Bp): X[r][:] = E[x of that position][:] (fp32), zero on padding.  Compressed
//     architecture (Xc != nullptr): the row is an operand of the contraction through the layer below the
//     state, so it is copied in the compute type from the tile-padded compute copy Ec[.][ldc] into Xc[r][ldc];
//   - zeros where the persistent recurrent kernels write nothing but the contractions read: padding positions, and
//     units from `width` on, of the state (next, r < T*Bp) and of the gradient (dA, training windows).
constexpr unsigned UNWRITTEN = 0xffffffffu;  // an exchanged word that its step has not written yet
constexpr int RING = 4;                      // steps the exchange buffer holds

// How the persistent recurrent kernel covers a shape (nwg = 0: it does not).
struct RecurrentPlan {
  int waves, units, nwg;  // per workgroup; workgroups per group
  int R, groups, rt;      // streams per group, groups, blocks of 16 streams per group
  int width;              // units the kernel writes: H rounded up to whole workgroups
  int nkb, ks;            // 32-wide blocks of the contraction, and how many a wave takes
  __host__ __device__ long ring_bytes(int es) const { return (long)RING * groups * rt * nkb * 512 * es; }
};

template <typename T>
struct PrepWindow {
  const int32_t *x, *y;
  int Tn, B, Bp, Mp, V;
  int32_t *xp, *yp;
  float *lse;
  int32_t *flags;
  const float *h_state;
  int H, Hp;
  T *slot;
  unsigned *counters;
  int prep_blocks;
  const float *E;
  float *X;
  const T *Ec;
  int ldc;
  T *Xc;
  T *next, *dA;
  RecurrentPlan plan;
  char *ring[2];
};

template <typename T>
__global__ void __launch_bounds__(256) prep_tokens_kernel(const PrepWindow<T> p) {
  const int B = p.B, Bp = p.Bp, H = p.H, Hp = p.Hp;
  if ((int)blockIdx.x >= p.prep_blocks) {
    const int row = blockIdx.x - p.prep_blocks;
    const int t = row / Bp, s = row % Bp;
    const bool valid = t < p.Tn && s < B;
    if (p.next) {
      const int n16 = Hp * (int)sizeof(T) / 16, first = valid ? p.plan.width * (int)sizeof(T) / 16 : 0;
      const u32x4_t zero = {0u, 0u, 0u, 0u};
      for (int c = first + threadIdx.x; c < n16; c += 256) {
        if (t < p.Tn) reinterpret_cast<u32x4_t *>(p.next + (long)row * Hp)[c] = zero;
        if (p.dA) reinterpret_cast<u32x4_t *>(p.dA + (long)row * Hp)[c] = zero;
      }
    }
    if (t >= p.Tn) return;
    int w = -1;
    if (valid) w = min(max(p.x[t * B + s], 0), p.V - 1);
    if (p.Xc) {
      const u32x4_t *src16 = reinterpret_cast<const u32x4_t *>(p.Ec + (long)max(w, 0) * p.ldc);
      u32x4_t *dst16 = reinterpret_cast<u32x4_t *>(p.Xc + (long)row * p.ldc);
      const int n16 = p.ldc * (int)sizeof(T) / 16;
      const u32x4_t zero = {0u, 0u, 0u, 0u};
      for (int c = threadIdx.x; c < n16; c += 256) dst16[c] = (w >= 0) ? src16[c] : zero;
      return;
    }
    const float *src = p.E + (long)max(w, 0) * H;
    float *dst = p.X + (long)row * Hp;
    if ((H & 3) == 0) {
      for (int c = threadIdx.x * 4; c < Hp; c += 256 * 4) {
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (w >= 0 && c < H) v = *reinterpret_cast<const float4 *>(src + c);
        *reinterpret_cast<float4 *>(dst + c) = v;
      }
    } else {
      for (int c = threadIdx.x; c < Hp; c += 256) dst[c] = (w >= 0 && c < H) ? src[c] : 0.0f;
    }
    return;
  }
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (p.counters && i < SYNC_WORDS) p.counters[i] = 0u;
  if (p.slot && i < (long)Bp * Hp) {
    const int s = (int)(i / Hp), c = (int)(i % Hp);
    p.slot[i] = from_f32<T>((s < B && c < H) ? p.h_state[(long)s * H + c] : 0.0f);
  }
  if (p.ring[0] && i < p.plan.ring_bytes(sizeof(T)) / 16) {
    constexpr int E16 = 16 / (int)sizeof(T), PIECES = 2 / (E16 / 4);  // values in 16 bytes; pieces of a fragment
    const u32x4_t unwritten = {UNWRITTEN, UNWRITTEN, UNWRITTEN, UNWRITTEN};
    const RecurrentPlan &q = p.plan;
    const long per = q.ring_bytes(sizeof(T)) / 16 / RING;
    u32x4_t v = unwritten;
    if (i / per == RING - 1) {  // what step 0 reads
      long c = i % per;
      const int l = (int)(c & 63);
      c >>= 6;
      const int piece = (int)(c % PIECES);
      c /= PIECES;
      const int kb = (int)(c % q.nkb);
      c /= q.nkb;
      const int r = (int)(c % q.rt) * 16 + (l & 15), s = (int)(c / q.rt) * q.R + r;
      const int unit = kb * 32 + (l >> 4) * 8 + piece * E16;
      union {
        u32x4_t u;
        T t[E16];
      } o;
#pragma unroll
      for (int e = 0; e < E16; ++e)
        o.t[e] = from_f32<T>((r < q.R && s < B && unit + e < H) ? p.h_state[(long)s * H + unit + e] : 0.0f);
      v = o.u;
    }
    reinterpret_cast<u32x4_t *>(p.ring[0])[i] = v;
    if (p.ring[1]) reinterpret_cast<u32x4_t *>(p.ring[1])[i] = unwritten;
  }
  if (i >= p.Mp) return;
  const int t = (int)i / Bp, s = (int)i % Bp;
  int xv = -1, yv = -1;
  if (t < p.Tn && s < B) {
    xv = p.x[t * B + s];
    yv = p.y ? p.y[t * B + s] : 0;
    if (xv < 0 || xv >= p.V || yv < 0 || yv >= p.V) {
      p.flags[0] = 1;
      xv = min(max(xv, 0), p.V - 1);
      yv = min(max(yv, 0), p.V - 1);
    }
  } else {
    p.lse[i] = INFINITY;
  }
  p.xp[i] = xv;
  if (p.yp) p.yp[i] = yv;
}

template <typename T>
__global__ void fill_kernel(T *__restrict__ p, long n, T v) {
  long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long stride = (long)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = v;
}

// fp32 master -> padded compute copy.
template <typename T>
__global__ void to_compute_copy_kernel(const float *__restrict__ W, int R, int C, int Cp, long n,
                                       T *__restrict__ Wc) {
  long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long stride = (long)gridDim.x * blockDim.x;
  for (; i < n; i += stride) {
    const long r = i / Cp;
    const int c = (int)(i % Cp);
    Wc[i] = from_f32<T>((r < R && c < C) ? W[r * C + c] : 0.0f);
  }
}

// Square transpose of a compute-type matrix (n x n, n a multiple of 32): dst[c][r] = src[r][c].
template <typename T>
__global__ void __launch_bounds__(256) transpose_kernel(const T *__restrict__ src, int n, T *__restrict__ dst) {
  __shared__ T tile[32][33];
  const int bx = blockIdx.x * 32, by = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int r = ty; r < 32; r += 8) tile[r][tx] = src[(long)(by + r) * n + bx + tx];
  __syncthreads();
  for (int r = ty; r < 32; r += 8) dst[(long)(bx + r) * n + by + tx] = tile[tx][r];
}

// ---- a2 / a8, per-step path for hidden sizes beyond the persistent kernel: the step's contraction runs
// split over the contraction dimension (so that every compute unit gets a workgroup and each operand panel
// is fetched by few of them); these kernels sum the partial products in a fixed order and apply the step's
// elementwise part.  n4 = Bp*Hp/4 groups of 4 columns; part[split][rows][Hp], rows >= Bp of whole tiles (split_stride).
template <typename T>
__global__ void rnn_step_fwd_kernel(const float *__restrict__ part, long split_stride, int splits,
                                    const float *__restrict__ X, int B, int H, int Hp, long n4,
                                    T *__restrict__ Hnext, float *__restrict__ h_state) {
  const long i4 = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i4 >= n4) return;
  const long i = i4 * 4;
  const int row = (int)(i / Hp), col = (int)(i % Hp);
  f32x4_t a = *reinterpret_cast<const f32x4_t *>(part + i);
  for (int s = 1; s < splits; ++s) a += *reinterpret_cast<const f32x4_t *>(part + (long)s * split_stride + i);
  const f32x4_t x = *reinterpret_cast<const f32x4_t *>(X + i);
  f32x4_t hv;
#pragma unroll
  for (int e = 0; e < 4; ++e) hv[e] = (row < B && col + e < H) ? sigmoidf_(a[e] + x[e]) : 0.0f;
  if constexpr (sizeof(T) == 2) {
    bf16x4_t o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (bf16_t)hv[e];
    *reinterpret_cast<bf16x4_t *>(Hnext + i) = o;
  } else {
    *reinterpret_cast<f32x4_t *>(Hnext + i) = hv;
  }
  if (h_state && row < B)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (col + e < H) h_state[(long)row * H + col + e] = hv[e];
}

template <typename T>
__global__ void rnn_step_bwd_kernel(const float *__restrict__ part, long split_stride, int splits,
                                    const float *__restrict__ dHs, const T *__restrict__ Hs, int B, int H, int Hp,
                                    long n4, float *__restrict__ dA32, T *__restrict__ dAc) {
  const long i4 = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i4 >= n4) return;
  const long i = i4 * 4;
  const int row = (int)(i / Hp), col = (int)(i % Hp);
  f32x4_t a = {0.0f, 0.0f, 0.0f, 0.0f};
  for (int s = 0; s < splits; ++s) a += *reinterpret_cast<const f32x4_t *>(part + (long)s * split_stride + i);
  const f32x4_t g = *reinterpret_cast<const f32x4_t *>(dHs + i);
  f32x4_t d;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float hv = to_f32(Hs[i + e]);
    d[e] = (row < B && col + e < H) ? (g[e] + a[e]) * hv * (1.0f - hv) : 0.0f;
  }
  *reinterpret_cast<f32x4_t *>(dA32 + i) = d;
  if constexpr (sizeof(T) == 2) {
    bf16x4_t o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (bf16_t)d[e];
    *reinterpret_cast<bf16x4_t *>(dAc + i) = o;
  } else {
    *reinterpret_cast<f32x4_t *>(dAc + i) = d;
  }
}

// Sum of n log-probabilities in fp64 with a fixed reduction tree, by a workgroup; raises flags[1] when
// the result is not finite.  counters != nullptr: also clears the counters of the persistent recurrent kernel (the sum
// sits between its forward and its backward launch).
struct WindowSum {
  double *out, *running;  // either may be nullptr: the sum, and what it is added to
  int32_t *flags;
  unsigned *counters;
};
template <int THREADS = 1024, class Load>
__device__ inline void window_sum(const WindowSum &w, int n, Load &&load) {
  constexpr int WAVES = THREADS / 64;
  __shared__ double sh[WAVES];
  if (w.counters)
    for (int i = threadIdx.x; i < SYNC_WORDS; i += THREADS) w.counters[i] = 0u;
  double a = 0.0;
  for (int i = threadIdx.x; i < n; i += THREADS) a += (double)load(i);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = a;
  __syncthreads();
  if (threadIdx.x < WAVES) {
    a = sh[threadIdx.x];
#pragma unroll
    for (int o = WAVES / 2; o > 0; o >>= 1) a += __shfl_xor(a, o, 64);
  }
  if (threadIdx.x == 0) {
    const double s = a;
    if (w.out) *w.out = s;
    if (w.running) *w.running += s;
    if (!(s == s) || s - s != 0.0) w.flags[1] = 1;
  }
}
// ---- a4 (part 1): merge the per-row-block (max, sum exp) partials of each position into the log
// normaliser, and form log P(target) = z_target - lse (Sec. 4.2: explicitly normalised output).
// Workgroup = MERGE_M positions x 1024 / MERGE_M groups of partials: a group is merged sequentially in a fixed order,
// the four groups of a wave by exchanges between its lanes, then the 16 waves' results in order.  Bound by memory
// latency: with 64 positions per workgroup 2560 positions ran on 40 compute units (9.5 us, and 5 for the sum; here 8 for both).
// done != nullptr: the last workgroup to finish also forms the window's sum (a launch of its own took 4-5 us): the
// log-probabilities it adds up move with agent-scope accesses, each workgroup's before its arrival at the counter.
constexpr int MERGE_M = 16;
__global__ void __launch_bounds__(1024) merge_stats_kernel(const float2 *__restrict__ part, int nPart, long ldz, int T,
                                                           int B, int Bp, const float *__restrict__ zy,
                                                           float *__restrict__ lse, float *__restrict__ logp_int,
                                                           float *__restrict__ logp_out, unsigned *__restrict__ done,
                                                           const WindowSum w) {
  constexpr int GROUPS = 1024 / MERGE_M;
  __shared__ float2 sh[16][MERGE_M];
  __shared__ int last;
  const int pos = threadIdx.x % MERGE_M, grp = threadIdx.x / MERGE_M;
  const int m = blockIdx.x * MERGE_M + pos;
  const bool valid = m < T * Bp;
  float mx = -INFINITY, sum = 0.0f;
  auto merge = [&](const float2 q) {
    if (q.y > 0.0f) {
      const float nmx = fmaxf(mx, q.x);
      sum = sum * __expf(mx - nmx) + q.y * __expf(q.x - nmx);
      mx = nmx;
    }
  };
  if (valid) {
    int p = grp;
    for (; p + 3 * GROUPS < nPart; p += 4 * GROUPS) {  // four partials per round: their loads are independent
      float2 q[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) q[u] = part[(long)(p + GROUPS * u) * ldz + m];
#pragma unroll
      for (int u = 0; u < 4; ++u) merge(q[u]);
    }
    for (; p < nPart; p += GROUPS) merge(part[(long)p * ldz + m]);
  }
#pragma unroll
  for (int o = MERGE_M; o < 64; o <<= 1) {
    float2 q;
    q.x = __shfl_xor(mx, o, 64);
    q.y = __shfl_xor(sum, o, 64);
    merge(q);
  }
  if ((threadIdx.x & 63) < MERGE_M) sh[threadIdx.x >> 6][pos] = make_float2(mx, sum);
  __syncthreads();
  const int t = m / Bp, s = m % Bp;
  if (threadIdx.x < MERGE_M && valid && s < B) {  // padding keeps lse = +inf
    for (int g = 1; g < 16; ++g) merge(sh[g][pos]);
    const float l = mx + __logf(sum);
    lse[m] = l;
    const float lp = zy[m] - l;
    __hip_atomic_store(logp_int + t * B + s, lp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (logp_out) logp_out[t * B + s] = lp;
  }
  if (!done) return;
  if (threadIdx.x < 64) {  // the wave that stored: its stores are acknowledged before the arrival
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (threadIdx.x == 0)
      last = __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == gridDim.x;
  }
  __syncthreads();
  if (!last) return;
  window_sum(w, T * B, [&](int i) { return __hip_atomic_load(logp_int + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); });
}

// ---- a4 (part 2) + a5: fused softmax gradient, in place on the vocabulary-major logits ----------
//   dz[v][m] = (exp(z[v][m] - lse[m]) - [v == y[m]]) / M      (gradient of the mean NLL)
//   db[v]    = sum_m dz[v][m];   b_out[v] = alpha*b[v] - lr*db[v]
// One wavefront owns ROWS_PER_WAVE vocabulary rows and walks the window positions once, so the
// per-position lse / target id loaded for a 16-byte column chunk serve all of its rows and several row
// loads are in flight per lane.  Rows v >= V and padded positions (lse = +inf) become zero.  Workgroups take the
// vocabulary from its top down, so that what this pass writes last is what the contraction over the vocabulary
// that follows reads first (still in the memory-side cache: 1-3 % on that contraction).
// MERGE: every workgroup first merges the statistics of the positions for itself, and the first one also forms the
// log-probabilities and their sum (merge_stats_kernel's work).  Where there are few (SHORT_STATS) that takes less than the
// launch it saves: fp32 V = 1000, H = 64, 4x8 a window of 49.3 us without and 46.0 with it; bf16, one position, 40.5 and 32.7.
constexpr int SHORT_POSITIONS = 256, SHORT_STATS = 4096;
struct StatsMerge {
  const float2 *part;
  int nPart, T, B, Bp;
  const float *zy;
  float *logp_int, *logp_out;
  WindowSum sum;
};
template <typename T, bool MERGE>
__global__ void __launch_bounds__(256) softmax_grad_kernel(T *__restrict__ ZT, long ldz, int Mp, int V, int Vp,
                                                           const float *__restrict__ lse,
                                                           const int32_t *__restrict__ yp, float invM,
                                                           const float *__restrict__ b, float *__restrict__ b_out,
                                                           float alpha, float lr, const StatsMerge s) {
  __shared__ __attribute__((aligned(16))) float l_sh[MERGE ? SHORT_POSITIONS : 4];
  if constexpr (MERGE) {
    constexpr int FLIGHT = 8;
    __shared__ float2 sh[4][64];
    const int pos = threadIdx.x & 63, grp = threadIdx.x >> 6;  // (Mp is a multiple of 64)
    auto merge = [](float2 a, const float2 q) {
      if (!(q.y > 0.0f)) return a;
      const float m = fmaxf(a.x, q.x);
      return make_float2(m, a.y * __expf(a.x - m) + q.y * __expf(q.x - m));
    };
    for (int m0 = 0; m0 < Mp; m0 += 64) {
      float2 a = make_float2(-INFINITY, 0.0f);
      for (int p = grp; p < s.nPart; p += 4 * FLIGHT) {
        float2 q[FLIGHT];
#pragma unroll
        for (int u = 0; u < FLIGHT; ++u)
          q[u] = p + 4 * u < s.nPart ? s.part[(long)(p + 4 * u) * Mp + m0 + pos] : make_float2(-INFINITY, 0.0f);
#pragma unroll
        for (int u = 0; u < FLIGHT; ++u) a = merge(a, q[u]);
      }
      sh[grp][pos] = a;
      __syncthreads();
      if (grp == 0) {
#pragma unroll
        for (int g = 1; g < 4; ++g) a = merge(a, sh[g][pos]);
        const int m = m0 + pos, t = m / s.Bp, st = m % s.Bp;
        const bool valid = t < s.T && st < s.B;
        const float l = valid ? a.x + __logf(a.y) : INFINITY;  // padding: zeros below
        l_sh[m] = l;
        if (valid && blockIdx.x == 0) {
          const float lp = s.zy[m] - l;
          s.logp_int[t * s.B + st] = lp;
          if (s.logp_out) s.logp_out[t * s.B + st] = lp;
        }
      }
      __syncthreads();
    }
    if (blockIdx.x == 0) window_sum<256>(s.sum, s.T * s.B, [&](int i) {
      const int m = (i / s.B) * s.Bp + i % s.B;
      return s.zy[m] - l_sh[m];
    });
  }
  constexpr int VEC = Elem<T>::VEC;
  constexpr int R = 4;  // rows per wave
  const int lane = threadIdx.x & 63;
  const int v0 = ((gridDim.x - 1 - blockIdx.x) * 4 + (threadIdx.x >> 6)) * R;
  if (v0 >= Vp) return;
  T *row = ZT + (long)v0 * ldz;
  float db[R];
#pragma unroll
  for (int r = 0; r < R; ++r) db[r] = 0.0f;
  for (int c = lane * VEC; c < Mp; c += 64 * VEC) {
    u32x4_t raw[R];
#pragma unroll
    for (int r = 0; r < R; ++r) raw[r] = *reinterpret_cast<const u32x4_t *>(row + (long)r * ldz + c);
    float l[VEC];
    int y[VEC];
#pragma unroll
    for (int e = 0; e < VEC; e += 4) {
      const f32x4_t lv = *reinterpret_cast<const f32x4_t *>((MERGE ? l_sh : lse) + c + e);
      const u32x4_t yv = *reinterpret_cast<const u32x4_t *>(yp + c + e);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        l[e + q] = lv[q];
        y[e + q] = (int)yv[q];
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      union {
        u32x4_t u;
        T t[VEC];
      } in, o;
      in.u = raw[r];
      const int v = v0 + r;
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        float p = __expf(to_f32(in.t[e]) - l[e]);
        if (y[e] == v) p -= 1.0f;
        p = (v < V) ? p * invM : 0.0f;
        db[r] += p;
        o.t[e] = from_f32<T>(p);
      }
      *reinterpret_cast<u32x4_t *>(row + (long)r * ldz + c) = o.u;
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    float d = db[r];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) d += __shfl_xor(d, o, 64);
    const int v = v0 + r;
    if (lane == 0 && v < V) b_out[v] = ((alpha != 0.0f) ? alpha * b[v] : 0.0f) - lr * d;
  }
}

// ---- a6: fixed-order reduction of the split-K partial sums -------------------------------------
// T: what the sum is stored as (the compressed architecture wants a contraction operand; converted by a launch of its own it
// took 5 us more of a 2560-position window, P = 512).
template <typename T>
__device__ inline void store_sum4(T *out, f32x4_t v) {
  if constexpr (sizeof(T) == 2) {
    bf16x4_t h;
#pragma unroll
    for (int e = 0; e < 4; ++e) h[e] = (bf16_t)v[e];
    *reinterpret_cast<bf16x4_t *>(out) = h;
  } else {
    *reinterpret_cast<f32x4_t *>(out) = v;
  }
}
template <typename T>
__global__ void splitk_reduce_kernel(const float *__restrict__ part, long n, int splits, T *__restrict__ out) {
  const long i = ((long)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (i >= n) return;
  f32x4_t a = *reinterpret_cast<const f32x4_t *>(part + i);
  constexpr int FLIGHT = 5;
  for (int s = 1; s < splits; s += FLIGHT) {  // (loads left in the loop one by one would wait for one another)
    f32x4_t v[FLIGHT];
#pragma unroll
    for (int q = 0; q < FLIGHT; ++q)
      if (s + q < splits) v[q] = *reinterpret_cast<const f32x4_t *>(part + (s + q) * n + i);
#pragma unroll
    for (int q = 0; q < FLIGHT; ++q)
      if (s + q < splits) a += v[q];
  }
  store_sum4(out + i, a);
}

// Many parts (more than 16) of a small output: bound by memory latency.  The waves of a workgroup share out the parts of 256
// values, eight in flight a lane, and the four sums are added in order.
template <typename T>
__global__ void __launch_bounds__(256) splitk_reduce_many_kernel(const float *__restrict__ part, long n, int splits,
                                                                 T *__restrict__ out) {
  constexpr int WAVES = 4, FLIGHT = 8;
  __shared__ f32x4_t sh[WAVES][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long i = ((long)blockIdx.x * 64 + lane) * 4;
  f32x4_t a = {0.0f, 0.0f, 0.0f, 0.0f};
  if (i < n) {
    const int per = (splits + WAVES - 1) / WAVES, s1 = min((wave + 1) * per, splits);
    for (int s = wave * per; s < s1; s += FLIGHT) {
      f32x4_t v[FLIGHT];
#pragma unroll
      for (int q = 0; q < FLIGHT; ++q)
        if (s + q < s1) v[q] = *reinterpret_cast<const f32x4_t *>(part + (s + q) * n + i);
#pragma unroll
      for (int q = 0; q < FLIGHT; ++q)
        if (s + q < s1) a += v[q];
    }
  }
  sh[wave][lane] = a;
  __syncthreads();
  if (wave != 0 || i >= n) return;
#pragma unroll
  for (int q = 1; q < WAVES; ++q) a += sh[q][lane];
  store_sum4(out + i, a);
}

// ---- a10 helpers (integer-exact): stable order of window positions by input id ------------------
// rank[m] = #{m' : (x[m'], m') < (x[m], m)};  perm[rank[m]] = m.
// Block = 64 positions x 16 slices of the key array (1024 threads).
__global__ void __launch_bounds__(1024) rank_sort_kernel(const int32_t *__restrict__ xp, int M, int B, int Bp,
                                                         int32_t *__restrict__ perm) {
  __shared__ int32_t keys[4096];
  __shared__ int32_t cnt[16][64];
  const int lane = threadIdx.x & 63, slice = threadIdx.x >> 6;
  const int m = blockIdx.x * 64 + lane;
  const int mykey = (m < M) ? xp[(m / B) * Bp + (m % B)] : 0;
  int rank = 0;
  for (int base = 0; base < M; base += 4096) {
    const int n = min(4096, M - base);
    for (int i = threadIdx.x; i < n; i += 1024) {
      const int mm = base + i;
      keys[i] = xp[(mm / B) * Bp + (mm % B)];
    }
    __syncthreads();
    for (int i = slice; i < n; i += 16) {
      const int k = keys[i];
      rank += (k < mykey) || (k == mykey && base + i < m);
    }
    __syncthreads();
  }
  cnt[slice][lane] = rank;
  __syncthreads();
  if (slice == 0 && m < M) {
    int r = 0;
    for (int g = 0; g < 16; ++g) r += cnt[g][lane];
    perm[r] = m;
  }
}

// Run starts of equal ids in sorted order; single workgroup of 1024 threads, fixed scan order.
__global__ void segment_kernel(const int32_t *__restrict__ xp, const int32_t *__restrict__ perm, int M, int B,
                               int Bp, int32_t *__restrict__ seg_start, int32_t *__restrict__ nseg) {
  __shared__ int32_t sc[1024];
  __shared__ int32_t carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int base = 0; base < M; base += 1024) {
    const int r = base + threadIdx.x;
    int head = 0;
    if (r < M) {
      const int m = perm[r];
      const int k = xp[(m / B) * Bp + (m % B)];
      if (r == 0) {
        head = 1;
      } else {
        const int mq = perm[r - 1];
        head = xp[(mq / B) * Bp + (mq % B)] != k;
      }
    }
    sc[threadIdx.x] = head;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
      int add = 0;
      if ((int)threadIdx.x >= off) add = sc[threadIdx.x - off];
      __syncthreads();
      sc[threadIdx.x] += add;
      __syncthreads();
    }
    const int incl = sc[threadIdx.x];
    const int c0 = carry;
    if (head) seg_start[c0 + incl - 1] = r;
    __syncthreads();
    if (threadIdx.x == 1023) carry = c0 + incl;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    seg_start[carry] = M;
    *nseg = carry;
  }
}

// ---- a10: sums over the members of a run, atomic-free and order-fixed ----------------------------
// The row updates (embedding rows here, touched output rows in nce.h) add up, per word, one source row per member of
// the word's run.  They are made of dependent round trips (run bounds -> positions -> coefficients -> rows) and a
// Zipf text has runs of one member by the thousand and a few of hundreds, so a wave sums a short run by itself, over 256
// columns, and the RUN_WAVES waves of a workgroup share out a run of more than RUN_ALONE members in slices.  A wave
// loads 64 members' positions at once, one a lane, and then has RUN_FLIGHT rows in flight.  Member i of a slice goes to
// sum i mod RUN_FLIGHT, the sums are added as a tree, slices in order: results are bitwise reproducible.
// H = 1024, 2560 positions: embedding rows 34 -> 11 us (a workgroup of four waves took a run, one row group of 16 after the
// other), the noise-contrastive update of 3584 entries 56 -> 16 us (sixteen waves a run, most of them idle).
constexpr int RUN_WAVES = 8, RUN_ALONE = 16, RUN_FLIGHT = 8, RUN_COLS = 256;
struct RunSum {
  f32x4_t part[RUN_FLIGHT];
  __device__ RunSum() {
#pragma unroll
    for (int q = 0; q < RUN_FLIGHT; ++q) part[q] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
  }
  // members i = first .. n-1, the same in every lane: raw(i) asks for a member's row, add(i, value, sum) takes it up
  template <class Raw, class Add>
  __device__ void take(int first, int n, Raw raw, Add add) {
    for (int i = first; i < n; i += RUN_FLIGHT) {
      decltype(raw(0)) v[RUN_FLIGHT];
#pragma unroll
      for (int q = 0; q < RUN_FLIGHT; ++q)
        if (i + q < n) v[q] = raw(i + q);
#pragma unroll
      for (int q = 0; q < RUN_FLIGHT; ++q)
        if (i + q < n) add(i + q, v[q], part[q]);
    }
  }
  __device__ f32x4_t total() const {
    return ((part[0] + part[1]) + (part[2] + part[3])) + ((part[4] + part[5]) + (part[6] + part[7]));
  }
};

// Four columns of an updated row: out = alpha * old - lr * sum.  ALIGNED: 16-byte accesses; otherwise element by element,
// the last group partly (rows of H values; the compute copy's rows are padded).
template <bool ALIGNED>
__device__ inline f32x4_t load_row4(const float *__restrict__ row, int col, int H) {
  f32x4_t v = {0.0f, 0.0f, 0.0f, 0.0f};
  if (ALIGNED) {
    if (col < H) v = *reinterpret_cast<const f32x4_t *>(row + col);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (col + e < H) v[e] = row[col + e];
  }
  return v;
}
template <bool ALIGNED, typename T>
__device__ inline void store_row4(f32x4_t v, int col, int H, float *__restrict__ row, T *__restrict__ copy) {
  if (col >= H) return;
  if (ALIGNED) {
    *reinterpret_cast<f32x4_t *>(row + col) = v;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (col + e < H) row[col + e] = v[e];
  }
  if (!copy) return;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (ALIGNED || col + e < H) copy[col + e] = from_f32<T>(v[e]);
}

// The runs of a workgroup: runs blockIdx.x + k * gridDim.x, k < RUN_WAVES (frequent words often lie side by side: a
// workgroup takes runs that are far apart).  request(r0) asks for what is updated, sum(r0, r1) is a wave's sum over members
// [r0, r1) of the sorted list, finish(run, requested, sum) stores the run's result.
struct RowSum {
  f32x4_t v;  // the lane's four columns
  float b;    // a term of the whole row (bias), the same in every lane
};
struct RunShared {  // the slices' sums of a run that the waves share out
  f32x4_t v[RUN_WAVES][64];
  float b[RUN_WAVES];
};
template <class Request, class Sum, class Finish>
__device__ inline void walk_runs(const int32_t *__restrict__ seg_start, int nseg, RunShared &shared, Request request, Sum sum,
                                 Finish finish) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int run = (int)blockIdx.x + (lane % RUN_WAVES) * (int)gridDim.x;
  const int lo = run < nseg ? seg_start[run] : 0, hi = run < nseg ? seg_start[run + 1] : 0;
  {
    const int r0 = __builtin_amdgcn_readlane(lo, wave), r1 = __builtin_amdgcn_readlane(hi, wave);
    if (r1 > r0 && r1 - r0 <= RUN_ALONE) {
      const auto old = request(r0);
      finish((int)blockIdx.x + wave * (int)gridDim.x, old, sum(r0, r1));
    }
  }
  for (int k = 0; k < RUN_WAVES; ++k) {
    const int r0 = __builtin_amdgcn_readlane(lo, k), r1 = __builtin_amdgcn_readlane(hi, k);
    if (r1 - r0 <= RUN_ALONE) continue;  // (the same in every wave)
    const int per = (r1 - r0 + RUN_WAVES - 1) / RUN_WAVES, s0 = min(r0 + wave * per, r1), s1 = min(s0 + per, r1);
    const auto old = request(r0);
    const RowSum mine = sum(s0, s1);
    __syncthreads();  // the sums of the shared run before have been read
    shared.v[wave][lane] = mine.v;
    if (lane == 0) shared.b[wave] = mine.b;
    __syncthreads();
    if (wave == k) {
      RowSum tot = {shared.v[0][lane], shared.b[0]};
#pragma unroll
      for (int q = 1; q < RUN_WAVES; ++q) {
        tot.v += shared.v[q][lane];
        tot.b += shared.b[q];
      }
      finish((int)blockIdx.x + k * (int)gridDim.x, old, tot);
    }
  }
}

// ---- a10: segmented embedding update, atomic-free and order-fixed -------------------------------
//   out[w][:] = alpha*E[w][:] - lr * sum_{m in run of w} dA[m][:]
// Sorted windows: RUN_WAVES runs a workgroup, blockIdx.y = block of 256 columns (see walk_runs).
// Ec (may be nullptr): compute copy [.][ldc] of the updated matrix, refreshed with the new row (the tied word
// matrix of the compressed architecture is an operand of the output layer as well).
template <bool ALIGNED, typename T>
__global__ void __launch_bounds__(64 * RUN_WAVES) scatter_runs_kernel(const float *__restrict__ dA, int Hp, int H, int B,
                                                                      int Bp, const int32_t *__restrict__ xp,
                                                                      const int32_t *__restrict__ perm,
                                                                      const int32_t *__restrict__ seg_start,
                                                                      const int32_t *__restrict__ nseg,
                                                                      const float *__restrict__ E,
                                                                      float *__restrict__ out, float alpha, float lr,
                                                                      int compact_ld, T *__restrict__ Ec, int ldc) {
  __shared__ RunShared shared;
  const int lane = threadIdx.x & 63, col = blockIdx.y * RUN_COLS + lane * 4;
  auto row_of = [&](int m) { return (m / B) * Bp + m % B; };
  struct Old {
    int w;
    f32x4_t v;
  };
  walk_runs(
      seg_start, *nseg, shared,
      [&](int r0) {  // the row being updated does not depend on the sum: ask for it first
        Old o;
        o.w = __builtin_amdgcn_readfirstlane(xp[row_of(perm[r0])]);
        o.v = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
        if (alpha != 0.0f) o.v = load_row4<ALIGNED>(E + (long)o.w * H, col, H) * alpha;
        return o;
      },
      [&](int r0, int r1) {
        RunSum s;
        for (int c = r0; c < r1; c += 64) {
          const int n = min(64, r1 - c), row = lane < n ? row_of(perm[c + lane]) : 0;
          s.take(0, n,
                 [&](int i) {
                   return *reinterpret_cast<const f32x4_t *>(dA + (long)__builtin_amdgcn_readlane(row, i) * Hp + col);
                 },
                 [](int, f32x4_t v, f32x4_t &acc) { acc += v; });
        }
        return RowSum{s.total(), 0.0f};
      },
      [&](int run, const Old &o, const RowSum &tot) {
        // compact_ld > 0: the run's result goes to row `run` of a compact [runs][compact_ld] buffer instead of row w
        float *dst = compact_ld > 0 ? out + (long)run * compact_ld : out + (long)o.w * H;
        store_row4<ALIGNED>(o.v - lr * tot.v, col, H, dst, Ec ? Ec + (long)o.w * ldc : nullptr);
      });
}

// Windows of at most SCAN_MAX positions can do without a sorted list.  blockIdx.x = window position m; the workgroup
// compares m's id with all others, gives up if it is not the first of its run, and otherwise has the run's members, in
// ascending order, in LDS.  The keys a thread compares are loaded together, so this costs one memory round trip and
// two barriers, where the sort is two launches on a second stream and the events that tie it in (a window of 32
// positions spent 30 us of host time on them).  The waves are then laid out as column blocks of 256 (`blocks` of them, a
// power of two) times slices of the run's members; the sums are the same tree as a sorted window's.  P = 512, 2560
// positions: 35 -> 21 us.
constexpr int SCAN_MAX = 4096;
template <typename T>
struct ScanUpdate {
  const float *dA;
  int Hp, H, B, Bp;
  const int32_t *xp;
  const float *E;
  float *out;
  float alpha, lr;
  T *Ec;
  int ldc, M, blocks;
};
struct ScanShared {
  f32x4_t sums[2 * RUN_WAVES][64];  // (RUN_WAVES - each) * blocks rows are in use
  unsigned long long found[64];     // group of 64 positions -> which of them
  int before[64], total;
  unsigned short members[SCAN_MAX];
};
// By a workgroup of WAVES waves; g: its position, y: its group of column blocks.
template <int WAVES, bool ALIGNED, typename T>
__device__ inline void scatter_scan(const ScanUpdate<T> &p, ScanShared &sh, int g, int y) {
  constexpr int THREADS = 64 * WAVES, KEYS = SCAN_MAX / THREADS;  // keys per thread: threadIdx.x + THREADS k
  static_assert(KEYS * WAVES == 64 && RUN_WAVES % WAVES == 0, "one lane per group");
  const int H = p.H, M = p.M, blocks = p.blocks;
  auto row_of = [&](int m) { return (m / p.B) * p.Bp + m % p.B; };
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int w = p.xp[row_of(g)];
  int key[KEYS];
#pragma unroll
  for (int k = 0; k < KEYS; ++k) key[k] = threadIdx.x + THREADS * k < M ? p.xp[row_of(threadIdx.x + THREADS * k)] : -1;
  unsigned mine = 0;
#pragma unroll
  for (int k = 0; k < KEYS; ++k) {
    const unsigned long long b = __ballot(key[k] == w);
    if (lane == 0) sh.found[k * WAVES + wave] = b;
    mine |= (unsigned)(key[k] == w) << k;
  }
  __syncthreads();
  if (wave == 0) {  // members before each group of 64 positions
    const int n = __popcll(sh.found[lane]);
    int incl = n;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int up = __shfl_up(incl, o, 64);
      if (lane >= o) incl += up;
    }
    sh.before[lane] = incl - n;
    if (lane == 63) sh.total = incl;
  }
  __syncthreads();
  auto rank = [&](int m) { return sh.before[m >> 6] + __popcll(sh.found[m >> 6] & ((1ull << (m & 63)) - 1)); };
  if (rank(g) != 0) return;  // an earlier position starts this run
  for (; mine; mine &= mine - 1) {
    const int m = threadIdx.x + THREADS * (__ffs(mine) - 1);
    sh.members[rank(m)] = (unsigned short)m;
  }
  __syncthreads();
  const int slices = WAVES / blocks, slice = wave / blocks, cb = wave % blocks;
  const int each = RUN_WAVES / slices;  // slices of the members a wave takes
  const int n = __builtin_amdgcn_readfirstlane(sh.total);
  const int col = (y * blocks + cb) * RUN_COLS + lane * 4;
  f32x4_t old = {0.0f, 0.0f, 0.0f, 0.0f};
  if (slice == 0 && p.alpha != 0.0f) old = load_row4<ALIGNED>(p.E + (long)w * H, col, H) * p.alpha;
  auto sum = [&](int s0, int s1) {
    RunSum s;
    if (col < p.Hp)
      s.take(s0, s1,
             [&](int i) {
               return *reinterpret_cast<const f32x4_t *>(
                   p.dA + (long)row_of(__builtin_amdgcn_readfirstlane(sh.members[i])) * p.Hp + col);
             },
             [](int, f32x4_t v, f32x4_t &acc) { acc += v; });
    return s.total();
  };
  f32x4_t tot;
  if (n <= RUN_ALONE) {
    if (slice != 0) return;
    tot = sum(0, n);
  } else {
    const int per = (n + RUN_WAVES - 1) / RUN_WAVES;
    for (int j = 0; j < each; ++j) {
      const int q = slice * each + j, s0 = min(q * per, n);
      const f32x4_t v = sum(s0, min(s0 + per, n));
      if (slice != 0)
        sh.sums[(q - each) * blocks + cb][lane] = v;
      else
        tot = j == 0 ? v : tot + v;
    }
    __syncthreads();
    if (slice != 0) return;
    for (int q = each; q < RUN_WAVES; ++q) tot += sh.sums[(q - each) * blocks + cb][lane];
  }
  store_row4<ALIGNED>(old - p.lr * tot, col, H, p.out + (long)w * H, p.Ec ? p.Ec + (long)w * p.ldc : nullptr);
}
template <bool ALIGNED, typename T>
__global__ void __launch_bounds__(64 * RUN_WAVES) scatter_scan_kernel(const ScanUpdate<T> p) {
  __shared__ ScanShared sh;
  scatter_scan<RUN_WAVES, ALIGNED>(p, sh, blockIdx.x, blockIdx.y);
}

// 8-bit row-wise quantisation (Sec. 5.4 quantises all the weights; the scheme is a reading): one workgroup
// per row r of W[R][C]: scale = max|row| / 127 (1 for an all-zero row), code = round-half-to-even(w / scale)
// clipped to [-127, 127], all in fp32 with correctly rounded division; the compute copy Wc[r][ldc] receives
// code * scale.  max is order-independent, so the result does not depend on the reduction tree.
template <typename T>
__global__ void __launch_bounds__(256) quantize_rows_kernel(const float *__restrict__ W, int C,
                                                            int8_t *__restrict__ codes, float *__restrict__ scale,
                                                            T *__restrict__ Wc, int ldc) {
  __shared__ float red[256];
  const int r = blockIdx.x;
  const float *row = W + (long)r * C;
  float amax = 0.0f;
  for (int c = threadIdx.x; c < C; c += 256) amax = fmaxf(amax, fabsf(row[c]));
  red[threadIdx.x] = amax;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + s]);
    __syncthreads();
  }
  amax = red[0];
  const float sc = amax > 0.0f ? amax / 127.0f : 1.0f;
  if (threadIdx.x == 0) scale[r] = sc;
  for (int c = threadIdx.x; c < C; c += 256) {
    float q = rintf(row[c] / sc);
    q = fminf(fmaxf(q, -127.0f), 127.0f);
    codes[(long)r * C + c] = (int8_t)q;
    Wc[(long)r * ldc + c] = from_f32<T>(q * sc);
  }
}

// ---- measured peaks of the box (reported next to the published ones) -----------------------------
// Register-resident MFMA loop: 8 independent 32x32x16 bf16 accumulations per iteration and wave, operands
// rotated every iteration.  RANDOM = operand bits drawn from a hash (the sustained rate with realistic
// data: power management lowers the clock when operands toggle); otherwise constant operands.
template <bool RANDOM>
__global__ void __launch_bounds__(512) mfma_rate_kernel(float *out, int iters) {
  auto hashu = [](unsigned x) {
    x ^= x >> 16;
    x *= 0x7feb352dU;
    x ^= x >> 15;
    x *= 0x846ca68bU;
    x ^= x >> 16;
    return x;
  };
  bf16x8_t a[4], b[2];
  for (int q = 0; q < 4; ++q)
    for (int e = 0; e < 8; ++e) {
      const unsigned hsh = hashu(threadIdx.x * 131 + q * 17 + e + blockIdx.x * 7919);
      a[q][e] = RANDOM ? (bf16_t)(((int)(hsh & 0xffff) - 32768) / 65536.0f) : (bf16_t)0.5f;
    }
  for (int q = 0; q < 2; ++q)
    for (int e = 0; e < 8; ++e) {
      const unsigned hsh = hashu(threadIdx.x * 733 + q * 29 + e + 1234567);
      b[q][e] = RANDOM ? (bf16_t)(((int)(hsh & 0xffff) - 32768) / 65536.0f) : (bf16_t)0.25f;
    }
  f32x16_t acc[8];
  for (int i = 0; i < 8; ++i)
    for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[i * 2 + j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i * 2 + j], 0, 0, 0);
    bf16x8_t t = a[0];
    a[0] = a[1];
    a[1] = a[2];
    a[2] = a[3];
    a[3] = t;
    t = b[0];
    b[0] = b[1];
    b[1] = t;
  }
  float sum = 0;
  for (int i = 0; i < 8; ++i)
    for (int r = 0; r < 16; ++r) sum += acc[i][r];
  out[blockIdx.x * blockDim.x + threadIdx.x] = sum;
}

// Plain device copy, 16 bytes per lane, grid-stride.
__global__ void __launch_bounds__(256) copy_kernel(const u32x4_t *__restrict__ src, u32x4_t *__restrict__ dst, long n16) {
  long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long stride = (long)gridDim.x * blockDim.x;
  for (; i < n16; i += stride) dst[i] = src[i];
}

}  // namespace rnnlm_dev
