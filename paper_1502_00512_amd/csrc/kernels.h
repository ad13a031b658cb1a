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

// Sum of n log-probabilities in fp64 with a fixed reduction tree, by a workgroup of 1024 threads; raises flags[1] when
// the result is not finite.  counters != nullptr: also clears the counters of the persistent recurrent kernel (the sum
// sits between its forward and its backward launch).
struct WindowSum {
  double *out, *running;  // either may be nullptr: the sum, and what it is added to
  int32_t *flags;
  unsigned *counters;
};
template <class Load>
__device__ inline void window_sum(const WindowSum &w, int n, Load &&load) {
  __shared__ double sh[1024];
  if (w.counters)
    for (int i = threadIdx.x; i < SYNC_WORDS; i += 1024) w.counters[i] = 0u;
  double a = 0.0;
  for (int i = threadIdx.x; i < n; i += 1024) a += (double)load(i);
  sh[threadIdx.x] = a;
  __syncthreads();
  for (int k = 512; k > 0; k >>= 1) {
    if ((int)threadIdx.x < k) sh[threadIdx.x] += sh[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double s = sh[0];
    if (w.out) *w.out = s;
    if (w.running) *w.running += s;
    if (!(s == s) || s - s != 0.0) w.flags[1] = 1;
  }
}
__global__ void __launch_bounds__(1024) sum_logp_kernel(const float *__restrict__ logp, int n, const WindowSum w) {
  window_sum(w, n, [&](int i) { return logp[i]; });
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
template <typename T>
__global__ void __launch_bounds__(256) softmax_grad_kernel(T *__restrict__ ZT, long ldz, int Mp, int V, int Vp,
                                                           const float *__restrict__ lse,
                                                           const int32_t *__restrict__ yp, float invM,
                                                           const float *__restrict__ b, float *__restrict__ b_out,
                                                           float alpha, float lr) {
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
      const f32x4_t lv = *reinterpret_cast<const f32x4_t *>(lse + c + e);
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
__global__ void splitk_reduce_kernel(const float *__restrict__ part, long n, long split_stride, int splits,
                                     float *__restrict__ out) {
  const long i = ((long)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (i >= n) return;
  float4 a = *reinterpret_cast<const float4 *>(part + i);
  for (int s = 1; s < splits; ++s) {
    const float4 q = *reinterpret_cast<const float4 *>(part + (long)s * split_stride + i);
    a.x += q.x;
    a.y += q.y;
    a.z += q.z;
    a.w += q.w;
  }
  *reinterpret_cast<float4 *>(out + i) = a;
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

// ---- a10: segmented embedding update, atomic-free and order-fixed -------------------------------
//   out[w][:] = alpha*E[w][:] - lr * sum_{m in run of w} dA[m][:]
// blockIdx.x = run index (exits when >= *nseg), blockIdx.y = block of 1024 columns.  The run's members are dealt
// round-robin to PARTS partial sums (member i of the run goes
// to sum i mod PARTS, each sum accumulated in ascending m), which are then added in order 0..PARTS-1: a fixed
// summation tree, so results are bitwise reproducible.  All PARTS sums live in the thread's registers: a group
// of 16 members is 16 independent row loads in flight, and the small workgroups (with a sorted list no LDS and no
// barrier) leave eight of them resident per compute unit, which is what a pass made of dependent memory round trips
// (run bounds -> position -> rows) needs: it is bound by latency times occupancy, not by bandwidth.
// A thread owns 4 consecutive columns (the rows of dA are tile-padded and aligned).  ALIGNED: H % 4 == 0, the rows of the
// updated matrix are accessed 16 bytes at a time; otherwise (any H) element by element, the last group partly.
// Ec (may be nullptr): compute copy [.][ldc] of the updated matrix, refreshed with the new row (the tied word
// matrix of the compressed architecture is an operand of the output layer as well).
// SCAN (windows of at most SCAN_MAX positions): no sorted list at all.  blockIdx.x = window position m; the workgroup
// compares m's id with all others, gives up if it is not the first of its run, and otherwise has the run's members, in
// ascending order, in LDS.  The 16 keys a thread compares are loaded together, so this costs one memory round trip and
// two barriers, where the sort is two launches on a second stream and the events that tie it in (a window of 32
// positions spent 30 us of host time on them).
constexpr int SCAN_MAX = 4096;
template <bool ALIGNED, bool SCAN, typename T>
__global__ void __launch_bounds__(256) scatter_update_kernel(const float *__restrict__ dA, int Hp, int H, int B,
                                                             int Bp, const int32_t *__restrict__ xp,
                                                             const int32_t *__restrict__ perm,
                                                             const int32_t *__restrict__ seg_start,
                                                             const int32_t *__restrict__ nseg,
                                                             const float *__restrict__ E, float *__restrict__ out,
                                                             float alpha, float lr, int compact_ld,
                                                             T *__restrict__ Ec, int ldc, int M) {
  constexpr int PARTS = 4, GROUP = 4 * PARTS, VEC = 4;
  const int g = blockIdx.x;
  const int col = (blockIdx.y * 256 + threadIdx.x) * VEC;
  __shared__ unsigned short members[SCAN ? SCAN_MAX : 1];
  int r0, r1, w;
  if constexpr (SCAN) {
    constexpr int KEYS = SCAN_MAX / 256;  // keys per thread: positions threadIdx.x + 256 k
    __shared__ unsigned long long found[KEYS][4];
    __shared__ int before[KEYS * 4], total;
    auto key_of = [&](int m) { return xp[(m / B) * Bp + (m % B)]; };
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    w = key_of(g);
    int key[KEYS];
#pragma unroll
    for (int k = 0; k < KEYS; ++k) key[k] = threadIdx.x + 256 * k < M ? key_of(threadIdx.x + 256 * k) : -1;
    unsigned mine = 0;
#pragma unroll
    for (int k = 0; k < KEYS; ++k) {
      const unsigned long long b = __ballot(key[k] == w);
      if (lane == 0) found[k][wave] = b;
      mine |= (unsigned)(key[k] == w) << k;
    }
    __syncthreads();
    if (wave == 0) {  // members before each group of 64 positions
      const int n = __popcll(found[lane >> 2][lane & 3]);
      int incl = n;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int up = __shfl_up(incl, o, 64);
        if (lane >= o) incl += up;
      }
      before[lane] = incl - n;
      if (lane == 63) total = incl;
    }
    __syncthreads();
    auto rank = [&](int m) {  // members before position m
      return before[m >> 6] + __popcll(found[m >> 8][(m >> 6) & 3] & ((1ull << (m & 63)) - 1));
    };
    if (rank(g) != 0) return;  // an earlier position starts this run
    for (; mine; mine &= mine - 1) {
      const int m = threadIdx.x + 256 * (__ffs(mine) - 1);
      members[rank(m)] = (unsigned short)m;
    }
    __syncthreads();
    r0 = 0;
    r1 = total;
  } else {
    if (g >= *nseg) return;
    r0 = seg_start[g];
    r1 = seg_start[g + 1];
    const int m0 = perm[r0];
    w = xp[(m0 / B) * Bp + (m0 % B)];
  }
  if (col >= H) return;
  const long idx = (long)w * H + col;
  // the row being updated does not depend on the sum: ask for it first
  float old[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) old[e] = 0.0f;
  if (alpha != 0.0f) {
    if (ALIGNED) {
      const f32x4_t t = *reinterpret_cast<const f32x4_t *>(E + idx);
#pragma unroll
      for (int e = 0; e < VEC; ++e) old[e] = t[e];
    } else {
#pragma unroll
      for (int e = 0; e < VEC; ++e)
        if (col + e < H) old[e] = E[idx + e];
    }
  }
  auto row_of = [&](int r) {
    const int m = SCAN ? members[r] : perm[r];
    return ((long)(m / B) * Bp + (m % B)) * Hp + col;
  };
  auto load_row = [&](long at, float (&v)[VEC]) {
    const f32x4_t t = *reinterpret_cast<const f32x4_t *>(dA + at);
#pragma unroll
    for (int e = 0; e < VEC; ++e) v[e] = t[e];
  };
  float acc[PARTS][VEC];
#pragma unroll
  for (int p = 0; p < PARTS; ++p)
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[p][e] = 0.0f;
  int r = r0;
  for (; r + GROUP <= r1; r += GROUP) {
    long at[GROUP];
#pragma unroll
    for (int k = 0; k < GROUP; ++k) at[k] = row_of(r + k);
    float v[GROUP][VEC];
#pragma unroll
    for (int k = 0; k < GROUP; ++k) load_row(at[k], v[k]);
#pragma unroll
    for (int k = 0; k < GROUP; ++k)  // member r + k belongs to sum k % PARTS (r - r0 is a multiple of GROUP)
#pragma unroll
      for (int e = 0; e < VEC; ++e) acc[k % PARTS][e] += v[k][e];
  }
  for (; r < r1; r += PARTS) {
    float v[PARTS][VEC];
#pragma unroll
    for (int p = 0; p < PARTS; ++p) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) v[p][e] = 0.0f;
      if (r + p < r1) load_row(row_of(r + p), v[p]);
    }
#pragma unroll
    for (int p = 0; p < PARTS; ++p)
      if (r + p < r1) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[p][e] += v[p][e];
      }
  }
#pragma unroll
  for (int p = 1; p < PARTS; ++p)
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[0][e] += acc[p][e];
  // compact_ld > 0: the run's result goes to row g of a compact [runs][compact_ld] buffer instead of row w
  const long oidx = compact_ld > 0 ? (long)g * compact_ld + col : idx;
  float nv[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) nv[e] = ((alpha != 0.0f) ? alpha * old[e] : 0.0f) - lr * acc[0][e];
  if (ALIGNED) {
    f32x4_t t;
#pragma unroll
    for (int e = 0; e < VEC; ++e) t[e] = nv[e];
    *reinterpret_cast<f32x4_t *>(out + oidx) = t;
  } else {
#pragma unroll
    for (int e = 0; e < VEC; ++e)
      if (col + e < H) out[oidx + e] = nv[e];
  }
  if (Ec) {
#pragma unroll
    for (int e = 0; e < VEC; ++e)
      if (ALIGNED || col + e < H) Ec[(long)w * ldc + col + e] = from_f32<T>(nv[e]);
  }
}

// fp32 -> compute type, element by element (n elements).
template <typename T>
__global__ void to_compute_kernel(const float *__restrict__ src, long n, T *__restrict__ dst) {
  long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long stride = (long)gridDim.x * blockDim.x;
  for (; i < n; i += stride) dst[i] = from_f32<T>(src[i]);
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
