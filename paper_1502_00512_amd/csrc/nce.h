// Kernels of the noise-contrastive training criterion (Sec. 4.2 of the paper names it; the estimator
// is Gutmann & Hyvarinen's, in the form Mnih & Teh use for language models).
//
// For window position m with hidden state h_m and target y_m, and K noise words n_0..n_{K-1} shared by
// the whole window, with scores z_m(w) = Wo[w].h_m + b[w] and D_m(w) = z_m(w) - lnZ - ln(K q(w)):
//   J_m = softplus(-D_m(y_m)) + sum_j softplus(D_m(n_j)),        softplus(d) = ln(1 + e^d)
//   dJ_m/dz_m(y_m) = -(1 - sigmoid(D_m(y_m))),  dJ_m/dz_m(n_j) = sigmoid(D_m(n_j)),
// window loss = mean of J_m.  The dense parts (all positions x all noise words) run on the contraction
// kernels over a gathered panel of Wo rows; the kernels here do the gathers, the elementwise pass, the
// per-target terms and the order-fixed, atomic-free update of the touched rows of Wo and b.
//
// Index conventions: "row" = t*Bp + s is a padded window position; "m" = t*B + s the compact one; entry
// e of the update list is noise word e for e < K and the target of compact position e - K otherwise.
#pragma once
#include "common.h"
#include "gemm.h"
#include "kernels.h"

namespace rnnlm_dev {

__device__ inline float softplusf_(float d) { return fmaxf(d, 0.0f) + log1pf(__expf(-fabsf(d))); }
__device__ inline float logisticf_(float d) {
  const float e = __expf(-fabsf(d));
  return (d >= 0.0f) ? 1.0f / (1.0f + e) : e / (1.0f + e);
}

// Both at once, as the elementwise pass over all scores wants them: the exponent's rounding error taken along, divisions by
// the hardware reciprocal and a correction by the remainder, ln(1 + e) = 2 artanh(e / (2 + e)) by the series in the
// argument's square (to t^4; coefficients through the Chebyshev nodes of [0, 1/9], 8e-9 relative).  Some 30 instructions
// instead of 80, which bound the pass (2560 positions, 1024 noise words, 160 workgroups: contraction and pass 28 us, without
// the pass 12; window with rmsprop 224 and 214, with the target words' share formed in the next contraction).  Relative error against 64
// bits, root mean square over scores of -30..30, with the exponential and the reciprocal an ulp off at random, before and now:
// logistic 2.3e-7 and 0.6e-7, softplus 2.3e-7 and 0.6e-7.
__device__ inline void noise_terms(float d, float &logistic, float &softplus) {
  const float a = -fabsf(d), x = a * 1.44269502f;
  float lo = fmaf(a, 1.92596303e-8f, fmaf(a, 1.44269502f, -x));  // what the product lost
  lo = a > -128.0f ? lo : 0.0f;                                  // (an infinite score has no remainder)
  float e = __builtin_amdgcn_exp2f(x);
  e = fmaf(e * lo, 0.693147181f, e);
  const float d1 = 1.0f + e, n1 = d >= 0.0f ? 1.0f : e, q1 = __builtin_amdgcn_rcpf(d1), r1 = n1 * q1;
  logistic = fmaf(fmaf(-d1, r1, n1), q1, r1);
  const float d2 = 2.0f + e, q2 = __builtin_amdgcn_rcpf(d2), r2 = e * q2;
  const float s = fmaf(fmaf(-r2, e - (d2 - 2.0f), fmaf(-d2, r2, e)), q2, r2), t = s * s;
  const float p = fmaf(fmaf(fmaf(0.14078889f, t, 0.13982579f), t, 0.20012298f), t, 0.33333161f);
  softplus = fmaxf(d, 0.0f) + fmaf((s + s) * t, p, s + s);
}

// Dot product of two compute-type rows of n values (n a multiple of 16 / sizeof(T)), one wave: 16-byte loads, per-lane
// sums, then a butterfly.  Every lane returns the sum.
template <typename T>
__device__ inline float wave_dot(const T *__restrict__ x, const T *__restrict__ y, int n, int lane) {
  constexpr int VEC = 16 / (int)sizeof(T);
  float acc = 0.0f;
  for (int c = lane * VEC; c < n; c += 64 * VEC) {
    union {
      u32x4_t u;
      T t[VEC];
    } a, b;
    a.u = *reinterpret_cast<const u32x4_t *>(x + c);
    b.u = *reinterpret_cast<const u32x4_t *>(y + c);
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc = fmaf(to_f32(a.t[e]), to_f32(b.t[e]), acc);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  return acc;
}

// Score of the target word of a position, by one wave: dt[row] = Wo_c[y].Hs[row] + b[y] - shift - lnq[y]
// (lnq == nullptr: no noise term).  out (may be nullptr) receives the valid positions in compact order t*B + s.
template <typename T>
__device__ inline void target_score(int row, int lane, const T *__restrict__ Hs1, const T *__restrict__ Wo_c, int Hp,
                                    const int32_t *__restrict__ yp, const float *__restrict__ b,
                                    const float *__restrict__ lnq, float shift, int B, int Bp, float *__restrict__ dt,
                                    float *__restrict__ out) {
  const int y = yp[row];
  if (y < 0) {
    if (lane == 0) dt[row] = 0.0f;
    return;
  }
  const T *hrow = Hs1 + (long)row * Hp, *wrow = Wo_c + (long)y * Hp;
  const float acc = wave_dot(hrow, wrow, Hp, lane);
  if (lane == 0) {
    const float v = acc + b[y] - shift - (lnq ? lnq[y] : 0.0f);
    dt[row] = v;
    if (out) out[(row / Bp) * B + (row % Bp)] = v;
  }
}
// All padded positions, 4 per workgroup.
template <typename T>
__global__ void __launch_bounds__(256) nce_target_score_kernel(const T *__restrict__ Hs1, const T *__restrict__ Wo_c,
                                                               int Hp, const int32_t *__restrict__ yp,
                                                               const float *__restrict__ b,
                                                               const float *__restrict__ lnq, float shift, int rows,
                                                               int B, int Bp, float *__restrict__ dt,
                                                               float *__restrict__ out) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row < rows) target_score(row, threadIdx.x & 63, Hs1, Wo_c, Hp, yp, b, lnq, shift, B, Bp, dt, out);
}

// Preparation of a window's noise words, one workgroup per (padded) noise slot j < Kp plus ceil(M/256)
// workgroups for the targets and rows / 4 for the targets' own scores:
//   noise id checked (flags[0] on an id outside [0,V), clamped); offset off[j] = b[n_j] - lnZ - ln K - lnq[n_j]
//   (0 for the padding j >= K); panel row Wn[j][:] = Wo_c[n_j][:] (zero rows for the padding; Hp is a multiple
//   of 256); update list ids[0..K) = noise words, ids[K + m] = target of compact position m.
template <typename T>
__global__ void __launch_bounds__(256) nce_prep_kernel(const int32_t *__restrict__ noise, int K, int Kp, int V,
                                                       const float *__restrict__ lnq, const float *__restrict__ b,
                                                       float lnZ_lnK, const int32_t *__restrict__ yp, int M, int B,
                                                       int Bp, const T *__restrict__ Wo_c, int Hp,
                                                       T *__restrict__ Wn, float *__restrict__ off,
                                                       int32_t *__restrict__ ids, int32_t *__restrict__ flags,
                                                       const T *__restrict__ Hs1, int rows, float *__restrict__ dt) {
  constexpr int VEC = 16 / (int)sizeof(T);
  const int j = blockIdx.x;
  if (j >= Kp) {  // target part of the update list
    const int part = j - Kp, lists = (M + 255) / 256, m = part * 256 + threadIdx.x;
    if (part >= lists) {
      const int row = (part - lists) * 4 + (threadIdx.x >> 6);
      if (row < rows) target_score(row, threadIdx.x & 63, Hs1, Wo_c, Hp, yp, b, lnq, lnZ_lnK, B, Bp, dt, (float *)nullptr);
    } else if (m < M) {
      ids[K + m] = yp[(m / B) * Bp + (m % B)];
    }
    return;
  }
  int w = 0;
  if (j < K) {
    w = noise[j];
    const bool bad = w < 0 || w >= V;
    w = min(max(w, 0), V - 1);
    if (threadIdx.x == 0) {
      if (bad) flags[0] = 1;
      off[j] = b[w] - lnZ_lnK - lnq[w];
      ids[j] = w;
    }
  } else if (threadIdx.x == 0) {
    off[j] = 0.0f;
  }
  const u32x4_t *src = reinterpret_cast<const u32x4_t *>(Wo_c + (long)w * Hp);
  u32x4_t *dst = reinterpret_cast<u32x4_t *>(Wn + (long)j * Hp);
  const u32x4_t zero = {0u, 0u, 0u, 0u};
  for (int c = threadIdx.x; c < Hp / VEC; c += 256) dst[c] = (j < K) ? src[c] : zero;
}

// Scores of a shortlist of C candidate words per position (Sec. 5.4 ranks a shortlist of candidates):
// out[(t*B + s)*C + c] = Wc[cand].F[row] + b[cand] - shift, F = what the output layer reads (ld = width
// Dp).  One wave per (position, candidate); ids outside [0, V) are clamped and raise flags[0].
template <typename T>
__global__ void __launch_bounds__(256) score_candidates_kernel(const T *__restrict__ F, const T *__restrict__ Wc, int Dp,
                                                               const int32_t *__restrict__ cand, int C, int V,
                                                               const float *__restrict__ b, float shift, long total,
                                                               int B, int Bp, int32_t *__restrict__ flags,
                                                               float *__restrict__ out) {
  const long item = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (item >= total) return;
  const long pos = item / C;  // compact position index t*B + s
  const long row = (pos / B) * Bp + (pos % B);
  int w = cand[item];
  if (w < 0 || w >= V) {
    if (lane == 0) flags[0] = 1;
    w = min(max(w, 0), V - 1);
  }
  const T *frow = F + row * Dp, *wrow = Wc + (long)w * Dp;
  const float acc = wave_dot(frow, wrow, Dp, lane);
  if (lane == 0) out[item] = acc + b[w] - shift;
}

// The value of lane ^ MASK (inside a half-wave), without an address register.
template <int MASK>
__device__ inline int swap_lanes(int v) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (MASK == 1) return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true);   // quad_perm 1, 0, 3, 2
  if constexpr (MASK == 2) return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true);   // quad_perm 2, 3, 0, 1
  if constexpr (MASK == 8) return __builtin_amdgcn_mov_dpp(v, 0x128, 0xF, 0xF, true);  // a row of 16 rotated by 8
  return __builtin_amdgcn_ds_swizzle(v, (MASK << 10) | 0x1F);
#else
  return v;
#endif
}

// Epilogue of the score contraction S = Hs . Wn^T (rows: padded positions, columns: noise slots), elementwise while the
// scores are in registers: dS[row][j] = sigmoid(S + off[j]) * scale in the contraction operand type (0 for padding rows and
// columns), and, per 32x32 block, the sums of softplus(S + off[j]) over its columns (jpart[column block][row]) and of dS
// before rounding over its rows (gpart[row block][j]).  V = 64000, H = 1024, 2560 positions, 1024 noise words: the
// contraction, a pass over its fp32 scores and one more for the column sums took 17 + 15 + 7 us.  Whole windows with those
// passes and with this, every tile form (bf16 us): V = 64000, H = 1024, 16x4, 64 words 124 and 116; 128x20, 256 words 170 and
// 162, 1024 words 193 and 182; 256x32, 2048 words 527 and 459; V = 10000, H = 300, 256x32, 2000 words 362 and 327; V = 20000,
// H = 2048, 32x20, 500 words 228 and 231; fp32: 394 and 400 at 128x20, 1024 words, 1312 and 1277 at 256x32, 2048 words.
template <typename T>
struct EpiNce : EpiZeroInit {
  T *dS;
  long ld;  // Kp
  const float *off;
  const int *yp;  // [Mp] target id per position, -1 on padding
  float scale;
  int K, Mp;
  float *jpart;  // [Kp / 32][Mp]
  float *gpart;  // [Mp / 32][Kp]
  template <int BM, int BN>
  static constexpr int lds_bytes() { return 0; }
  template <int BM, int BN, int TM, int TN, int NT>
  __device__ inline void run(f32x16_t (&acc)[TM][TN], const EpiCtx &c) const {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int row0 = c.tile_row0 + c.wrow + i * 32;
      unsigned valid = 0;
#pragma unroll
      for (int r = 0; r < 16; ++r) valid |= (unsigned)(yp[row0 + RNNLM_ACC_ROW(r, c.lane)] >= 0) << r;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int col0 = c.tile_col0 + c.wcol + j * 32, col = col0 + (c.lane & 31);
        const float o = off[col];
        const unsigned live = col < K ? valid : 0u;
        float cost[16], grad[16], gsum = 0.0f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const bool on = (live >> r) & 1u;
          float g, s;
          noise_terms(acc[i][j][r] + o, g, s);
          grad[r] = on ? g * scale : 0.0f;
          cost[r] = on ? s : 0.0f;
          gsum += grad[r];
        }
        if constexpr (sizeof(T) == 2) {  // neighbouring lanes swap one value: each owns two adjacent columns of one row
          typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
          const bool odd = c.lane & 1;
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            bf16x2_t h;
            h[0] = (bf16_t)grad[2 * q];
            h[1] = (bf16_t)grad[2 * q + 1];
            const unsigned mine = __builtin_bit_cast(unsigned, h);
            const unsigned theirs = (unsigned)swap_lanes<1>((int)mine);
            const long row = row0 + RNNLM_ACC_ROW(2 * q, c.lane) + (odd ? 1 : 0);
            *reinterpret_cast<unsigned *>(dS + row * ld + (col & ~1)) = join_pair(mine, theirs, odd);
          }
        } else {
#pragma unroll
          for (int r = 0; r < 16; ++r) dS[(long)(row0 + RNNLM_ACC_ROW(r, c.lane)) * ld + col] = from_f32<T>(grad[r]);
        }
        gsum += __shfl_xor(gsum, 32, 64);
        if (c.lane < 32) gpart[(long)(row0 >> 5) * ld + col] = gsum;
        // sums over the 32 lanes of a row: at each exchange a lane keeps half of its rows and gives the other half away
        auto halve = [&](auto n_) {
          constexpr int n = decltype(n_)::value;
          const bool upper = c.lane & (2 * n);
#pragma unroll
          for (int k = 0; k < n; ++k) {
            const float give = upper ? cost[k] : cost[k + n];
            cost[k] = (upper ? cost[k + n] : cost[k]) + __int_as_float(swap_lanes<2 * n>(__float_as_int(give)));
          }
        };
        halve(std::integral_constant<int, 8>());
        halve(std::integral_constant<int, 4>());
        halve(std::integral_constant<int, 2>());
        halve(std::integral_constant<int, 1>());
        cost[0] += __int_as_float(swap_lanes<1>(__float_as_int(cost[0])));
        const int r = (c.lane & 31) >> 1;  // the row this lane has kept
        if (!(c.lane & 1)) jpart[(long)(col0 >> 5) * Mp + row0 + RNNLM_ACC_ROW(r, c.lane)] = cost[0];
      }
    }
  }
};

// Adds up the blocks' partial sums, in fixed order.  The first rowBlocks workgroups, 64 positions each: the position's
// loss J and the target coefficient ct[row] = -(1 - sigmoid(dt)) * scale (0 on padding rows); the others, 64 noise slots
// each: their bias gradient gcol[j].  16 groups of threads share out the partials (bound by memory latency).
// done != nullptr: the last workgroup to finish forms the window's sum as well, as in merge_stats_kernel.
__global__ void __launch_bounds__(1024) nce_merge_kernel(const float *__restrict__ jpart, const float *__restrict__ gpart,
                                                         int Kp, int Mp, int rowBlocks, const float *__restrict__ dt,
                                                         const int32_t *__restrict__ yp, int rows, int B, int Bp,
                                                         float scale, float *__restrict__ ct,
                                                         float *__restrict__ J_int, float *__restrict__ J_out,
                                                         float *__restrict__ gcol, unsigned *__restrict__ done,
                                                         const WindowSum w, int M) {
  __shared__ float sh[16][64];
  __shared__ int last;
  const int c = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const bool positions = (int)blockIdx.x < rowBlocks;
  const int i = (positions ? blockIdx.x : blockIdx.x - rowBlocks) * 64 + c;
  const float *part = positions ? jpart : gpart;
  const int n = (positions ? Kp : Mp) / 32, ld = positions ? Mp : Kp;
  float acc = 0.0f;
  if (i < ld) {
#pragma unroll 8
    for (int p = grp; p < n; p += 16) acc += part[(long)p * ld + i];
  }
  sh[grp][c] = acc;
  __syncthreads();
  if (grp == 0) {
#pragma unroll
    for (int g = 1; g < 16; ++g) acc += sh[g][c];
    if (!positions) {
      gcol[i] = acc;
    } else if (i < rows && yp[i] < 0) {
      ct[i] = 0.0f;
    } else if (i < rows) {
      const float d = dt[i];
      const float total = acc + softplusf_(-d);
      ct[i] = -logisticf_(-d) * scale;
      const int m = (i / Bp) * B + i % Bp;
      __hip_atomic_store(J_int + m, total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (J_out) J_out[m] = total;
    }
  }
  if (!done) return;
  if (threadIdx.x < 64) {  // the wave that stored: its stores are acknowledged before the arrival
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (threadIdx.x == 0)
      last = __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == gridDim.x;
  }
  __syncthreads();
  if (!last) return;
  window_sum(w, M, [&](int m) { return __hip_atomic_load(J_int + m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); });
}

// Epilogue of dHs = dS . Wn + ct * Wo[target]: the accumulators start at the target word's share of what the output layer
// sends back, gathered while the first blocks of the contraction are on their way.  (As a pass over dHs of its own, 7 us and a launch at
// 2560 positions; gathered in the epilogue, a dependent load per row, 4 us more than the pass.)
template <typename T>
struct EpiNceDhs : EpiPartial {
  const T *Wo_c;
  const int *yp;  // [Mp] target id per position, -1 on padding
  const float *ct;
  template <int TM, int TN>
  __device__ inline void init(f32x16_t (&acc)[TM][TN], int row0, int col0, int lane, int) const {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = row0 + i * 32 + RNNLM_ACC_ROW(r, lane), y = yp[row];
        const float c = y >= 0 ? ct[row] : 0.0f;
        const T *const w = Wo_c + (long)max(y, 0) * ld + col0 + (lane & 31);
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j][r] = c * to_f32(w[j * 32]);
      }
  }
};

// Update of the touched rows of Wo, atomic-free and order-fixed:
//   out[w][:] = alpha*Wo[w][:] - lr * ( sum_{noise entries e of w} G[e][:] + sum_{target entries} ct*Hs[row][:] )
// Runs of equal ids of the sorted update list, RUN_WAVES a workgroup; blockIdx.y = block of 256 columns (walk_runs).  A
// run's noise entries come before its target entries.  Also refreshes the compute copy of the row when Wc != nullptr.
// compact_ld > 0 redirects the results to compact per-run buffers (see below).
// The first column block also updates the word's bias, one member a lane:
//   b_out[w] = alpha*b[w] - lr * (sum over w's noise entries of their column sums + sum of ct over its target
//   entries), the column sums from gcol.
template <bool ALIGNED, typename T>
__global__ void __launch_bounds__(64 * RUN_WAVES) nce_row_update_kernel(
    const float *__restrict__ G, const T *__restrict__ Hs1, int Hp, int H, int K, int B, int Bp,
    const float *__restrict__ ct, const int32_t *__restrict__ ids, const int32_t *__restrict__ perm,
    const int32_t *__restrict__ seg_start, const int32_t *__restrict__ nseg, const float *__restrict__ W,
    float *__restrict__ out, T *__restrict__ Wc, const float *__restrict__ gcol, const float *__restrict__ b,
    float *__restrict__ b_out, float alpha, float lr, int compact_ld) {
  __shared__ RunShared shared;
  const int lane = threadIdx.x & 63;
  const int col = blockIdx.y * RUN_COLS + lane * 4;
  const bool bias = blockIdx.y == 0;
  struct Old {
    int w;
    f32x4_t v;
    float b;
  };
  walk_runs(
      seg_start, *nseg, shared,
      [&](int r0) {  // what is being updated does not depend on the sum: ask for it first
        Old o;
        o.w = __builtin_amdgcn_readfirstlane(ids[perm[r0]]);
        o.v = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
        o.b = 0.0f;
        if (alpha != 0.0f) {
          o.v = load_row4<ALIGNED>(W + (long)o.w * H, col, H) * alpha;
          if (bias) o.b = alpha * b[o.w];
        }
        return o;
      },
      [&](int r0, int r1) {
        RunSum s;
        float bacc = 0.0f;
        for (int c = r0; c < r1; c += 64) {
          const int n = min(64, r1 - c);
          int row = 0;
          float coef = 0.0f;
          bool noise = false;
          if (lane < n) {
            row = perm[c + lane];
            noise = row < K;
            if (!noise) {
              const int m = row - K;
              row = (m / B) * Bp + m % B;
              coef = ct[row];
            }
            if (bias) bacc += noise ? gcol[row] : coef;
          }
          const int nn = __popcll(__ballot(noise));
          s.take(0, nn,
                 [&](int i) {
                   return *reinterpret_cast<const f32x4_t *>(G + (long)__builtin_amdgcn_readlane(row, i) * Hp + col);
                 },
                 [](int, f32x4_t v, f32x4_t &acc) { acc += v; });
          typedef T t4 __attribute__((ext_vector_type(4)));
          s.take(nn, n,
                 [&](int i) {
                   return *reinterpret_cast<const t4 *>(Hs1 + (long)__builtin_amdgcn_readlane(row, i) * Hp + col);
                 },
                 [&](int i, t4 v, f32x4_t &acc) {
                   const float k = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(coef), i));
#pragma unroll
                   for (int e = 0; e < 4; ++e) acc[e] = fmaf(k, to_f32((T)v[e]), acc[e]);
                 });
        }
        if (bias) {
#pragma unroll
          for (int o = 32; o > 0; o >>= 1) bacc += __shfl_xor(bacc, o, 64);
        }
        return RowSum{s.total(), bacc};
      },
      [&](int run, const Old &o, const RowSum &tot) {
        // compact_ld > 0: the run's result goes to row `run` of a compact [runs][compact_ld] buffer (and its bias term to
        // entry `run` of b_out) instead of the word's own row
        float *dst = compact_ld > 0 ? out + (long)run * compact_ld : out + (long)o.w * H;
        if (bias && lane == 0) b_out[compact_ld > 0 ? run : o.w] = o.b - lr * tot.b;
        store_row4<ALIGNED>(o.v - lr * tot.v, col, H, dst, Wc ? Wc + (long)o.w * Hp : nullptr);
      });
}

}  // namespace rnnlm_dev