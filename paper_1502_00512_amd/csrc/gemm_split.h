// fp32 contraction on the bf16 matrix cores: every operand value is taken apart into three bf16 values, and six of their
// nine products are formed.
//
// x = h + m + l with h = bf16(x), m = bf16(x - h), l = bf16(x - h - m), rounded to nearest: both differences are exact and so
// is l, and |m| <= 2^-8 |h|, |l| <= 2^-17 |h|.  x y = hh' + hm' + mh' + hl' + lh' + mm' + (terms below 2^-24 |x y|); the six
// products accumulate in fp32, smallest first.  The bf16 rate is sixteen times the fp32 one, so six products take 3/8 of its
// time.  An operand keeps its 24 bits, a product some 2^-24 of itself, and an instruction rounds the sum once per 16 terms
// instead of once or twice per 2.  Distance from 64 bits against the fp32 matrix cores, shape by shape (thirty windows of V =
// 1000..64000, H = 64..3659, 6..32768 positions): gradients of U and of the rows of E 0.12 to 0.75, of Wo 0.01 to 0.63; log-
// probabilities, whose own rounding is most of it, 0.2 to 1.13, below 0.96 in the mean.  Subnormal operands keep fewer bits:
// rows of logit gradients of 8e-39 come out to 1e-4, of 4e-40 to 2e-2, where the fp32 cores give 4e-6 and 1e-6.
//
// What bounds it: power, at the large tiles (matrix cores busy 78 % of the cycles, at 1.4 GHz after some milliseconds of it; a
// conversion that costs one instruction instead of eleven: 3 % faster; another order of the products, no bank conflicts: no
// change).  64,000 x 1280 outputs, depth 1024 / 1280 x 1024 outputs, depth 64,000 / 64,000 x 1024, depth 1280 with its update,
// us in a training window: 1231 / 1285 / 1330 on the fp32 cores, now 766 / 790 / 841 (219, 212, 200 TFLOP/s).  The forward
// output layer's epilogue (EpiOutFwd) does not fit the registers next to the accumulators: 27 of them spill at 256 x 256 (112
// bytes of scratch a lane), 4 at 128 x 128, all outside the loop over the blocks.  Small outputs
// are bound by a workgroup's chain per block (barrier, fragments, products, conversion), which WGK shortens: 256 tiles of
// 64 x 64, depth 1280: 33 us on the fp32 cores, 37 on four waves, 24 on sixteen.
//
// Operands stay fp32 in memory: a workgroup converts a block once while it moves it to LDS, between the products of the block
// before, and its waves then read ordinary bf16 fragments.  (Taken apart at the fragments instead, every wave would convert
// for itself, eight times as many instructions at 256 x 256.)
#pragma once
#include "gemm.h"

namespace rnnlm_dev {

// From here on a value rounds to a bf16 infinity.
constexpr unsigned SPLIT_MAX = 0x7f7f8000u;

#if defined(__HIP_DEVICE_COMPILE__)
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));

__device__ inline unsigned pack_bf16(float a, float b) {
  bf16x2_t h;
  h[0] = (bf16_t)a;
  h[1] = (bf16_t)b;
  return __builtin_bit_cast(unsigned, h);
}
__device__ inline void split_pair(float a, float b, unsigned &h, unsigned &m, unsigned &l) {
  h = pack_bf16(a, b);
  const float ra = a - __builtin_bit_cast(float, h << 16), rb = b - __builtin_bit_cast(float, h & 0xffff0000u);
  m = pack_bf16(ra, rb);
  l = pack_bf16(ra - __builtin_bit_cast(float, m << 16), rb - __builtin_bit_cast(float, m & 0xffff0000u));
}

// LDS tile of one operand: [KS steps of 16][3 planes][ROWS / 32][half of the step][32 rows] x 8 values of k (16 bytes):
// a fragment (32 rows x 16 k) is one contiguous kilobyte.  The rows of a half are permuted so that the 8-byte writes of
// 16 neighbouring lanes of the loader fill 128 bytes, too.
__device__ inline int split_pos(int r, int h) { return r ^ ((r >> 3) & 1) ^ (h << 2); }

// Moves one ROWS x 16 KS tile global -> registers -> three bf16 planes in LDS.  A thread's values are groups of 4
// consecutive k of one row: K-contiguous operands are read 4 k at a time, K-major ones RW rows at a time for 4 values of
// k, so the transposition costs nothing but the choice of registers.
template <int ROWS, int LAYOUT, int NT, int KS>
struct SplitLoader {
  static constexpr int BK = 16 * KS, KQ = BK / 4;
  static constexpr int E = ROWS * BK / NT;  // values per thread
  static constexpr int G = E / 4;           // groups of 4 k
  static constexpr int RW = LAYOUT == KROW ? G : 1;
  static_assert(E % 4 == 0 && (RW == 1 || RW == 2 || RW == 4), "tile does not divide over the workgroup");
  static constexpr int PLANE = ROWS * 32, BYTES = KS * 3 * PLANE;
  struct Raw {
    float v[G][4];  // [group][k]
  };
  int off[LAYOUT == ROWK ? G : 4];  // byte offsets of the loads inside a block
  int lds[G];
  const char *base;
  long step;

  __device__ inline void init(const char *op, long ld_bytes, long row0, long k0, int tid) {
    if constexpr (LAYOUT == ROWK) {
#pragma unroll
      for (int i = 0; i < G; ++i) {
        const int c = tid + i * NT, r = c / KQ, q = c % KQ;
        off[i] = (int)(r * ld_bytes + q * 16);
        lds[i] = at(r, q);
      }
      base = op + row0 * ld_bytes + k0 * 4;
      step = BK * 4;
    } else {
      // lane bits 0..2: row group, 3: quad of k; then the rest of the row groups (whole lines per k), then of the quads
      constexpr int LPW = RW == 1 ? 32 : 16, QPW = 64 / LPW;  // row groups and quads of k in a wave
      const int lane = tid & 63, wave = tid >> 6;
      constexpr int WQ = KQ / QPW;  // waves along k
      const int lg = RW == 1 ? (lane & 7) | (lane >> 4) << 3 : (lane & 7) | (lane >> 4 & 1) << 3;
      const int lq = RW == 1 ? lane >> 3 & 1 : (lane >> 3 & 1) | (lane >> 5) << 1;
      const int q = (wave % WQ) * QPW + lq, r = ((wave / WQ) * LPW + lg) * RW;
#pragma unroll
      for (int e = 0; e < 4; ++e) off[e] = (int)((q * 4 + e) * ld_bytes + r * 4);
#pragma unroll
      for (int i = 0; i < G; ++i) lds[i] = at(r + i, q);
      base = op + k0 * ld_bytes + row0 * 4;
      step = BK * ld_bytes;
    }
  }
  // byte offset of quad q of row r in the first plane
  __device__ static inline int at(int r, int q) {
    const int ks = q >> 2, h = (q >> 1) & 1;
    return ks * 3 * PLANE + (r >> 5) * 1024 + h * 512 + split_pos(r & 31, h) * 16 + (q & 1) * 8;
  }
  // (re-based at every block: the operand may exceed 32-bit offsets)
  __device__ inline void load(Raw &raw, int kb) const {
    const unsigned long long b = reinterpret_cast<unsigned long long>(base + kb * step);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)b), hi = __builtin_amdgcn_readfirstlane((unsigned)(b >> 32));
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<void *>(((unsigned long long)hi << 32) | lo), 0, 0x7fffffff, 0x00020000);
    if constexpr (LAYOUT == ROWK) {
#pragma unroll
      for (int i = 0; i < G; ++i) {
        const f32x4_t t = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, off[i], 0, 0));
#pragma unroll
        for (int e = 0; e < 4; ++e) raw.v[i][e] = t[e];
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if constexpr (RW == 4) {
          const f32x4_t t = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, off[e], 0, 0));
#pragma unroll
          for (int i = 0; i < 4; ++i) raw.v[i][e] = t[i];
        } else if constexpr (RW == 2) {
          typedef float f32x2_t __attribute__((ext_vector_type(2)));
          const f32x2_t t = __builtin_bit_cast(f32x2_t, __builtin_amdgcn_raw_buffer_load_b64(rs, off[e], 0, 0));
#pragma unroll
          for (int i = 0; i < 2; ++i) raw.v[i][e] = t[i];
        } else {
          raw.v[0][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, off[e], 0, 0));
        }
      }
    }
  }
  __device__ inline void store(char *tile, const Raw &raw, float &big) const {
#pragma unroll
    for (int i = 0; i < G; ++i) {
      const float(&v)[4] = raw.v[i];
      u32x2_t p[3];
      unsigned h, m, l;
      split_pair(v[0], v[1], h, m, l);
      p[0][0] = h, p[1][0] = m, p[2][0] = l;
      split_pair(v[2], v[3], h, m, l);
      p[0][1] = h, p[1][1] = m, p[2][1] = l;
      asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(big) : "v"(v[0]), "v"(v[1]));
      asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(big) : "v"(v[2]), "v"(v[3]));
#pragma unroll
      for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x2_t *>(tile + lds[i] + q * PLANE) = p[q];
    }
  }
};
#endif

template <int BM, int BN, int KS, class Epi>
constexpr int split_lds_bytes() {
  constexpr int loop = 2 * KS * 96 * (BM + BN), epi = Epi::template lds_bytes<BM, BN>();
  return (loop > epi ? loop : epi);
}

// KS = steps of 16 values of k per block; WGK = groups of WGM x WGN waves that share out the steps of a block (their sums
// are added at the end, in order); PF = blocks in registers ahead of the two in LDS.
#if defined(__HIP_DEVICE_COMPILE__)
template <int BM, int BN, int WGM, int WGN, int WGK, int LA, int LB, int KS, int PF, class Epi>
__device__ inline void gemm_split_item(const GemmShape &g, const Epi &epi, int item, char *const smem) {
  constexpr int NT = WGM * WGN * WGK * 64;
  constexpr int BK = 16 * KS, KSW = KS / WGK;
  static_assert(KS % WGK == 0 && (32 % BK == 0 || BK % 32 == 0), "");
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  using LoadA = SplitLoader<BM, LA, NT, KS>;
  using LoadB = SplitLoader<BN, LB, NT, KS>;
  constexpr int STAGE = LoadA::BYTES + LoadB::BYTES;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % WGM, wn = wave / WGM % WGN, wk = wave / (WGM * WGN);
  int tile_m, tile_n, split;
  if (!map_workgroup(g, item, split, tile_m, tile_n)) return;  // uniform for the workgroup
  const int kb0 = split * g.kBlocksPerSplit, nk = min((split + 1) * g.kBlocksPerSplit, g.kBlocks) - kb0;

  f32x16_t acc[TM][TN];
  epi.template init<TM, TN>(acc, tile_m * BM + wm * WTM, tile_n * BN + wn * WTN, lane, split);
  if (WGK > 1 && wk > 0) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
  }

  // where registers allow, the five lesser products have accumulators of their own: the main one is then rounded once per
  // 16 values of k and not six times, and consecutive instructions of a wave do not wait for one another
  constexpr bool SMALL = TM * TN <= 4;
  f32x16_t corr[SMALL ? TM : 1][SMALL ? TN : 1];
#pragma unroll
  for (int i = 0; i < (SMALL ? TM : 1); ++i)
#pragma unroll
    for (int j = 0; j < (SMALL ? TN : 1); ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) corr[i][j][r] = 0.0f;

  LoadA la;
  LoadB lb;
  typename LoadA::Raw ra[PF];
  typename LoadB::Raw rb[PF];
  float big = 0.0f;
  bf16x8_t fa[2][3], fb[2][TN][3];
  // this lane's 16 bytes of a fragment of this wave's first step
  const int pre = (lane >> 5) * 512 + split_pos(lane & 31, lane >> 5) * 16;
  const int pre_a = wk * KSW * 3 * LoadA::PLANE + wm * TM * 1024 + pre;
  const int pre_b = LoadA::BYTES + wk * KSW * 3 * LoadB::PLANE + wn * TN * 1024 + pre;
  auto read_a = [&](const char *stage, int s, int i, int buf) {
#pragma unroll
    for (int p = 0; p < 3; ++p)
      fa[buf][p] = *reinterpret_cast<const bf16x8_t *>(stage + pre_a + (s * 3 + p) * LoadA::PLANE + i * 1024);
  };
  auto read_b = [&](const char *stage, int s, int buf) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int p = 0; p < 3; ++p)
        fb[buf][j][p] = *reinterpret_cast<const bf16x8_t *>(stage + pre_b + (s * 3 + p) * LoadB::PLANE + j * 1024);
  };
  auto mfmas = [&](int i, int bufa, int bufb) {
    constexpr int PA[6] = {0, 2, 1, 0, 1, 0}, PB[6] = {2, 0, 1, 1, 0, 0};  // smallest first
#pragma unroll
    for (int p = 0; p < 6; ++p)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        f32x16_t &c = SMALL && p < 5 ? corr[i][j] : acc[i][j];
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[bufa][PA[p]], fb[bufb][j][PB[p]], c, 0, 0, 0);
      }
  };

  if (nk > 0) {
    la.init(static_cast<const char *>(g.A), g.lda * 4, (long)tile_m * BM, (long)kb0 * BK, tid);
    lb.init(static_cast<const char *>(g.B), g.ldb * 4, (long)tile_n * BN, (long)kb0 * BK, tid);
    auto request = [&](int kb, int set) {  // past the end: the last block again, which nobody reads
      kb = min(kb, nk - 1);
      la.load(ra[set], kb);
      lb.load(rb[set], kb);
    };
    auto land = [&](char *stage, int set) {
      la.store(stage, ra[set], big);
      lb.store(stage + LoadA::BYTES, rb[set], big);
    };
    request(0, 0);
    land(smem, 0);
#pragma unroll
    for (int p = 0; p < PF; ++p) request(p + 1, (p + 1) % PF);
    __syncthreads();
    read_b(smem, 0, 0);
    read_a(smem, 0, 0, 0);
    constexpr int GROUPS = KSW * TM;
    constexpr int UNROLL = PF > 2 ? PF : 2;
    for (int it0 = 0; it0 < nk; it0 += UNROLL) {
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) {
        const int it = it0 + u;
        if (it < nk) {
          const char *cur = smem + (u & 1) * STAGE;
          char *next = smem + ((u & 1) ^ 1) * STAGE;
          land(next, (u + 1) % PF);
          request(it + 1 + PF, (u + 1) % PF);
          // group q = (step, row block); fragments of A alternate by group, those of B by step
#pragma unroll
          for (int q = 0; q < GROUPS; ++q) {
            const int ga = u * GROUPS + q, gb = u * KSW + q / TM;
            if (q + 1 < GROUPS) {
              if ((q + 1) % TM == 0) read_b(cur, (q + 1) / TM, (gb + 1) & 1);
              read_a(cur, (q + 1) / TM, (q + 1) % TM, (ga + 1) & 1);
            } else {
              __syncthreads();
              __builtin_amdgcn_sched_barrier(0);
              read_b(next, 0, (gb + 1) & 1);
              read_a(next, 0, 0, (ga + 1) & 1);
            }
            mfmas(q % TM, ga & 1, gb & 1);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  }
  if constexpr (SMALL)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] += corr[i][j];
  const bool again = __syncthreads_or(__builtin_bit_cast(unsigned, big) >= SPLIT_MAX);
  if constexpr (WGK > 1) {
    static_assert(WGM * WGN * (WGK - 1) * TM * TN * 4096 <= split_lds_bytes<BM, BN, KS, Epi>(), "");
    float *part = reinterpret_cast<float *>(smem) + (long)(wave % (WGM * WGN)) * (TM * TN * 1024);
    auto at = [&](int i, int j, int r) { return part + ((i * TN + j) * 16 + r) * 64 + lane; };
    if (wk > 0) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) at(i, j, r)[(wk - 1) * (WGM * WGN * TM * TN * 1024)] = acc[i][j][r];
    }
    __syncthreads();
    if (wk > 0) return;  // (barriers below wait for the waves that are left)
#pragma unroll
    for (int q = 0; q < WGK - 1; ++q)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][j][r] += at(i, j, r)[q * (WGM * WGN * TM * TN * 1024)];
    __syncthreads();
  }
  if (again) {
    // An operand of this tile is infinite, or finite and so large that its upper part would be: its parts' products are not
    // the product's parts.  The tile again, on the fp32 matrix cores.
    epi.template init<TM, TN>(acc, tile_m * BM + wm * WTM, tile_n * BN + wn * WTN, lane, split);
    const int lr = lane & 31, lh = lane >> 5;
    const float *A = static_cast<const float *>(g.A) + (LA == ROWK ? ((long)tile_m * BM + wm * WTM + lr) * g.lda + lh
                                                                   : (long)tile_m * BM + wm * WTM + lr + lh * g.lda);
    const float *B = static_cast<const float *>(g.B) + (LB == ROWK ? ((long)tile_n * BN + wn * WTN + lr) * g.ldb + lh
                                                                   : (long)tile_n * BN + wn * WTN + lr + lh * g.ldb);
#pragma unroll 1
    for (long k = (long)kb0 * BK; k < (long)(kb0 + nk) * BK; k += 2) {
      float xa[TM], xb[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) xa[i] = LA == ROWK ? A[i * 32 * g.lda + k] : A[k * g.lda + i * 32];
#pragma unroll
      for (int j = 0; j < TN; ++j) xb[j] = LB == ROWK ? B[j * 32 * g.ldb + k] : B[k * g.ldb + j * 32];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(xa[i], xb[j], acc[i][j], 0, 0, 0);
    }
  }
  EpiCtx ctx;
  ctx.smem_lo = smem;
  ctx.smem_hi = smem;
#pragma unroll
  for (int qi = 0; qi < 4; ++qi) ctx.q[qi] = smem;
  ctx.tile_row0 = tile_m * BM;
  ctx.tile_col0 = tile_n * BN;
  ctx.wrow = wm * WTM;
  ctx.wcol = wn * WTN;
  ctx.lane = lane;
  ctx.tid = tid;
  ctx.split = split;
  epi.template run<BM, BN, TM, TN, WGM * WGN * 64>(acc, ctx);
}
#endif

template <int BM, int BN, int WGM, int WGN, int WGK, int LA, int LB, int KS, int PF, class Epi>
__global__ void __launch_bounds__(WGM *WGN *WGK * 64, (BM == 64 ? 4 : 2)) gemm_split_kernel(const GemmShape g, const Epi epi) {
#if defined(__HIP_DEVICE_COMPILE__)
  __shared__ __attribute__((aligned(1024))) char smem[split_lds_bytes<BM, BN, KS, Epi>()];
  gemm_split_item<BM, BN, WGM, WGN, WGK, LA, LB, KS, PF, Epi>(g, epi, blockIdx.x, smem);
#endif
}

// The 32-bit byte offsets of the loads cover a tile's rows (ROWK), or a block's rows of k (KROW).
inline bool split_reaches(int layout, long ld, int rows, int bk) { return (layout == ROWK ? rows : bk) * ld * 4 < (1L << 31); }

template <int BM, int BN, int LA, int LB, int KS>
inline hipError_t split_shape(GemmShape &g, const void *A, long lda, const void *B, long ldb, long Mg, long Ng, long K,
                              int splits, int band) {
  if (Mg <= 0 || Ng <= 0 || K < 0 || Mg % BM || Ng % BN || K % 32 || splits < 1) return hipErrorInvalidValue;
  g.A = A;
  g.B = B;
  g.lda = lda;
  g.ldb = ldb;
  g.bytesA = g.bytesB = 0;
  g.tilesM = (int)(Mg / BM);
  g.tilesN = (int)(Ng / BN);
  // splits are made of blocks of 32, or of the kernel's own where those are larger
  constexpr int BK = 16 * KS, UNIT = BK > 32 ? BK : 32;
  if (K % BK || !split_reaches(LA, lda, BM, BK) || !split_reaches(LB, ldb, BN, BK)) return hipErrorInvalidValue;
  g.kBlocks = (int)(K / BK);
  g.kBlocksPerSplit = (int)((K / UNIT + splits - 1) / splits) * (UNIT / BK);
  g.splits = splits;
  const long total = (long)g.tilesM * g.tilesN * splits;
  if (band == 0 || total > (1L << 30)) return hipErrorInvalidValue;
  g.perXcd = (int)((total + NUM_XCD - 1) / NUM_XCD);
  g.bandOverN = band < 0;
  g.band = band < 0 ? -band : band;
  return hipSuccess;
}

template <int BM, int BN, int WGM, int WGN, int WGK, int LA, int LB, int KS, int PF, class Epi>
inline hipError_t launch_gemm_split(hipStream_t stream, const void *A, long lda, const void *B, long ldb, long Mg, long Ng,
                                    long K, int splits, const Epi &epi, int band = 4) {
  static_assert(split_lds_bytes<BM, BN, KS, Epi>() <= 160 * 1024, "tile does not fit the 160 KB of LDS");
  GemmShape g;
  const hipError_t e = split_shape<BM, BN, LA, LB, KS>(g, A, lda, B, ldb, Mg, Ng, K, splits, band);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((gemm_split_kernel<BM, BN, WGM, WGN, WGK, LA, LB, KS, PF, Epi>), dim3((unsigned)(g.perXcd * NUM_XCD)),
                     dim3(WGM * WGN * WGK * 64), 0, stream, g, epi);
  return hipGetLastError();
}

}  // namespace rnnlm_dev
