// Host side of the C ABI declared in include/rnnlm.h: argument validation, workspace carving and
// the kernel sequence of one window (Sec. 4.1 / 4.2 of the paper; see the header for the model).
#include "../../include/rnnlm.h"

#include <math.h>
#include <stdlib.h>

#include <algorithm>
#include <mutex>
#include <new>
#include <vector>

#include "common.h"
#include "gemm.h"
#include "gemm_dma.h"
#include "gemm_dma4.h"
#include "kernels.h"
#include "nce.h"
#include "rmsprop.h"
#include "gemm_ring64.h"
#include "gemm_split.h"
#include "gemm_tail.h"
#include "rnn_persistent.h"
#include "rnn_resident.h"
#include "rnn_step.h"
#include "update.h"

using namespace rnnlm_dev;

#define HIP_TRY(expr)                        \
  do {                                       \
    hipError_t e_ = (expr);                  \
    if (e_ != hipSuccess) return RNNLM_ERR_HIP; \
  } while (0)

struct WsLayout {
  size_t Wo_c, U_c, UT_c, Hs_c, ZT, dA_c, X32, dHs32, dA32, part32, stat, lse, zy, logp_int, xp, yp, perm, seg, xtmp, ytmp,
      scalars, total;
  // noise-contrastive calls (present when K_max > 0)
  size_t Wn_c, Spart, dS_c, G32, noff, ndt, nct, gcol, ids, perm2, seg2;
  // rmsprop calls (present when cfg.rmsprop != 0): gradient buffers the redirected update epilogues fill
  size_t gWo, gU, gb, gN, gbN;
  // compressed architecture (present when cfg.P > 0; then Wo_c holds the compute copy of the tied matrix E)
  size_t A_c, C_c, Xp_c, P_c, dP_c, dX32;
  // partial sums of the chip-resident recurrent kernel (present for Hp = 4096, 256 streams, bf16)
  size_t part_res, sync, ring;
  bool has_part_res;
  long partElems;
};

struct EventPair {
  hipEvent_t start, stop;
  int stage;
};

// How a window of so many positions runs: rows the contractions walk, and the bf16 contraction over the vocabulary.  Worked
// out when the length of the window changes (10 us of estimates).
struct SumPlan {
  int tile, splits;
  long feats;
  double us;
};
struct WindowPlan {
  long Mrows = -1, Mp = 0;
  int parts = 0;  // softmax statistics of a position
  SumPlan sum = {};
};

struct rnnlm {
  rnnlm_config cfg;
  rnnlm_buffers buf;
  int Hp, Vp, Bp, MpMax;
  int Pp;     // cfg.P rounded up to the tile size (0: plain architecture)
  int D, Dp;  // width of the output layer's input: H / Hp, or P / Pp for the compressed architecture
  int KpMax;  // K_max rounded up to the tile size (0: no noise-contrastive workspace)
  RecurrentPlan plan;
  WindowPlan window;
  WsLayout L;
  char *ws;
  // stage timing (host-side only)
  // the integer helpers of the row updates (sort by id, run starts) depend on the token ids only: they run
  // on a second stream (default priority) next to the recurrent forward pass and are joined before the updates
  hipStream_t side = nullptr;
  hipEvent_t ev_fork[2] = {nullptr, nullptr}, ev_join[2] = {nullptr, nullptr};
  bool xcd_local = false;        // the probe at init saw round-robin placement over 8 XCDs
  int exchange_mode = RNNLM_EXCHANGE_AUTO;  // how the persistent recurrent kernels exchange state between workgroups
  unsigned spin_limit = 1u << 18;  // polls of a recurrent kernel's wait before giving up (about a second)
  uint32_t prof_mask = 0;
  std::vector<EventPair> prof_pool;
  size_t prof_used = 0;
  long prof_open[RNNLM_STAGE_COUNT] = {0};
  double prof_ms[RNNLM_STAGE_COUNT] = {0};
  int64_t prof_n[RNNLM_STAGE_COUNT] = {0};
};

namespace {
constexpr size_t PROF_MAX_PAIRS = 16384;

// Records a start event now and a stop event when it goes out of scope, if the stage is enabled.
struct StageTimer {
  rnnlm *h;
  hipStream_t st;
  EventPair *p = nullptr;
  bool close_;
  // open/close: a stage made of several launches opens its pair at the first launch and closes it at
  // the last (stage < 0: nothing to do for the launches in between).
  StageTimer(rnnlm *h_, int stage, hipStream_t st_, bool open = true, bool close = true)
      : h(h_), st(st_), close_(close) {
    if (stage < 0 || !(h->prof_mask & (1u << stage))) return;
    if (!open) {
      if (h->prof_open[stage] >= 0) p = &h->prof_pool[h->prof_open[stage]];
      return;
    }
    h->prof_open[stage] = -1;
    if (h->prof_used == h->prof_pool.size()) {
      if (h->prof_pool.size() >= PROF_MAX_PAIRS) return;
      EventPair e;
      if (hipEventCreate(&e.start) != hipSuccess) return;
      if (hipEventCreate(&e.stop) != hipSuccess) {
        (void)hipEventDestroy(e.start);
        return;
      }
      h->prof_pool.push_back(e);
    }
    h->prof_open[stage] = (long)h->prof_used;
    p = &h->prof_pool[h->prof_used++];
    p->stage = stage;
    (void)hipEventRecord(p->start, st);
  }
  ~StageTimer() {
    if (p && close_) (void)hipEventRecord(p->stop, st);
  }
};
// Stages that would share a launch take launches of their own while one of them is timed.
bool timed(const rnnlm *h, std::initializer_list<int> stages) {
  for (int s : stages)
    if (h->prof_mask & (1u << s)) return true;
  return false;
}
}  // namespace

namespace {

// Tile shape of the three output-layer contractions and of the recurrent weight gradient: 256x256
// output tile, 8 waves as 2 x 4 (wave tile 128 x 64).
constexpr int BIG = 256;

// fp32 contractions (gemm_split.h): 256x256 output tiles on eight waves, 128x128 on eight that share out the contraction in
// pairs, 64x64 on four or, where there are few tiles, on eight or sixteen that share it out.  The contraction over the
// vocabulary (ld > 0: row length of its K-major logits) takes 256x128 tiles instead of 256x256, which leave registers for the
// lesser products' own accumulators: 7 % slower, but with all products in one accumulator its gradients are further from 64
// bits than through the fp32 matrix cores (input rows, V = 3209, H = 852, 512x32: 1.56 times as far, now 0.74; V = 1200, H =
// 2000, 256x32: 1.83 and 0.75).
// Contractions of up to 64 terms take 64x64 tiles on the fp32 cores (parts = 0, gemm_dma4.h), which round less there (split,
// 4..30 terms: 1.3 times as far from 64 bits); longer ones take them where the estimate is lowest.
// The tile and the number of splits of the contraction dimension minimise an estimate of the time, fitted to runs of
// 16..2560 tiles and depths of 32..4096 (both operands K-contiguous, both K-major; us, kb = 32-deep blocks): every full
// round of 256 tiles 10.5 + 4.45 kb (256x256) and 4.6 + 1.3 kb (128x128: one workgroup per compute unit; a partly filled
// round runs at a higher clock); 64x64, one workgroup per compute unit 3.2 + 0.69 kb on four waves, 3.8 + 0.51 kb on eight,
// 5.7 + 0.47 kb on sixteen, four per compute unit 5.2 + 1.77 kb; every split adds a pass over the output.
struct F32Plan {
  // parts: groups of waves that share out the contraction (0: fp32 matrix cores; tile 256, parts 2: 256x128)
  int tile, parts, splits;
  double us;
};
// A handle of millions of positions takes the forms whose blocks of 16 KS rows of ld values the loads' 32-bit offsets still
// reach (64 x 64 in steps of 16 always).
constexpr long F32_SHORT = 64;  // terms up to which a sum rounds less on the fp32 cores
F32Plan f32_plan(long Mg, long Ng, long K, int max_splits, long ld = 0) {
  const long kb = (K + 31) / 32;
  const bool split = K > F32_SHORT;
  const bool reach32 = split_reaches(KROW, ld, 0, 32), reach64 = split_reaches(KROW, ld, 0, 64);
  F32Plan best = {64, 0, 1, 1e30};
  for (int S = 1; S <= max_splits && S <= kb; ++S) {
    const long per = (kb + S - 1) / S;
    const double pass = S > 1 ? 5.0 + (S + 1) * (double)Mg * Ng * 4.0 / 4e6 : 0.0;
    auto consider = [&](int tile, int parts, double us) {
      if (us + pass < best.us) best = {tile, parts, S, us + pass};
    };
    auto whole = [&](int rows, int cols, double fixed, double unit, double half) {  // one workgroup per compute unit
      const long w = (Mg / rows) * (Ng / cols) * S, rest = w % 256;
      return 2.0 + w / 256 * (fixed + unit * per) + (rest ? fixed + (half + (unit - half) * rest / 256) * per : 0.0);
    };
    if (split && ld == 0 && Mg % 256 == 0 && Ng % 256 == 0) consider(256, 1, whole(256, 256, 10.5, 4.45, 3.2));
    if (split && ld > 0 && reach32 && Mg % 256 == 0 && Ng % 128 == 0) consider(256, 2, whole(256, 128, 7.0, 2.4, 1.75));
    if (split && reach32 && Mg % 128 == 0 && Ng % 128 == 0) consider(128, 2, whole(128, 128, 4.6, 1.3, 1.05));
    const long w = (Mg / 64) * (Ng / 64) * S, share = std::min<long>((w + 255) / 256, 4);
    const double more = std::max(1.0, w / 1024.0);
    consider(64, 0, 2.1 + 0.85 * share + (more - 1) * 2.0 + (0.15 + 0.49 * share) * per * more);
    if (!split) continue;
    consider(64, 1, 2.6 + 0.65 * share + (more - 1) * 2.2 + (0.33 + 0.36 * share) * per * more);
    if (w <= 256 && reach32) consider(64, 2, 3.8 + 0.51 * per);
    if (w <= 256 && reach64) consider(64, 4, 5.7 + 0.47 * (per + per % 2));
  }
  return best;
}
// fp32: an extent of `valid` rows or columns, padded to 64, 128 or 256 by what the product with the other extent takes
// (the buffers are padded to 256).
long f32_extent(long valid, long other, long K, int max_splits, long ld = 0) {
  long best = round_up(valid, 256);
  double us = f32_plan(other, best, K, max_splits, ld).us;
  for (long pad = 128; pad >= 64; pad /= 2) {
    const long n = round_up(valid, pad);
    const double t = f32_plan(other, n, K, max_splits, ld).us;
    if (t <= us) {
      us = t;
      best = n;
    }
  }
  return best;
}
// Terms of a contraction of n: what lies between them and the padded extent (tiles of 256) is zero in both operands, so
// only the last block of 128 bytes is taken whole (bf16, V = 33278, H = 650, 100x9, padded terms and these: window 338.8 and
// 335.5 us).
template <typename T>
long terms(long n) {
  return round_up(n, Elem<T>::BK);
}
template <int LA, int LB, class Epi>
hipError_t f32_gemm(hipStream_t st, const void *A, long lda, const void *B, long ldb, long Mg, long Ng, long K,
                    const F32Plan &plan, const Epi &epi, int band = 4) {
  if constexpr (LA == KROW && LB == KROW && std::is_same_v<Epi, EpiPartial>)
    if (plan.tile == 256 && plan.parts == 2)
      return launch_gemm_split<256, 128, 4, 2, 1, LA, LB, 2, 1>(st, A, lda, B, ldb, Mg, Ng, K, plan.splits, epi, band);
  if (plan.tile == 256)
    return launch_gemm_split<256, 256, 2, 4, 1, LA, LB, 1, 1>(st, A, lda, B, ldb, Mg, Ng, K, plan.splits, epi, band);
  if (plan.tile == 128)
    return launch_gemm_split<128, 128, 2, 2, 2, LA, LB, 2, 1>(st, A, lda, B, ldb, Mg, Ng, K, plan.splits, epi, band);
  if (plan.parts == 4)  // (operands are padded to 64 at least)
    return launch_gemm_split<64, 64, 2, 2, 4, LA, LB, 4, 2>(st, A, lda, B, ldb, Mg, Ng, round_up(K, 64), plan.splits, epi, band);
  if (plan.parts == 2)
    return launch_gemm_split<64, 64, 2, 2, 2, LA, LB, 2, 2>(st, A, lda, B, ldb, Mg, Ng, K, plan.splits, epi, band);
  if (plan.parts == 1)
    return launch_gemm_split<64, 64, 2, 2, 1, LA, LB, 1, 2>(st, A, lda, B, ldb, Mg, Ng, K, plan.splits, epi, band);
  return launch_gemm_dma4<float, 64, 64, 2, 2, LA, LB>(st, A, lda, B, ldb, Mg, Ng, K, plan.splits, epi, band);
}

// bf16 contractions: output tiles of 256x256 (one persistent workgroup of eight waves per compute unit), 128x128 (eight
// waves, two workgroups per compute unit) or 64x64 (four waves).  The large tiles read an operand least often and win where
// they fill the chip for some rounds; with fewer, most compute units idle and a lone workgroup is slow (its epilogue alone
// takes 8-20 us).  The tile minimises an estimate of the time, fitted to runs of 16..20480 tiles and depths of 64..2560
// (us; w workgroups, K terms each); a hot run of each form at V x M (H = 512) resp. V x H (1024 positions), 256 / 128 / 64:
//   output layer 10240 x 256: 19.1 / 8.4 / 9.6; 4096 x 1024: 19.8 / 9.0 / 11.6; 10240 x 2560: 43.9 / 44.2 / 56; 32768 x 2560:
//   117 / 127 / 184;
//   output update 4096 x 256: 31.4 / 11.1 / 7.7; 10240 x 512: 34.3 / 22.8 / 24.3; 10240 x 1024: 38.8 / 36.2 / 44; 32768 x 1024:
//   102 / 104 / 139.
// Windows whose operands are not in the caches take longer than a hot run (V = 33278, H = 650, 900 positions: the output layer,
// put at 62, takes 78).
// 128x128 on four waves is slower nearly everywhere (output layer 10240 x 1024: 22.3, on eight 19.5), waves that share out
// the contraction gain 10-15 % only where 64x64 tiles are few and deep.
enum Bf16Kind { OUT_FWD, OUT_UPDATE, PLAIN_SUM };  // by epilogue: statistics and logits, weight update, fp32 store
double bf16_all_us(Bf16Kind kind, int tile, long Mg, long Ng, long K, int splits = 1) {
  const double w = (double)(Mg / tile) * (Ng / tile) * splits, k = (double)((K / 64 + splits - 1) / splits * 64);
  // MB of an update (10 bytes a weight) beyond what the memory-side cache holds
  const double beyond = std::max(0.0, (double)Mg * Ng * 1e-5 - 170.0);
  if (tile == 256) {
    if (kind == PLAIN_SUM) return 6.0 + std::ceil(w / 256) * k * (0.0078 + 0.018 * std::min(1.0, w / 256));
    const double rounds = std::floor(w / 256), rest = w / 256 - rounds;
    const bool fwd = kind == OUT_FWD;
    double us = 1.0 + rounds * (fwd ? 10.9 + 0.024 * k : 24.0 + 0.0265 * k);
    if (rest > 0) us += fwd ? 10.9 + 0.0155 * k + rest * (1.5 + 0.0045 * k) : 13.5 + 0.0168 * k + rest * rest * (10.5 + 0.0095 * k);
    return us + (fwd ? 0.0 : std::max(0.03, 0.105 - 4.4e-5 * k) * beyond);
  }
  // one workgroup alone; a workgroup's share of the chip's time, where every compute unit has some
  double alone, share;
  if (tile == 128) {
    alone = (kind == OUT_UPDATE ? 5.0 : kind == OUT_FWD ? 4.9 : 4.0) + 0.0053 * k;
    share = kind == OUT_UPDATE ? 0.0235 + 2.65e-5 * k + 2e-9 * k * k : kind == OUT_FWD ? 0.0095 + 3.38e-5 * k : 0.006 + 2.95e-5 * k;
  } else {
    alone = (kind == OUT_UPDATE ? 3.6 : kind == OUT_FWD ? 4.0 : 2.9) + 0.0033 * k;
    share = kind == OUT_UPDATE ? 0.005 + 1.4e-5 * k : kind == OUT_FWD ? 0.0023 + 1.43e-5 * k : 0.0024 + 1.18e-5 * k;
  }
  // per_cu: workgroups a compute unit takes before its matrix cores are busy
  const double per_cu = tile == 128 ? 1.0 : 4.0, full = 3.0 + 256 * per_cu * share;
  const double fill = (w <= 256 ? w / 256 : std::ceil(w / 256)) / per_cu;
  double us;
  if (fill <= 1.0)
    us = alone + std::max(0.0, full - alone) * fill * fill;
  else  // (up to twice that, the fuller compute units take longer than the mean)
    us = std::max(alone, 3.0 + share * (fill <= 2.0 ? (2 * w + 512 * per_cu) / 3 : w));
  if (kind == OUT_UPDATE) us += (tile == 128 ? std::min(0.14, 0.08 + 1.2e-4 * k) : std::min(0.12, 0.05 + 3e-4 * k)) * beyond;
  // long sums whose operands no L2 holds: what all tiles fetch, at what the fabric delivers
  if (kind == PLAIN_SUM && (double)(Mg + Ng) * K > 4e7) {
    const double f = 4.0 * K * Mg * Ng / tile / 11e6;
    us = std::sqrt(std::sqrt(us * us * us * us + f * f * f * f));
  }
  return us;
}
// Rows of the output layer that 256x256 tiles take (gemm_tail.h): whole rounds of them where the rest is faster on 128x128 by
// a good part of a round, or all (V = 10000, P = 512, 128x20, 1.56 rounds, whose rest is as long on small tiles: output layer
// 49.7 and 52.4 us).
long large_rows(long Mg, long Ng, long K, double *us = nullptr) {
  const double all = Mg % 256 || Ng % 256 ? 0.0 : bf16_all_us(OUT_FWD, 256, Mg, Ng, K);
  if (us) *us = all;
  if (Mg % 256 || Ng % 256) return Mg;  // (no large tiles)
  const long cols = Ng / 256, rounds = Mg / 256 * cols / 256, rows = rounds * 256 / cols * 256;
  if (rows == 0 || rows >= Mg) return Mg;  // (0: the whole rounds do not fill a row of tiles)
  const double mixed = bf16_all_us(OUT_FWD, 256, rows, Ng, K) + bf16_all_us(OUT_FWD, 128, Mg - rows, Ng, K) - 3.0;
  if (mixed >= 0.85 * all && all - mixed < 8.0) return Mg;
  if (us) *us = mixed;
  return rows;
}
double bf16_us(Bf16Kind kind, int tile, long Mg, long Ng, long K, int splits = 1) {
  if (tile != 256 || kind != OUT_FWD) return bf16_all_us(kind, tile, Mg, Ng, K, splits);
  double us;
  large_rows(Mg, Ng, K, &us);
  return us;
}
// Mg a multiple of 256, Ng of 64: the tile that is fastest among those that divide them (window positions and widths of
// layers are padded to as little as the tile asks for: a window of 77 positions has 128, not 256).  The persistent 256x256
// forms are kept where the gain would be small (update 16 %: it shares the chip with the other stream's work, for
// which they leave room; V = 40000, H = 500, 120x18, update on 157 x 2 large tiles 539.7 us a window, on 128x128 544.1).
constexpr double KEEP_LARGE = 0.95, KEEP_LARGE_SUM = 0.92, KEEP_LARGE_UPDATE = 0.84;
int bf16_tile(Bf16Kind kind, long Mg, long Ng, long K, int splits = 1) {
  int best = 64;
  double us = bf16_us(kind, 64, Mg, Ng, K, splits);
  for (int tile : {128, 256}) {
    if (Mg % tile || Ng % tile) continue;
    const double t = bf16_us(kind, tile, Mg, Ng, K, splits) *
                     (tile < 256 ? 1.0 : kind == OUT_UPDATE ? KEEP_LARGE_UPDATE : KEEP_LARGE);
    if (t <= us) {
      us = t;
      best = tile;
    }
  }
  return best;
}
// Softmax statistics of the output layer: a partial per tile row block and position.
long stat_parts(long Vp, long Mp, long K) {
  const int tile = bf16_tile(OUT_FWD, Vp, Mp, K);
  if (tile < 256) return Vp / tile;
  const long rows = large_rows(Vp, Mp, K);
  return rows / 256 + (Vp - rows) / 128;
}
// An extent of `valid` rows or columns, padded to 64, 128 or 256 by what the contraction with the other extent takes.
long bf16_extent(Bf16Kind kind, long valid, long other, long K) {
  long best = 0;
  double us = 1e30;
  for (long pad : {256, 128, 64}) {
    const long n = round_up(valid, pad);
    const double t = bf16_us(kind, bf16_tile(kind, other, n, K), other, n, K);
    if (t < us) {
      us = t;
      best = n;
    }
  }
  return best;
}

// The large bf16 contractions take the direct global->LDS kernels.
// RING4: the four-stage ring of 32-deep K blocks (deeper prefetch; pays when at least one operand is
// K-major, whose 32-deep blocks are still made of full cache lines) instead of two stages of 64.
template <int WGM, int WGN, int LA, int LB, bool RING4, class Epi>
hipError_t big_gemm(hipStream_t st, const void *A, long lda, const void *B, long ldb, long Mg, long Ng, long K,
                    int splits, const Epi &epi, int band = 4) {
  if constexpr (RING4) {
    // epilogues that leave the LDS alone run as one persistent workgroup per compute unit, which requests the
    // next tile's first K blocks before its epilogue
    constexpr bool PERSIST = Epi::template lds_bytes<BIG, BIG>() == 0;
    return launch_gemm_dma4<bf16_t, BIG, BIG, WGM, WGN, LA, LB, PERSIST>(st, A, lda, B, ldb, Mg, Ng, K, splits, epi, band);
  } else {
    return launch_gemm_dma<BIG, BIG, WGM, WGN, LA, LB>(st, A, lda, B, ldb, Mg, Ng, K, splits, epi, band);
  }
}

// bf16 contractions on 128x128 or 64x64 tiles: the ring, whose three K blocks in flight are what keeps a lone workgroup's
// matrix cores fed (register-staged 64x64 tiles took 0.65 us per 64 values of the contraction, the ring 0.4).
template <int LA, int LB, class Epi>
hipError_t bf16_small_gemm(hipStream_t st, const void *A, long lda, const void *B, long ldb, long Mg, long Ng, long K,
                           int tile, int splits, const Epi &epi, int band = 4) {
  if (tile == 128) return launch_gemm_dma4<bf16_t, 128, 128, 4, 2, LA, LB>(st, A, lda, B, ldb, Mg, Ng, K, splits, epi, band);
  return launch_gemm_dma4<bf16_t, 64, 64, 2, 2, LA, LB>(st, A, lda, B, ldb, Mg, Ng, K, splits, epi, band);
}

// The mid-sized contractions (noise-panel products, the layers of the compressed architecture, the recurrent weight
// gradient): 128x128 or 64x64 output tiles, whichever the estimate favours (128 where it is close: those read less).
int mid_tile(long Mg, long Ng, long K, int splits) {
  if (Mg % 128 || Ng % 128) return 64;
  return bf16_us(PLAIN_SUM, 128, Mg, Ng, K, splits) <= bf16_us(PLAIN_SUM, 64, Mg, Ng, K, splits) ? 128 : 64;
}
template <typename T, int LA, int LB, class Epi>
hipError_t mid_gemm(hipStream_t st, const void *A, long lda, const void *B, long ldb, long Mg, long Ng, long K,
                    int splits, const Epi &epi, int band = 4) {
  // the direct-load kernels address a bf16 K-major operand's k blocks with a 32-bit scalar offset
  const bool fits = !((LA == KROW && K * lda * 2 >= (1L << 31)) || (LB == KROW && K * ldb * 2 >= (1L << 31)) ||
                      lda * 2 * 128 >= (1L << 31) || ldb * 2 * 128 >= (1L << 31));
  if constexpr (sizeof(T) == 4) {
    F32Plan plan = f32_plan(Mg, Ng, K, 1);
    plan.splits = splits;
    return f32_gemm<LA, LB>(st, A, lda, B, ldb, Mg, Ng, K, plan, epi, band);
  } else {
    if (fits) return bf16_small_gemm<LA, LB>(st, A, lda, B, ldb, Mg, Ng, K, mid_tile(Mg, Ng, K, splits), splits, epi, band);
    if (Mg % 128 || Ng % 128) return launch_gemm<T, 64, 64, 2, 2, LA, LB>(st, A, lda, B, ldb, Mg, Ng, K, splits, epi, band);
    return launch_gemm<T, 128, 128, 2, 2, LA, LB>(st, A, lda, B, ldb, Mg, Ng, K, splits, epi, band);
  }
}

inline size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

bool cfg_ok(const rnnlm_config *c) {
  if (!c) return false;
  if (c->V <= 0 || c->H <= 0 || c->B <= 0 || c->T_max <= 0) return false;
  if (c->precision != RNNLM_FP32 && c->precision != RNNLM_BF16_FP32MASTER) return false;
  if (c->device < 0) return false;
  if (c->K_max < 0 || c->K_max > 65536) return false;
  if (c->rmsprop != 0 && c->rmsprop != 1) return false;
  if ((long)c->B * c->T_max > (1L << 24)) return false;
  if (c->P < 0 || (c->P > 0 && (c->K_max != 0 || c->rmsprop != 0))) return false;
  return true;
}

constexpr int MAX_SPLITS = 16;
// Splits of the bf16 contraction over the vocabulary (kBlocks 64-deep blocks, 256x256 tiles, at most one workgroup per
// compute unit): up to 16, and more where the output has so few tiles that most of the chip would be idle and an estimate,
// in us, of a workgroup's share and of the pass that adds up the parts is a tenth lower.  Windows with at most 16 and with
// these: V = 30000, H = 256, 16x8 144.5 and 125.2 us, 32x16 161.2 and 144.8; V = 64000, H = 1024, 16x16 375.9 and 352.8; V =
// 100000, H = 2048, 8x8 925.3 and 891.5 (V = 33278, H = 650, 100x9: 16 splits 317.6, 21 would take 329.1).
constexpr int BF16_SPLITS = 64;
int desired_splits(long Mp, long Hp, long kBlocks) {
  const long tiles = (Mp / BIG) * (Hp / BIG), most = std::min<long>(std::max<long>(1, 256 / tiles), kBlocks);
  auto estimate = [&](long S) {
    return 6.0 + (kBlocks + S - 1) / S * (0.5 + 1.15 * std::min(1.0, tiles * S / 256.0)) +
           (S > 1 ? 5.0 + (S + 1) * (double)Mp * Hp * 4.0 / 3.5e6 : 0.0);
  };
  long best = std::min<long>(most, MAX_SPLITS);
  double us = 0.9 * estimate(best);
  for (long S = best + 1; S <= std::min<long>(most, BF16_SPLITS); ++S) {
    const long per = (kBlocks + S - 1) / S;
    if ((kBlocks + per - 1) / per == S && estimate(S) < us) {  // (else the last ones would be empty)
      us = estimate(S);
      best = S;
    }
  }
  return (int)best;
}

// Tile and splits of the bf16 contraction over the vocabulary: 256x256 tiles with the splits above, or smaller ones, where
// few splits fill the chip and the pass over the parts is short, by the same estimate.  Window positions and features are
// taken as 256-multiples by the large tiles; `feats` as the small ones take them.  (V = 10000, H = 512, 256 positions: 16
// parts on 256x256 tiles 18.3 us and a pass of 5.4, now 7.2 and 4.8.)
SumPlan bf16_sum_plan(long Mp, long D, long K, bool padded_feats) {
  const long Dp = round_up(D, PAD_H), kBlocks = K / 64;
  SumPlan best = {64, 1, padded_feats ? Dp : round_up(D, 64), 1e30};
  auto consider = [&](int tile, int S, long feats) {
    const double t = bf16_us(PLAIN_SUM, tile, Mp, feats, K, S) * (tile == 256 ? KEEP_LARGE_SUM : 1.0) + (S > 1 ? 5.0 + (S + 1) * (double)Mp * Dp * 4.0 / 7e6 : 0.0);
    if (t < best.us) best = {tile, S, feats, t};
  };
  if (Mp % 256 == 0) consider(256, desired_splits(Mp, Dp, kBlocks), Dp);
  for (int tile : {128, 64}) {
    if (Mp % tile) continue;
    const long feats = padded_feats ? Dp : round_up(D, tile), tiles = (Mp / tile) * (feats / tile);
    for (long S = 1; S <= std::min<long>(kBlocks, BF16_SPLITS) && (S == 1 || tiles * S <= 1024); ++S) {
      const long per = (kBlocks + S - 1) / S;
      if ((kBlocks + per - 1) / per == S) consider(tile, (int)S, feats);  // (else the last ones would be empty)
    }
  }
  return best;
}

// A wave's share of the matrix has to fit its registers: four waves and 32 units per workgroup up to 1024 units, eight
// waves with half the registers and 64 units up to 2048 (bf16 fragments only).  Streams are split into at most eight
// groups where 32 streams per group allow it (one group per XCD: a step's time grows with the state a compute unit
// loads), and the grid is small enough to be co-resident with one workgroup per compute unit.
RecurrentPlan recurrent_plan(const rnnlm_config &c) {
  RecurrentPlan p = {};
  if (c.H > (c.precision == RNNLM_FP32 ? 1024 : 2048)) return p;
  p.waves = c.H <= 1024 ? 4 : 8;
  p.units = c.H <= 1024 ? 32 : 64;
  const int nwg = (c.H + p.units - 1) / p.units;
  p.R = std::min(32, (c.B + NUM_XCD - 1) / NUM_XCD);
  p.groups = (c.B + p.R - 1) / p.R;
  p.rt = (p.R + 15) / 16;
  p.width = nwg * p.units;
  p.nkb = p.width / 32;
  p.ks = (p.nkb + p.waves - 1) / p.waves;
  if ((long)p.groups * nwg <= 256) p.nwg = nwg;
  return p;
}

// Per-step recurrent path for shapes neither the persistent kernel nor a step in one launch covers: the step's contraction is split over its
// contraction dimension, then one pass sums the parts and applies the elementwise part.  Whole blocks of 256 streams of a
// wide layer: 256 x 128 tiles (fp32: 256 x 64, register-staged), one workgroup per compute unit.  Everything else: 64 x 64
// tiles of the ring, up to eight splits and two workgroups per compute unit: the step is bound by the latency of a
// workgroup's share of the contraction and by the matrix's way through the caches, so many short shares beat few long
// ones (per step, 32 x 64 tiles over the whole contraction dimension against this: fp32 H = 1408, 64 streams 42 and 12.5 us;
// bf16 H = 4096, 64 streams 39 and 15, H = 2500, 8 streams 24 and 11).
struct StepPlan {
  bool wide;   // 256-row tiles
  int splits;
  long rows;   // rows of a partial product
};
StepPlan step_plan(const rnnlm_config &c, int Bp, int Hp) {
  const bool f32 = c.precision == RNNLM_FP32;
  const long kBlocks = (f32 ? terms<float>(c.H) / 32 : terms<bf16_t>(c.H) / 64);
  if (Bp % 256 == 0 && Hp >= 2048) {
    const long tiles = (long)(Bp / 256) * (Hp / (f32 ? 64 : 128));
    return {true, (int)std::min({std::max<long>(1, 256 / tiles), 8L, kBlocks}), Bp};
  }
  const long rows = round_up(Bp, 64), tiles = (rows / 64) * (Hp / 64);
  return {false, (int)std::min({std::max<long>(1, 512 / tiles), 8L, kBlocks}), rows};
}

// Rows the contractions of a window of Mrows positions walk (MpMax is a multiple of 256).  Long windows keep whole 256-row
// tiles: the padding is below 2 % there.
constexpr long TRIM_ROWS = 16384;
long window_rows(const rnnlm_config &c, long Mrows) {
  if (Mrows > TRIM_ROWS) return round_up(Mrows, PAD_M);
  if (c.precision != RNNLM_FP32) {
    // what the output layer, the pass over the logits and the contraction over the vocabulary take of them
    const long Vp = round_up(c.V, PAD_V), D = c.P > 0 ? c.P : c.H, K = terms<bf16_t>(D);
    long best = 0;
    double us = 1e30;
    for (long pad : {256, 128, 64}) {
      const long n = round_up(Mrows, pad);
      const double t = bf16_us(OUT_FWD, bf16_tile(OUT_FWD, Vp, n, K), Vp, n, K) + 0.75e-6 * n * Vp +
                       bf16_sum_plan(n, D, Vp, c.P > 0).us;
      if (t < us) {
        us = t;
        best = n;
      }
    }
    return best;
  }
  return f32_extent(Mrows, round_up(c.V, PAD_V), c.P > 0 ? c.P : c.H, 1);
}
// Columns the contraction over the vocabulary forms: the compressed architecture reads the padding, too.
long features_formed(const rnnlm_config &c, long Mp, int max_splits, long ldz) {
  return c.P > 0 ? round_up(c.P, PAD_H) : f32_extent(c.H, Mp, c.V, max_splits, ldz);
}

void make_layout(const rnnlm_config &c, int &Hp, int &Vp, int &Bp, int &MpMax, int &KpMax, WsLayout &L) {
  const size_t es = (c.precision == RNNLM_FP32) ? 4 : 2;
  const int Pp = (int)round_up(c.P, PAD_H);
  Hp = (int)round_up(c.H, PAD_H);
  const int Dp = Pp > 0 ? Pp : Hp;
  Vp = (int)round_up(c.V, PAD_V);
  // streams are taken as they come, except by the kernels built for whole blocks of 256
  const RecurrentPlan plan = recurrent_plan(c);
  Bp = plan.nwg == 0 && Hp >= 2048 && round_up(c.B, PAD_B) % 256 == 0 ? (int)round_up(c.B, PAD_B) : c.B;
  MpMax = (int)round_up((long)c.T_max * Bp, PAD_M);
  // softmax statistics: a partial per tile row block and position (fp32: of the smallest tile)
  long statElems = (long)(Vp / 64) * MpMax;
  if (es == 4) {
    L.partElems = (long)MpMax * Dp;
    for (long M = 64; M <= MpMax; M += M < TRIM_ROWS ? 64 : PAD_M)
      L.partElems = std::max(
          L.partElems, f32_plan(M, features_formed(c, M, MAX_SPLITS, MpMax), c.V, MAX_SPLITS, MpMax).splits * M * Dp);
  } else {
    L.partElems = statElems = 0;
    for (long M = 64; M <= MpMax; M += M < TRIM_ROWS ? 64 : PAD_M) {
      L.partElems = std::max(L.partElems, bf16_sum_plan(M, Pp > 0 ? c.P : c.H, Vp, Pp > 0).splits * M * Dp);
      statElems = std::max(statElems, stat_parts(Vp, M, terms<bf16_t>(Pp > 0 ? c.P : c.H)) * M);
    }
  }
  const StepPlan step = step_plan(c, Bp, Hp);
  if (plan.nwg == 0) L.partElems = std::max(L.partElems, (long)step.splits * step.rows * Hp);
  size_t o = 0;
  auto take = [&](size_t bytes) {
    size_t at = o;
    o = align256(o + bytes);
    return at;
  };
  L.Wo_c = take((size_t)Vp * Dp * es);
  L.U_c = take((size_t)Hp * Hp * es);
  L.UT_c = take((size_t)Hp * Hp * es);
  L.Hs_c = take((size_t)(MpMax + Bp + 64) * Hp * es);  // (+ 64: a per-step tile may read past the last stream)
  L.ZT = take((size_t)Vp * MpMax * es);
  L.dA_c = take((size_t)(MpMax + Bp + 64) * Hp * es);
  L.X32 = take((size_t)MpMax * Hp * 4);
  L.dHs32 = take((size_t)MpMax * Hp * 4);
  L.dA32 = take((size_t)MpMax * Hp * 4);
  L.part32 = take((size_t)L.partElems * 4);
  L.stat = take((size_t)statElems * 8);
  L.lse = take((size_t)MpMax * 4);
  L.zy = take((size_t)MpMax * 4);
  L.logp_int = take((size_t)MpMax * 4);
  L.xp = take((size_t)MpMax * 4);
  L.yp = take((size_t)MpMax * 4);
  L.perm = take((size_t)MpMax * 4);
  L.seg = take((size_t)(MpMax + 1) * 4);
  L.xtmp = take((size_t)c.T_max * c.B * 4);
  L.ytmp = take((size_t)c.T_max * c.B * 4);
  KpMax = (int)round_up(c.K_max, 256);
  L.Wn_c = L.Spart = L.dS_c = L.G32 = L.noff = L.ndt = L.nct = L.gcol = L.ids = L.perm2 = L.seg2 = 0;
  if (KpMax > 0) {
    const size_t nent = (size_t)KpMax + (size_t)c.T_max * c.B;
    L.Wn_c = take((size_t)KpMax * Hp * es);
    L.Spart = take((size_t)(MpMax / 32) * KpMax * 2 * 4);  // partial sums of the score blocks: losses, bias gradients
    L.dS_c = take((size_t)MpMax * KpMax * es);
    L.G32 = take((size_t)KpMax * Hp * 4);
    L.noff = take((size_t)KpMax * 4);
    L.ndt = take((size_t)MpMax * 4);
    L.nct = take((size_t)MpMax * 4);
    L.gcol = take((size_t)KpMax * 4);
    L.ids = take(nent * 4);
    L.perm2 = take(nent * 4);
    L.seg2 = take((nent + 1) * 4);
  }
  L.gWo = L.gU = L.gb = 0;
  if (c.rmsprop) {
    L.gWo = take((size_t)c.V * c.H * 4);
    L.gU = take((size_t)c.H * c.H * 4);
    L.gb = take((size_t)c.V * 4);
  }
  L.gN = L.gbN = 0;
  if (c.rmsprop && KpMax > 0) {  // compact per-touched-word gradient rows of the noise-contrastive calls
    const size_t nent = (size_t)KpMax + (size_t)c.T_max * c.B;
    L.gN = take(nent * Hp * 4);
    L.gbN = take(nent * 4);
  }
  L.A_c = L.C_c = L.Xp_c = L.P_c = L.dP_c = L.dX32 = 0;
  if (Pp > 0) {
    L.A_c = take((size_t)Hp * Pp * es);
    L.C_c = take((size_t)Pp * Hp * es);
    L.Xp_c = take((size_t)MpMax * Pp * es);
    L.P_c = take((size_t)MpMax * Pp * es);
    L.dP_c = take((size_t)MpMax * Pp * es);
    L.dX32 = take((size_t)MpMax * Pp * 4);
  }
  L.part_res = 0;
  L.has_part_res = es == 2 && Pp == 0 && Hp == RES_HP && Bp == RES_BP;
  if (L.has_part_res) L.part_res = take((size_t)RES_PART_STEP * 4);
  L.sync = take((size_t)SYNC_WORDS * 4);  // barrier / ticket counters of the persistent recurrent kernels
  L.ring = take(plan.nwg > 0 ? 2 * align256(plan.ring_bytes((int)es)) : 0);  // forward, backward
  L.scalars = take(256);  // [0]: int nseg, [4]: int nseg of the noise-contrastive update list, [8..19]: int flags[3], [32]: double sum, [40]: double running
  L.total = o;
}

const WindowPlan &window_plan(rnnlm_t *h, long Mrows) {
  WindowPlan &p = h->window;
  if (p.Mrows != Mrows) {
    p.Mp = window_rows(h->cfg, Mrows);
    if (h->cfg.precision != RNNLM_FP32) {
      p.sum = bf16_sum_plan(p.Mp, h->D, h->Vp, h->cfg.P > 0);
      p.parts = (int)stat_parts(h->Vp, p.Mp, terms<bf16_t>(h->D));
    } else {
      p.parts = h->Vp / f32_plan(h->Vp, p.Mp, h->D, 1).tile;
    }
    p.Mrows = Mrows;
  }
  return p;
}
// The softmax-gradient pass merges the statistics of a training window itself.
bool merged_in_pass(const rnnlm_t *h, const WindowPlan &p) {
  return p.Mp <= SHORT_POSITIONS && p.parts * p.Mp <= SHORT_STATS && !timed(h, {RNNLM_STAGE_STATS, RNNLM_STAGE_SOFTMAX_GRAD});
}

template <typename P>
P *at(rnnlm_t *h, size_t off) {
  return reinterpret_cast<P *>(h->ws + off);
}
int32_t *p_nseg(rnnlm_t *h) { return at<int32_t>(h, h->L.scalars); }
int32_t *p_nseg2(rnnlm_t *h) { return at<int32_t>(h, h->L.scalars + 4); }
int32_t *p_flags(rnnlm_t *h) { return at<int32_t>(h, h->L.scalars + 8); }
double *p_sum(rnnlm_t *h) { return at<double>(h, h->L.scalars + 32); }
double *p_running(rnnlm_t *h) { return at<double>(h, h->L.scalars + 40); }
unsigned *p_counter(rnnlm_t *h) { return at<unsigned>(h, h->L.sync); }

inline unsigned blocks_for(long n, int per) { return (unsigned)((n + per - 1) / per); }
template <typename T>
int reduce_splits(hipStream_t st, const float *part, long n, int splits, T *out) {
  // One after the other and shared out, us: 262144 values, 16 parts 3.4 and 2.8, 24 parts 4.2 and 3.1, 32 parts 5.7 and 3.6, 64
  // parts 18 and 12; 16384 values, 64 parts 8.1 and 2.8; but 524288 values, 24 parts 8.9 and 13, 64 parts 20 and 32; 2097152
  // values, 24 parts 30 and 31.  Up to 16 parts the two are within half a microsecond.
  if (splits > 16 && n <= 1 << 18)
    hipLaunchKernelGGL(splitk_reduce_many_kernel<T>, dim3(blocks_for(n / 4, 64)), dim3(256), 0, st, part, n, splits, out);
  else
    hipLaunchKernelGGL(splitk_reduce_kernel<T>, dim3(blocks_for(n / 4, 256)), dim3(256), 0, st, part, n, splits, out);
  HIP_TRY(hipGetLastError());
  return RNNLM_OK;
}

template <typename T>
int sync_copies(rnnlm_t *h, hipStream_t st) {
  const rnnlm_config &c = h->cfg;
  const long nWo = (long)h->Vp * h->Dp, nU = (long)h->Hp * h->Hp;
  // the output layer's matrix: Wo, or the tied matrix E of the compressed architecture
  hipLaunchKernelGGL(to_compute_copy_kernel<T>, dim3(std::min<long>(blocks_for(nWo, 256), 65535)), dim3(256), 0, st,
                     c.P > 0 ? h->buf.E : h->buf.Wo, c.V, h->D, h->Dp, nWo, at<T>(h, h->L.Wo_c));
  if (c.P > 0) {
    const long nA = (long)h->Hp * h->Pp;
    hipLaunchKernelGGL(to_compute_copy_kernel<T>, dim3(std::min<long>(blocks_for(nA, 256), 65535)), dim3(256), 0, st,
                       h->buf.A, c.H, c.P, h->Pp, nA, at<T>(h, h->L.A_c));
    hipLaunchKernelGGL(to_compute_copy_kernel<T>, dim3(std::min<long>(blocks_for(nA, 256), 65535)), dim3(256), 0, st,
                       h->buf.C, c.P, c.H, h->Hp, nA, at<T>(h, h->L.C_c));
  }
  hipLaunchKernelGGL(to_compute_copy_kernel<T>, dim3(std::min<long>(blocks_for(nU, 256), 65535)), dim3(256), 0, st,
                     h->buf.U, c.H, c.H, h->Hp, nU, at<T>(h, h->L.U_c));
  hipLaunchKernelGGL(transpose_kernel<T>, dim3(h->Hp / 32, h->Hp / 32), dim3(256), 0, st, at<T>(h, h->L.U_c), h->Hp,
                     at<T>(h, h->L.UT_c));
  HIP_TRY(hipGetLastError());
  return RNNLM_OK;
}

bool persistent_ok(const rnnlm_t *h) { return h->plan.nwg > 0; }

// Workgroups of a kernel that one compute unit holds at once, as the runtime computes it (asked once).
template <auto Kern>
int blocks_per_cu(int threads) {
  static int n = -1;
  if (n < 0) {
    int v = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&v, Kern, threads, 0) != hipSuccess) v = 0;
    n = v;
  }
  return n;
}

template <typename T, bool BACKWARD>
int launch_rnn_persistent(rnnlm_t *h, int Tn, bool advance_state, hipStream_t st) {
  RnnPersistArgs a;
  a.W = BACKWARD ? at<T>(h, h->L.UT_c) : at<T>(h, h->L.U_c);
  a.Hs = at<T>(h, h->L.Hs_c);
  a.X = BACKWARD ? at<float>(h, h->L.dHs32) : at<float>(h, h->L.X32);
  a.dA32 = at<float>(h, h->L.dA32);
  a.dAc = at<T>(h, h->L.dA_c);
  a.h_state = (!BACKWARD && advance_state) ? h->buf.h_state : nullptr;
  a.counter = p_counter(h);
  a.flags = p_flags(h);
  a.T = Tn;
  a.B = h->cfg.B;
  a.H = h->cfg.H;
  a.Bp = h->Bp;
  a.Hp = h->Hp;
  // This kernel's poll is one reload of a wave's fragments (0.21 us at H = 2048, 256 streams), a counter's 4 us: 20 for
  // one, or a workgroup that other work on the device keeps from starting is given up after 0.06 s instead of a second.
  // (Spacing the polls out inside the kernel cost 2 % of a scored sentence.)
  a.spin_limit = h->spin_limit == 1 ? 1u : (unsigned)std::min<unsigned long>(h->spin_limit * 20ul, 0xffffffffu);
  const RecurrentPlan &p = h->plan;
  a.ring = h->ws + h->L.ring + (BACKWARD ? align256(p.ring_bytes(sizeof(T))) : 0);
  a.R = p.R;
  a.groups = p.groups;
  a.nwg = p.nwg;
  a.nkb = p.nkb;
  a.ks = p.ks;
  // the counters are zero here: cleared by the token-preparation kernel (forward) and by the
  // log-probability sum (backward), which always run before this launch on the same stream
  a.xcd = h->xcd_local && h->exchange_mode != RNNLM_EXCHANGE_CHIP_WIDE && p.groups <= NUM_XCD;
  const dim3 grid((unsigned)((a.xcd ? NUM_XCD : p.groups) * p.nwg));
#define RNNLM_LAUNCH_PERSIST(KS, NW, UT)                                                                              \
  do {                                                                                                                \
    if (p.R <= 16) hipLaunchKernelGGL((rnn_persistent_kernel<T, KS, NW, UT, 1, BACKWARD>), grid, dim3(64 * NW), 0, st, a); \
    else hipLaunchKernelGGL((rnn_persistent_kernel<T, KS, NW, UT, 2, BACKWARD>), grid, dim3(64 * NW), 0, st, a);      \
  } while (0)
  if (p.waves == 4) {
    if (p.ks <= 1) RNNLM_LAUNCH_PERSIST(1, 4, 2);
    else if (p.ks <= 2) RNNLM_LAUNCH_PERSIST(2, 4, 2);
    else if (p.ks <= 3) RNNLM_LAUNCH_PERSIST(3, 4, 2);
    else if (p.ks <= 4) RNNLM_LAUNCH_PERSIST(4, 4, 2);
    else if (p.ks <= 6) RNNLM_LAUNCH_PERSIST(6, 4, 2);
    else if (p.ks <= 8) RNNLM_LAUNCH_PERSIST(8, 4, 2);
    else return RNNLM_ERR_ARG;
  } else if constexpr (sizeof(T) == 2) {
    if (p.ks <= 6) RNNLM_LAUNCH_PERSIST(6, 8, 4);
    else if (p.ks <= 8) RNNLM_LAUNCH_PERSIST(8, 8, 4);
    else return RNNLM_ERR_ARG;
  } else {
    return RNNLM_ERR_ARG;
  }
#undef RNNLM_LAUNCH_PERSIST
  HIP_TRY(hipGetLastError());
  return RNNLM_OK;
}

// Widest layer (Hp = 4096, 256 streams, bf16): one launch of 256 workgroups, one per compute unit, with the whole
// state-to-state matrix resident in registers.  Needs the round-robin placement the init probe checks (32
// workgroups on every XCD); RNNLM_EXCHANGE_CHIP_WIDE selects the per-step launches instead.
bool resident_ok(const rnnlm_t *h) {
  return h->L.has_part_res && h->xcd_local && h->exchange_mode != RNNLM_EXCHANGE_CHIP_WIDE &&
         blocks_per_cu<rnn_resident_kernel<false>>(512) >= 1 && blocks_per_cu<rnn_resident_kernel<true>>(512) >= 1;
}

template <bool BACKWARD>
int launch_rnn_resident(rnnlm_t *h, int Tn, bool advance_state, hipStream_t st) {
  typedef bf16_t T;
  RnnResidentArgs ra;
  RnnPersistArgs &a = ra.p;
  a.W = BACKWARD ? at<T>(h, h->L.UT_c) : at<T>(h, h->L.U_c);
  a.Hs = at<T>(h, h->L.Hs_c);
  a.X = BACKWARD ? at<float>(h, h->L.dHs32) : at<float>(h, h->L.X32);
  a.dA32 = at<float>(h, h->L.dA32);
  a.dAc = at<T>(h, h->L.dA_c);
  a.h_state = (!BACKWARD && advance_state) ? h->buf.h_state : nullptr;
  a.counter = p_counter(h);  // zero here, as for the other persistent kernels
  a.flags = p_flags(h);
  a.T = Tn;
  a.B = h->cfg.B;
  a.H = h->cfg.H;
  a.Bp = h->Bp;
  a.Hp = h->Hp;
  a.spin_limit = h->spin_limit;
  ra.part = at<float>(h, h->L.part_res);
  hipLaunchKernelGGL((rnn_resident_kernel<BACKWARD>), dim3(256), dim3(512), 0, st, ra);
  HIP_TRY(hipGetLastError());
  return RNNLM_OK;
}

// One step in one launch (rnn_step.h): where its workgroups, with up to 64 streams each, are at most one per compute unit.
// Blocks of 16 streams a workgroup takes: as few as that allows (more streams read the matrix less often, fewer load faster).
// us a window of 16 positions, V = 2000, two launches a step and one: bf16 H = 2816, 1 stream 434 and 248, 16 530 and 326, 64
// 618 and 467; H = 4000, 16 streams 648 and 446, 64 741 and 607; fp32 H = 1300, 16 streams 417 and 241, 128 866 and 678; H =
// 2816, 16 streams 793 and 421, 64 1020 and 909.  Beyond: bf16 H = 4000, 128 streams 898 and 933, fp32 H = 2816, 1536 and 1645.
int step_groups(const rnnlm_config &c, int blocks) { return (int)((c.H + 15) / 16 * ((c.B + 16L * blocks - 1) / (16 * blocks))); }
bool step_in_one(const rnnlm_config &c) { return c.H <= 4096 && c.B <= 4096 && step_groups(c, 4) <= 256; }
int step_blocks(const rnnlm_config &c) { return c.B <= 16 ? 1 : step_groups(c, 2) <= 256 ? 2 : 4; }
template <typename T, int MODE>
void launch_step_kernel(const RnnStepArgs &a, int rt, hipStream_t st) {
  hipLaunchKernelGGL((rt == 1   ? rnn_step_kernel<T, 1, MODE>
                      : rt == 2 ? rnn_step_kernel<T, 2, MODE>
                                : rnn_step_kernel<T, 4, MODE>),
                     dim3(blocks_for(MODE == STEP_STORE || MODE == STEP_STORE32 ? a.Hp : a.H, 16), blocks_for(a.B, 16 * rt)),
                     dim3(512), 0, st, a);
}
// out = rows . W^T for a few rows (row lengths ldo and ldk; `units` columns of out and zeros up to ldo, `terms_` values of a row).
constexpr int FEW_ROWS = 64;
template <int MODE>
int few_rows(const bf16_t *rows, const bf16_t *W, long ldk, long terms_, void *out, long ldo, int n, int units, hipStream_t st) {
  RnnStepArgs a = {};
  a.W = W;
  a.state = rows;
  a.out = out;
  a.out32 = static_cast<float *>(out);
  a.B = n;
  a.H = units;
  a.Hp = (int)ldo;
  a.lds = (int)ldk;
  a.pieces = (int)(terms_ * 2 / 128);
  launch_step_kernel<bf16_t, MODE>(a, n <= 16 ? 1 : n <= 32 ? 2 : 4, st);
  HIP_TRY(hipGetLastError());
  return RNNLM_OK;
}
template <typename T, bool BACKWARD>
int launch_rnn_step(rnnlm_t *h, int t, bool contract, float *h_state, hipStream_t st) {
  const rnnlm_config &c = h->cfg;
  const long slot = (long)h->Bp * h->Hp;
  T *Hs = at<T>(h, h->L.Hs_c) + (t + 1) * slot, *dA = at<T>(h, h->L.dA_c) + t * slot;
  RnnStepArgs a;
  a.W = BACKWARD ? at<T>(h, h->L.UT_c) : at<T>(h, h->L.U_c);
  a.state = BACKWARD ? dA + slot : Hs - slot;
  a.X = (BACKWARD ? at<float>(h, h->L.dHs32) : at<float>(h, h->L.X32)) + t * slot;
  a.h = Hs;
  a.out = BACKWARD ? dA : Hs;
  a.out32 = at<float>(h, h->L.dA32) + t * slot;
  a.h_state = h_state;
  a.B = c.B;
  a.H = c.H;
  a.Hp = a.lds = h->Hp;
  a.pieces = contract ? (int)(terms<T>(c.H) * (long)sizeof(T) / 128) : 0;
  launch_step_kernel<T, BACKWARD ? STEP_BACKWARD : STEP_FORWARD>(a, step_blocks(c), st);
  HIP_TRY(hipGetLastError());
  return RNNLM_OK;
}

struct UpdateTargets {
  // where each fused update writes: training -> the masters (alpha 1, lr), gradient export -> caller
  // buffers (alpha 0, lr -1, no compute-copy refresh, no state advance)
  float *E, *U, *Wo, *b;
  float alpha, lr;
  bool refresh_copies;
  bool advance_state;
  int e_compact_ld = 0;  // > 0: the embedding rows go to a compact [runs][e_compact_ld] buffer (one row per run)
  int wo_compact_ld = 0; // > 0: likewise the touched rows of Wo and entries of b of the noise-contrastive calls
  // compressed architecture: Wo is unused, E is the tied matrix (output-side update first, then the input rows)
  float *A = nullptr, *C = nullptr;
};

// Forward half of a window: tokens -> padded ids, state -> slot 0, gather, T recurrent steps,
// output layer with fused statistics, log-probabilities.
// Fork: work enqueued on the side stream after this call starts once everything enqueued on `st` so far has
// finished.  Join: `st` waits for everything enqueued on the side stream so far.  slot = which event pair.
int side_fork(rnnlm_t *h, int slot, hipStream_t st) {
  HIP_TRY(hipEventRecord(h->ev_fork[slot], st));
  HIP_TRY(hipStreamWaitEvent(h->side, h->ev_fork[slot], 0));
  return RNNLM_OK;
}
int side_join(rnnlm_t *h, int slot, hipStream_t st) {
  HIP_TRY(hipEventRecord(h->ev_join[slot], h->side));
  HIP_TRY(hipStreamWaitEvent(st, h->ev_join[slot], 0));
  return RNNLM_OK;
}

template <typename T>
int sort_segments(rnnlm_t *h, int Tn, int32_t *perm, int32_t *seg, int32_t *nseg, hipStream_t st);

// Does the embedding update find the positions of each word by itself (no sorted list)?  Not where the list names the
// rows of a compact buffer, nor in windows its workgroups cannot compare in one go.  Beyond 1024 positions the plain
// architecture sorts: its embedding update runs next to the output weight update, which every workgroup's comparisons
// slow down; in the compressed one the update stands alone and the sort delays the recurrent steps.  Compared and sorted,
// bf16: V = 10000, H = 256, 512 positions 132 and 139 us, 1024 155 and 153, 2560 220 and 223; V = 3000, H = 64, 512
// positions 128 and 132, 1024 154 and 148, 2560 216 and 189; V = 64000, H = 1024, 512 positions 470 and 473, 1024 631 and
// 628, 2560 1221 and 1210; compressed, V = 10000, H = 1024, P = 512, 512 positions 214 and 217, 2560 353 and 359, 4000 467
// and 483.
bool scan_ids(const rnnlm_t *h, int Tn, const UpdateTargets &u) {
  return u.e_compact_ld == 0 && (long)Tn * h->cfg.B <= (h->cfg.P > 0 ? SCAN_MAX : 1024);
}

// (Plain windows whose updates share a launch, update.h, need no second stream.)
// Where the output weight update is over before a second stream is tied in and out (four events: 20-30 us of host time
// and of latency between the streams), the small updates stay on the caller's stream.  With and without the second
// stream: fp32 V = 1000, H = 64, 4x8 92 and 67 us; bf16 V = 3000, H = 256, 16x8 111 and 106, 32x30 164 and 170.  Beyond the
// line fp32 still gains (V = 10000, H = 256, 32x10 165 and 146; V = 10000, H = 512, 32x30 476 and 469; V = 20000, H = 1024,
// 32x30 1269 and 1273), bf16 below some 500 positions (V = 30000, H = 256, 16x8 148 and 140; 32x30 227 and 231).
bool short_output_update(rnnlm_t *h, int Tn) {
  const double n = (double)h->Vp * h->Dp, rate = h->cfg.precision == RNNLM_FP32 ? 1e8 : 6e8;  // per us
  return 2.0 * n * window_plan(h, (long)Tn * h->Bp).Mp / rate + 8.0 * n / 4e6 < 15.0;
}

// train: a backward pass follows.  sort_inputs: its embedding update wants the input ids sorted: started on the side
// stream as soon as the padded ids exist (the update runs on that stream too).
template <typename T>
int forward_window(rnnlm_t *h, const int32_t *x, const int32_t *y, int Tn, float *logp_out, bool advance_state,
                   bool with_output, hipStream_t st, bool train = false, bool sort_inputs = false, bool need_feat = false,
                   const WindowSum *wsum = nullptr) {
  const rnnlm_config &c = h->cfg;
  const int Hp = h->Hp, Bp = h->Bp, Vp = h->Vp;
  const int Mrows = Tn * Bp;
  const int Mp = (int)window_plan(h, Mrows).Mp;
  const long ldz = h->MpMax;
  T *Hs_c = at<T>(h, h->L.Hs_c);
  float *X32 = at<float>(h, h->L.X32);
  int32_t *xp = at<int32_t>(h, h->L.xp), *yp = at<int32_t>(h, h->L.yp);
  float *lse = at<float>(h, h->L.lse), *zy = at<float>(h, h->L.zy);

  {
    StageTimer tm(h, RNNLM_STAGE_PREP, st);
    const long ring16 = persistent_ok(h) ? h->plan.ring_bytes(sizeof(T)) / 16 : 0;
    const int prep_blocks = (int)blocks_for(std::max({(long)Mp, (long)Bp * Hp, ring16, (long)SYNC_WORDS}), 256);
    PrepWindow<T> pw = {};
    pw.x = x;
    pw.y = y;
    pw.Tn = Tn;
    pw.B = c.B;
    pw.Bp = Bp;
    pw.Mp = Mp;
    pw.V = c.V;
    pw.xp = xp;
    pw.yp = yp;
    pw.lse = lse;
    pw.flags = p_flags(h);
    pw.h_state = h->buf.h_state;
    pw.H = c.H;
    pw.Hp = Hp;
    pw.slot = Hs_c;
    pw.counters = p_counter(h);
    pw.prep_blocks = prep_blocks;
    if (c.P > 0) {  // compressed architecture: the gathered rows are operands of the contraction below
      pw.Ec = at<T>(h, h->L.Wo_c);
      pw.ldc = h->Pp;
      pw.Xc = at<T>(h, h->L.Xp_c);
    } else {
      pw.E = h->buf.E;
      pw.X = X32;
    }
    int rows = Mrows;
    if (persistent_ok(h)) {
      pw.plan = h->plan;
      pw.next = Hs_c + (long)Bp * Hp;
      pw.ring[0] = h->ws + h->L.ring;
      if (train) {
        pw.ring[1] = pw.ring[0] + align256(h->plan.ring_bytes(sizeof(T)));
        pw.dA = at<T>(h, h->L.dA_c);
        rows = Mp;  // rows [Mrows, Mp) of dA take part in the dU contraction: zero
      }
    }
    hipLaunchKernelGGL(prep_tokens_kernel<T>, dim3(prep_blocks + rows), dim3(256), 0, st, pw);
    HIP_TRY(hipGetLastError());
    if (sort_inputs) {
      int rc = side_fork(h, 0, st);
      if (rc) return rc;
      rc = sort_segments<T>(h, Tn, at<int32_t>(h, h->L.perm), at<int32_t>(h, h->L.seg), p_nseg(h), h->side);
      if (rc) return rc;
    }
  }

  // (training windows contract over the padded rows of what the layers give as well; fp32 keeps its split operands, which
  // round less than the fp32 cores)
  const bool few = sizeof(T) == 2 && !train && Mrows <= FEW_ROWS;
  if (c.P > 0) {
    // layer below the state: X[m][i] = sum_p x_m[p] A[i][p], the additive input of every recurrent step
    StageTimer tm(h, RNNLM_STAGE_PROJ, st);
    if (few) {
      int rc = few_rows<STEP_STORE32>(at<bf16_t>(h, h->L.Xp_c), at<bf16_t>(h, h->L.A_c), h->Pp, terms<bf16_t>(c.P), X32, Hp, Mrows,
                                      c.H, st);
      if (rc) return rc;
    } else {
      EpiPartial epi;
      epi.part = X32;
      epi.ld = Hp;
      epi.split_stride = 0;
      HIP_TRY((mid_gemm<T, ROWK, ROWK>(st, at<T>(h, h->L.Xp_c), h->Pp, at<T>(h, h->L.A_c), h->Pp, Mp, Hp, terms<T>(c.P), 1,
                                        epi)));
    }
  }

  if (persistent_ok(h)) {
    StageTimer tm(h, RNNLM_STAGE_RNN_FWD, st);
    int rc = launch_rnn_persistent<T, false>(h, Tn, advance_state, st);
    if (rc) return rc;
  } else if (sizeof(T) == 2 && resident_ok(h)) {
    StageTimer tm(h, RNNLM_STAGE_RNN_FWD, st);
    int rc = launch_rnn_resident<false>(h, Tn, advance_state, st);
    if (rc) return rc;
  } else
  for (int t = 0; t < Tn; ++t) {
    StageTimer tm(h, (t == 0 || t == Tn - 1) ? RNNLM_STAGE_RNN_FWD : -1, st, t == 0, t == Tn - 1);
    float *const h_state = (advance_state && t == Tn - 1) ? h->buf.h_state : nullptr;
    if (step_in_one(c)) {
      int rc = launch_rnn_step<T, false>(h, t, true, h_state, st);
      if (rc) return rc;
      continue;
    }
    const T *A_ = Hs_c + (long)t * Bp * Hp;
    const T *B_ = at<T>(h, h->L.U_c);
    const StepPlan p = step_plan(c, Bp, Hp);
    const long per = (long)Bp * Hp, K = terms<T>(c.H);
    EpiPartial ep;
    ep.part = at<float>(h, h->L.part32);
    ep.ld = Hp;
    ep.split_stride = p.rows * Hp;
    if (!p.wide) {
      HIP_TRY((launch_gemm_dma4<T, 64, 64, 2, 2, ROWK, ROWK>(st, A_, Hp, B_, Hp, p.rows, Hp, K, p.splits, ep)));
    } else if constexpr (sizeof(T) == 2) {
      HIP_TRY((launch_gemm_dma<256, 128, 4, 2, ROWK, ROWK>(st, A_, Hp, B_, Hp, Bp, Hp, K, p.splits, ep)));
    } else {
      HIP_TRY((launch_gemm<T, 256, 64, 4, 2, ROWK, ROWK>(st, A_, Hp, B_, Hp, Bp, Hp, K, p.splits, ep)));
    }
    hipLaunchKernelGGL(rnn_step_fwd_kernel<T>, dim3(blocks_for(per / 4, 256)), dim3(256), 0, st,
                       at<float>(h, h->L.part32), p.rows * Hp, p.splits, X32 + (long)t * Bp * Hp, c.B, c.H, Hp, per / 4,
                       Hs_c + (long)(t + 1) * Bp * Hp, h_state);
    HIP_TRY(hipGetLastError());
  }
  if (!with_output && !(need_feat && c.P > 0)) return RNNLM_OK;  // the noise-contrastive calls score the hidden states themselves
  const T *feat = Hs_c + (long)Bp * Hp;  // what the output layer reads: the states, or the layer above them
  if (c.P > 0) {
    StageTimer tm(h, RNNLM_STAGE_PROJ, st);
    if (few) {
      int rc = few_rows<STEP_STORE>(at<bf16_t>(h, h->L.Hs_c) + (long)Bp * Hp, at<bf16_t>(h, h->L.C_c), Hp, terms<bf16_t>(c.H),
                                    at<bf16_t>(h, h->L.P_c), h->Pp, Mrows, c.P, st);
      if (rc) return rc;
    } else {
      EpiStore<T> epi;
      epi.outc = at<T>(h, h->L.P_c);
      epi.ld = h->Pp;
      HIP_TRY((mid_gemm<T, ROWK, ROWK>(st, Hs_c + (long)Bp * Hp, Hp, at<T>(h, h->L.C_c), Hp, Mp, h->Pp, terms<T>(c.H), 1, epi)));
    }
    feat = at<T>(h, h->L.P_c);
  }
  if (!with_output) return RNNLM_OK;  // the scoring calls only wanted the layer above the states
  {
    StageTimer tm(h, RNNLM_STAGE_OUT_FWD, st);
    EpiOutFwd<T> epi;
    epi.b = h->buf.b;
    epi.ZT = train ? at<T>(h, h->L.ZT) : nullptr;  // evaluation wants the statistics only
    epi.part = at<float2>(h, h->L.stat);
    epi.yp = yp;
    epi.zy = zy;
    epi.V = c.V;
    epi.ldz = ldz;
    epi.ldp = Mp;
    if constexpr (sizeof(T) == 2) {
      const int tile = bf16_tile(OUT_FWD, Vp, Mp, terms<T>(h->D));
      const long rows = large_rows(Vp, Mp, terms<T>(h->D));
      // thousands of short tiles: one persistent workgroup per compute unit walks them, in bands of 8 vocabulary
      // row panels (the 32 tiles an XCD works on at a time then share 8 row panels and 4 position panels in its L2:
      // measured best of 1..16 on all three large configurations)
      if (tile == BIG && rows == Vp) {
        HIP_TRY((launch_gemm_dma<BIG, BIG, 4, 2, ROWK, ROWK, true>(st, at<T>(h, h->L.Wo_c), h->Dp, feat, h->Dp, Vp, Mp,
                                                                   terms<T>(h->D), 1, epi, 8)));
      } else if (tile == BIG) {
        EpiOutFwd<T> tail = epi;
        tail.b += rows;
        if (tail.ZT) tail.ZT += rows * ldz;
        tail.part += rows / BIG * epi.ldp;
        tail.V -= (int)rows;
        tail.v0 = (int)rows;
        HIP_TRY((launch_gemm_tail<4, 2, ROWK>(st, at<T>(h, h->L.Wo_c), h->Dp, feat, h->Dp, Vp, Mp, terms<T>(h->D), rows, epi,
                                              tail, 8)));
      } else {
        HIP_TRY((bf16_small_gemm<ROWK, ROWK>(st, at<T>(h, h->L.Wo_c), h->Dp, feat, h->Dp, Vp, Mp, terms<T>(h->D), tile, 1,
                                             epi, 8)));
      }
    } else {
      const F32Plan plan = f32_plan(Vp, Mp, h->D, 1);
      HIP_TRY((f32_gemm<ROWK, ROWK>(st, at<T>(h, h->L.Wo_c), h->Dp, feat, h->Dp, Vp, Mp, round_up(h->D, 32), plan, epi, 8)));
    }
  }
  if (train && merged_in_pass(h, window_plan(h, Mrows))) return RNNLM_OK;
  StageTimer tm(h, RNNLM_STAGE_STATS, st);
  hipLaunchKernelGGL(merge_stats_kernel, dim3(blocks_for(Mrows, MERGE_M)), dim3(1024), 0, st, at<float2>(h, h->L.stat),
                     window_plan(h, Mrows).parts, Mp, Tn, c.B, Bp, zy, lse, at<float>(h, h->L.logp_int), logp_out,
                     wsum ? p_counter(h) + sync_word(0, 0) : nullptr, wsum ? *wsum : WindowSum{});
  HIP_TRY(hipGetLastError());
  return RNNLM_OK;
}

template <typename T>
int sort_segments(rnnlm_t *h, int Tn, int32_t *perm, int32_t *seg, int32_t *nseg, hipStream_t st) {
  const int M = Tn * h->cfg.B;
  hipLaunchKernelGGL(rank_sort_kernel, dim3(blocks_for(M, 64)), dim3(1024), 0, st, at<int32_t>(h, h->L.xp), M,
                     h->cfg.B, h->Bp, perm);
  hipLaunchKernelGGL(segment_kernel, dim3(1), dim3(1024), 0, st, at<int32_t>(h, h->L.xp), perm, M, h->cfg.B, h->Bp,
                     seg, nseg);
  HIP_TRY(hipGetLastError());
  return RNNLM_OK;
}

// One call of the noise-contrastive criterion (Sec. 4.2): K noise words shared by the window.
struct NceCall {
  const int32_t *noise;
  int K;
  const float *lnq;
  float lnZ;
  float *J_out;
  bool sort_ids;  // the call updates (or exports) rows: sort the touched-word list
};

// Scores of all positions against the gathered noise rows and the targets' own scores: coefficients dS (contraction
// operand), target coefficients, losses, bias column sums.
template <typename T>
int nce_forward(rnnlm_t *h, int Tn, const NceCall &n, const WindowSum *wsum, hipStream_t st) {
  const rnnlm_config &c = h->cfg;
  const int Hp = h->Hp, Bp = h->Bp;
  const int Mrows = Tn * Bp, Mp = (int)window_plan(h, Mrows).Mp, M = Tn * c.B;
  const int K = n.K, Kp = (int)round_up(K, 256);
  T *Hs1 = at<T>(h, h->L.Hs_c) + (long)Bp * Hp;
  T *Wn = at<T>(h, h->L.Wn_c);
  float *jpart = at<float>(h, h->L.Spart), *gpart = jpart + (long)(Kp / 32) * Mp;
  int32_t *yp = at<int32_t>(h, h->L.yp);
  const float lnZ_lnK = n.lnZ + logf((float)K);
  const float scale = 1.0f / (float)M;
  {
    StageTimer tm(h, RNNLM_STAGE_NCE_SCORE, st);
    hipLaunchKernelGGL(nce_prep_kernel<T>, dim3(Kp + blocks_for(M, 256) + blocks_for(Mrows, 4)), dim3(256), 0, st, n.noise, K, Kp, c.V, n.lnq,
                       h->buf.b, lnZ_lnK, yp, M, c.B, Bp, at<T>(h, h->L.Wo_c), Hp, Wn, at<float>(h, h->L.noff),
                       at<int32_t>(h, h->L.ids), p_flags(h), Hs1, Mrows, at<float>(h, h->L.ndt));
    if (n.sort_ids) {  // the touched-word list is complete: sort it next to the contractions
      int rc = side_fork(h, 1, st);
      if (rc) return rc;
      const int nent = K + M;
      int32_t *ids = at<int32_t>(h, h->L.ids);
      // the sort helpers index keys as key[(i / B) * Bp + i % B]: B = Bp = 1 reads the compact list
      hipLaunchKernelGGL(rank_sort_kernel, dim3(blocks_for(nent, 64)), dim3(1024), 0, h->side, ids, nent, 1, 1,
                         at<int32_t>(h, h->L.perm2));
      hipLaunchKernelGGL(segment_kernel, dim3(1), dim3(1024), 0, h->side, ids, at<int32_t>(h, h->L.perm2), nent, 1, 1,
                         at<int32_t>(h, h->L.seg2), p_nseg2(h));
      HIP_TRY(hipEventRecord(h->ev_join[1], h->side));  // here, not where it is waited for: more work follows on that stream
    }
    HIP_TRY(hipGetLastError());
    EpiNce<T> epi;
    epi.dS = at<T>(h, h->L.dS_c);
    epi.ld = Kp;
    epi.off = at<float>(h, h->L.noff);
    epi.yp = yp;
    epi.scale = scale;
    epi.K = K;
    epi.Mp = Mp;
    epi.jpart = jpart;
    epi.gpart = gpart;
    HIP_TRY((mid_gemm<T, ROWK, ROWK>(st, Hs1, Hp, Wn, Hp, Mp, Kp, terms<T>(c.H), 1, epi)));
  }
  StageTimer tm(h, RNNLM_STAGE_NCE_GRAD, st);
  const int rowBlocks = (int)blocks_for(Mrows, 64);
  hipLaunchKernelGGL(nce_merge_kernel, dim3(rowBlocks + Kp / 64), dim3(1024), 0, st, jpart, gpart, Kp, Mp, rowBlocks,
                     at<float>(h, h->L.ndt), yp, Mrows, c.B, Bp, scale, at<float>(h, h->L.nct), at<float>(h, h->L.logp_int),
                     n.J_out, at<float>(h, h->L.gcol), wsum ? p_counter(h) + sync_word(0, 0) : nullptr, wsum ? *wsum : WindowSum{}, M);
  HIP_TRY(hipGetLastError());
  return RNNLM_OK;
}

// dHs = dS . Wn + ct * Wo[target]  (what the output layer sends back to the hidden states)
template <typename T>
int nce_backward_h(rnnlm_t *h, int Tn, const NceCall &n, hipStream_t st) {
  const int Hp = h->Hp, Bp = h->Bp;
  const int Mrows = Tn * Bp, Mp = (int)window_plan(h, Mrows).Mp;
  const int Kp = (int)round_up(n.K, 256);
  float *dHs32 = at<float>(h, h->L.dHs32);
  StageTimer tm(h, RNNLM_STAGE_NCE_BWD_H, st);
  EpiNceDhs<T> epi;
  epi.part = dHs32;
  epi.ld = Hp;
  epi.split_stride = 0;
  epi.Wo_c = at<T>(h, h->L.Wo_c);
  epi.yp = at<int32_t>(h, h->L.yp);
  epi.ct = at<float>(h, h->L.nct);
  HIP_TRY((mid_gemm<T, ROWK, KROW>(st, at<T>(h, h->L.dS_c), Kp, at<T>(h, h->L.Wn_c), Hp, Mp, Hp, terms<T>(n.K),
                                      1, epi)));
  return RNNLM_OK;
}

// Gradient rows of the noise words (G = dS^T . Hs), then the order-fixed update of every touched row of
// Wo and entry of b (noise words and targets together).
template <typename T>
int nce_update(rnnlm_t *h, int Tn, const NceCall &n, const UpdateTargets &u, hipStream_t st) {
  const rnnlm_config &c = h->cfg;
  const int Hp = h->Hp, Bp = h->Bp;
  const int Mrows = Tn * Bp, M = Tn * c.B;
  const int K = n.K, Kp = (int)round_up(K, 256);
  T *Hs1 = at<T>(h, h->L.Hs_c) + (long)Bp * Hp;
  float *G = at<float>(h, h->L.G32);
  {
    StageTimer tm(h, RNNLM_STAGE_NCE_BWD_W, st);
    const long per = (long)Kp * Hp;
    constexpr int BK = Elem<T>::BK;
    long S = 256 / ((long)(Kp / 128) * (Hp / 128));  // aim at one round of workgroups
    const long terms_ = terms<T>(Mrows);
    S = std::min<long>(std::min<long>(S, 8), std::min<long>(terms_ / BK, h->L.partElems / per));
    if (S < 1) S = 1;
    EpiPartial epi;
    epi.part = (S == 1) ? G : at<float>(h, h->L.part32);
    epi.ld = Hp;
    epi.split_stride = per;
    HIP_TRY((mid_gemm<T, KROW, KROW>(st, at<T>(h, h->L.dS_c), Kp, Hs1, Hp, Kp, Hp, terms_, (int)S, epi)));
    if (S > 1) {
      int rc = reduce_splits(st, at<float>(h, h->L.part32), per, (int)S, G);
      if (rc) return rc;
    }
  }
  StageTimer tm(h, RNNLM_STAGE_NCE_UPDATE, st);
  const int nent = K + M;
  int32_t *ids = at<int32_t>(h, h->L.ids), *perm = at<int32_t>(h, h->L.perm2), *seg = at<int32_t>(h, h->L.seg2);
  HIP_TRY(hipStreamWaitEvent(st, h->ev_join[1], 0));  // the sort of the list, started on the side stream by nce_forward
  T *Wc = u.refresh_copies ? at<T>(h, h->L.Wo_c) : nullptr;
  hipLaunchKernelGGL((c.H % 4 == 0 ? nce_row_update_kernel<true, T> : nce_row_update_kernel<false, T>),
                     dim3(blocks_for(nent, RUN_WAVES), blocks_for(c.H, RUN_COLS)), dim3(64 * RUN_WAVES), 0, st, G, Hs1, Hp, c.H,
                     K, c.B, Bp, at<float>(h, h->L.nct), ids, perm, seg, p_nseg2(h), h->buf.Wo, u.Wo, Wc,
                     at<float>(h, h->L.gcol), h->buf.b, u.b, u.alpha, u.lr, u.wo_compact_ld);
  HIP_TRY(hipGetLastError());
  return RNNLM_OK;
}

// Fills in the contractions of a window's updates in one launch; the tile, or 0 where they take launches of their own: where
// the output update's tiles are large, or an operand is beyond the loads' offsets.
template <typename T>
int window_update_shape(rnnlm_t *h, int Mrows, const T *ZT, const T *Hs_c, const T *dA_c, WindowUpdate<T> &w) {
  const rnnlm_config &c = h->cfg;
  const int Hp = h->Hp, Vp = h->Vp;
  const long ldz = h->MpMax, K = terms<T>(Mrows);
  const T *Hs1 = Hs_c + (long)h->Bp * Hp;
  int tile;
  hipError_t e = hipErrorInvalidValue;
  if constexpr (sizeof(T) == 4) {
    const long Dn = f32_extent(c.H, Vp, Mrows, 1), Hn = round_up(c.H, 64);
    tile = f32_plan(Vp, Dn, Mrows, 1).tile;
    if (tile == 64 && Mrows <= F32_SHORT) {
      e = dma4_shape<T, 64, 64, ROWK, KROW>(w.out_g, ZT, ldz, Hs1, Hp, Vp, Dn, K, 1, -4);
      if (e == hipSuccess) e = dma4_shape<T, 64, 64, KROW, KROW>(w.rec_g, Hs_c, Hp, dA_c, Hp, Hn, Hn, K, 1, 4);
    } else if (tile == 64) {
      e = split_shape<64, 64, ROWK, KROW, 1>(w.out_g, ZT, ldz, Hs1, Hp, Vp, Dn, K, 1, -4);
      if (e == hipSuccess) e = split_shape<64, 64, KROW, KROW, 1>(w.rec_g, Hs_c, Hp, dA_c, Hp, Hn, Hn, K, 1, 4);
    }
  } else {
    const long Dn = bf16_extent(OUT_UPDATE, c.H, Vp, K), Hn = round_up(c.H, 128);
    tile = bf16_tile(OUT_UPDATE, Vp, Dn, K);
    if (tile == 64) {
      e = dma4_shape<T, 64, 64, ROWK, KROW>(w.out_g, ZT, ldz, Hs1, Hp, Vp, Dn, K, 1, -4);
      if (e == hipSuccess) e = dma4_shape<T, 64, 64, KROW, KROW>(w.rec_g, Hs_c, Hp, dA_c, Hp, round_up(c.H, 64), round_up(c.H, 64), K, 1, 4);
    } else if (tile == 128) {
      e = dma4_shape<T, 128, 128, ROWK, KROW>(w.out_g, ZT, ldz, Hs1, Hp, Vp, Dn, K, 1, -4);
      if (e == hipSuccess) e = dma4_shape<T, 128, 128, KROW, KROW>(w.rec_g, Hs_c, Hp, dA_c, Hp, Hn, Hn, K, 1, 4);
    }
  }
  return e == hipSuccess ? tile : 0;
}
template <typename T>
int launch_window_update(rnnlm_t *h, WindowUpdate<T> &w, int tile, int Mrows, hipStream_t st) {
  const int W = h->D;
  const bool aligned = W % 4 == 0;
  auto launch = [&](int rec, int out, int scan) -> int {  // workgroups of each update
    w.nRec = rec;
    w.nOut = out;
    const dim3 grid(rec + out + scan), threads(tile * 4);
    if constexpr (sizeof(T) == 4) {
      if (Mrows <= F32_SHORT)
        hipLaunchKernelGGL((aligned ? window_update_kernel<T, 64, 0, true> : window_update_kernel<T, 64, 0, false>), grid, threads, 0, st, w);
      else
        hipLaunchKernelGGL((aligned ? window_update_kernel<T, 64, 1, true> : window_update_kernel<T, 64, 1, false>), grid, threads, 0, st, w);
    } else if (tile == 64) {
      hipLaunchKernelGGL((aligned ? window_update_kernel<T, 64, 0, true> : window_update_kernel<T, 64, 0, false>), grid, threads, 0, st, w);
    } else {
      hipLaunchKernelGGL((aligned ? window_update_kernel<T, 128, 0, true> : window_update_kernel<T, 128, 0, false>), grid, threads, 0, st, w);
    }
    HIP_TRY(hipGetLastError());
    return RNNLM_OK;
  };
  const int rec = w.rec_g.perXcd * NUM_XCD, out = w.out_g.perXcd * NUM_XCD;
  const int scan = w.scan.M * (int)blocks_for(W, w.scan.blocks * RUN_COLS);
  if (!timed(h, {RNNLM_STAGE_OUT_BWD_W, RNNLM_STAGE_REC_W, RNNLM_STAGE_EMB})) return launch(rec, out, scan);
  int rc;
  {
    StageTimer tm(h, RNNLM_STAGE_EMB, st);
    rc = launch(0, 0, scan);
  }
  if (rc) return rc;
  {
    StageTimer tm(h, RNNLM_STAGE_REC_W, st);
    rc = launch(rec, 0, 0);
  }
  if (rc) return rc;
  StageTimer tm(h, RNNLM_STAGE_OUT_BWD_W, st);
  return launch(0, out, 0);
}

// Backward half of a window + fused updates.  Everything it starts is ordered before whatever comes next on st.
// rec_stream (may be nullptr) receives the stream whose next launch is ordered behind the recurrent update: work on the
// other stream is not.
template <typename T>
int backward_window(rnnlm_t *h, int Tn, const UpdateTargets &u, const NceCall *nce, hipStream_t st, hipStream_t *rec_stream,
                    float *logp_out, const WindowSum &wsum) {
  const rnnlm_config &c = h->cfg;
  const int Hp = h->Hp, Bp = h->Bp, Vp = h->Vp;
  const int Mrows = Tn * Bp;
  const int Mp = (int)window_plan(h, Mrows).Mp;
  const long ldz = h->MpMax, rowTerms = terms<T>(Mrows);
  T *Hs_c = at<T>(h, h->L.Hs_c);
  T *ZT = at<T>(h, h->L.ZT);
  T *Wo_c = at<T>(h, h->L.Wo_c);
  T *U_c = at<T>(h, h->L.U_c);
  T *dA_c = at<T>(h, h->L.dA_c);
  float *dA32 = at<float>(h, h->L.dA32);
  float *dHs32 = at<float>(h, h->L.dHs32);
  int32_t *xp = at<int32_t>(h, h->L.xp), *yp = at<int32_t>(h, h->L.yp);
  int32_t *perm = at<int32_t>(h, h->L.perm), *seg = at<int32_t>(h, h->L.seg);

  // the integer helpers of the embedding update were started on the side stream by forward_window

  if (nce) {
    int rc = nce_backward_h<T>(h, Tn, *nce, st);
    if (rc) return rc;
  } else {
  // fused softmax gradient + bias update, in place on the vocabulary-major logits
  {
    StageTimer tm(h, RNNLM_STAGE_SOFTMAX_GRAD, st);
    const WindowPlan &wp = window_plan(h, Mrows);
    const StatsMerge merge = {at<float2>(h, h->L.stat), wp.parts, Tn, c.B, Bp, at<float>(h, h->L.zy), at<float>(h, h->L.logp_int),
                              logp_out, wsum};
    hipLaunchKernelGGL((merged_in_pass(h, wp) ? softmax_grad_kernel<T, true> : softmax_grad_kernel<T, false>), dim3(Vp / 16),
                       dim3(256), 0, st, ZT, ldz, Mp, c.V, Vp, at<float>(h, h->L.lse), yp, 1.0f / (float)(Tn * c.B), h->buf.b, u.b,
                       u.alpha, u.lr, merge);
    HIP_TRY(hipGetLastError());
  }

  // dHs[m][j] = sum_v dz[v][m] Wo[v][j]   (contraction over the vocabulary, split-K); compressed
  // architecture: the same contraction with the tied matrix gives the gradient of the layer above the state
  {
    const int Dp = h->Dp;
    T *dP_c = c.P > 0 ? at<T>(h, h->L.dP_c) : nullptr;  // (an operand of the contraction below)
    const long per = (long)Mp * Dp;
    const int max_splits = (int)std::min<long>(MAX_SPLITS, std::max<long>(1, h->L.partElems / per));
    const long Dn = sizeof(T) == 4 ? features_formed(c, Mp, max_splits, ldz) : Dp;
    const F32Plan plan = sizeof(T) == 4 ? f32_plan(Mp, Dn, c.V, max_splits, ldz) : F32Plan{};
    const SumPlan sum = window_plan(h, Mrows).sum;
    int S = sizeof(T) == 4 ? plan.splits : sum.splits;
    if ((long)S * per > h->L.partElems) S = (int)(h->L.partElems / per);
    if (S < 1) S = 1;
    EpiPartial epi;
    epi.part = at<float>(h, h->L.part32);
    if (S == 1 && c.P == 0) epi.part = dHs32;
    if constexpr (sizeof(T) == 4)
      if (S == 1 && c.P > 0) epi.part = dP_c;
    epi.ld = Dp;
    epi.split_stride = per;
    {
      StageTimer tm(h, RNNLM_STAGE_OUT_BWD_H, st);
      if constexpr (sizeof(T) == 4) {
        HIP_TRY((f32_gemm<KROW, KROW>(st, ZT, ldz, Wo_c, Dp, Mp, Dn, round_up(c.V, 32), plan, epi)));
      } else if (sum.tile == BIG) {
        HIP_TRY((big_gemm<2, 4, KROW, KROW, true>(st, ZT, ldz, Wo_c, Dp, Mp, Dp, Vp, S, epi)));
      } else {
        HIP_TRY((bf16_small_gemm<KROW, KROW>(st, ZT, ldz, Wo_c, Dp, Mp, sum.feats, Vp, sum.tile, S, epi)));
      }
    }
    if (S > 1 || (c.P > 0 && sizeof(T) == 2)) {
      StageTimer tm(h, RNNLM_STAGE_REDUCE, st);
      int rc = c.P > 0 ? reduce_splits(st, epi.part, per, S, dP_c) : reduce_splits(st, epi.part, per, S, dHs32);
      if (rc) return rc;
    }
  }
  if (c.P > 0) {
    // through the layer above the state: dHs[m][j] = sum_p dp[m][p] C[p][j]
    StageTimer tm(h, RNNLM_STAGE_PROJ, st);
    const T *dP_c = at<T>(h, h->L.dP_c);
    EpiPartial epi;
    epi.part = dHs32;
    epi.ld = Hp;
    epi.split_stride = 0;
    HIP_TRY((mid_gemm<T, ROWK, KROW>(st, dP_c, h->Pp, at<T>(h, h->L.C_c), Hp, Mp, Hp, terms<T>(c.P), 1, epi)));
  }
  }

  // rows [Mrows, Mp) of dA take part in the dU contraction: keep them zero (the persistent path has them from
  // the token preparation)
  if (Mp > Mrows && !persistent_ok(h)) {
    const long n = (long)(Mp - Mrows) * Hp * (long)sizeof(T) / 4;
    hipLaunchKernelGGL(fill_kernel<uint32_t>, dim3(blocks_for(n, 256)), dim3(256), 0, st,
                       reinterpret_cast<uint32_t *>(dA_c + (long)Mrows * Hp), n, 0u);
  }

  // back-propagation through time over the window (stops at the window start)
  if (persistent_ok(h)) {
    StageTimer tm(h, RNNLM_STAGE_RNN_BWD, st);
    int rc = launch_rnn_persistent<T, true>(h, Tn, false, st);
    if (rc) return rc;
  } else if (sizeof(T) == 2 && resident_ok(h)) {
    StageTimer tm(h, RNNLM_STAGE_RNN_BWD, st);
    int rc = launch_rnn_resident<true>(h, Tn, false, st);
    if (rc) return rc;
  } else
  for (int t = Tn - 1; t >= 0; --t) {
    StageTimer tm(h, (t == 0 || t == Tn - 1) ? RNNLM_STAGE_RNN_BWD : -1, st, t == Tn - 1, t == 0);
    const bool contract = t < Tn - 1;  // nothing flows into the window's last position
    if (step_in_one(c)) {
      int rc = launch_rnn_step<T, true>(h, t, contract, nullptr, st);
      if (rc) return rc;
      continue;
    }
    const T *A_ = dA_c + (long)(t + 1) * Bp * Hp;
    const StepPlan p = step_plan(c, Bp, Hp);
    const long per = (long)Bp * Hp, at_t = (long)t * per, K = terms<T>(c.H);
    EpiPartial ep;
    ep.part = at<float>(h, h->L.part32);
    ep.ld = Hp;
    ep.split_stride = p.rows * Hp;
    if (contract) {
      if (!dma4_reaches<T>(KROW, Hp, 64, Hp)) {  // bf16, a matrix of 2^31 bytes and more
        HIP_TRY((launch_gemm<T, 64, 64, 2, 2, ROWK, KROW>(st, A_, Hp, U_c, Hp, p.rows, Hp, K, p.splits, ep)));
      } else if (!p.wide) {
        HIP_TRY((launch_gemm_dma4<T, 64, 64, 2, 2, ROWK, KROW>(st, A_, Hp, U_c, Hp, p.rows, Hp, K, p.splits, ep)));
      } else if constexpr (sizeof(T) == 2) {
        HIP_TRY((launch_gemm_dma4<bf16_t, 256, 128, 4, 2, ROWK, KROW>(st, A_, Hp, U_c, Hp, Bp, Hp, K, p.splits, ep)));
      } else {
        HIP_TRY((launch_gemm<T, 256, 64, 4, 2, ROWK, KROW>(st, A_, Hp, U_c, Hp, Bp, Hp, K, p.splits, ep)));
      }
    }
    hipLaunchKernelGGL(rnn_step_bwd_kernel<T>, dim3(blocks_for(per / 4, 256)), dim3(256), 0, st,
                       at<float>(h, h->L.part32), p.rows * Hp, contract ? p.splits : 0, dHs32 + at_t, Hs_c + at_t + per,
                       c.B, c.H, Hp, per / 4, dA32 + at_t, dA_c + at_t);
    HIP_TRY(hipGetLastError());
  }

  auto scan_update = [&](const float *rows, const float *src, float alpha, T *copy, int waves) {
    ScanUpdate<T> s = {rows, h->Dp, h->D, c.B, Bp, xp, src, u.E, alpha, u.lr, copy, h->Dp, Tn * c.B, 1};
    while (s.blocks < waves && s.blocks * RUN_COLS < h->D) s.blocks *= 2;  // 256-column blocks a workgroup has waves for
    return s;
  };
  auto recurrent_epilogue = [&]() {
    EpiSgdT<T> epi;
    epi.W = h->buf.U;
    epi.out = u.U;
    epi.Wc = u.refresh_copies ? U_c : nullptr;
    epi.WcT = u.refresh_copies ? at<T>(h, h->L.UT_c) : nullptr;  // the backward pass reads the transposed copy
    epi.ldw = c.H;
    epi.ldc = Hp;
    epi.R = c.H;
    epi.C = c.H;
    epi.alpha = u.alpha;
    epi.lr = u.lr;
    return epi;
  };
  auto aim = [&](auto &epi) {  // at the output layer's matrix
    epi.W = c.P > 0 ? h->buf.E : h->buf.Wo;
    epi.out = c.P > 0 ? u.E : u.Wo;
    epi.Wc = u.refresh_copies ? Wo_c : nullptr;
    epi.ldw = h->D;
    epi.ldc = h->Dp;
    epi.R = c.V;
    epi.C = h->D;
    epi.alpha = u.alpha;
    epi.lr = u.lr;
  };
  const bool big_rec = sizeof(T) == 2 && (long)(Hp / BIG) * (Hp / BIG) >= 64;  // the recurrent update fills the chip
  if (!nce && c.P == 0 && !big_rec && scan_ids(h, Tn, u)) {
    WindowUpdate<T> w;
    const int tile = window_update_shape<T>(h, Mrows, ZT, Hs_c, dA_c, w);
    if (tile > 0) {
      aim(w.out);
      w.rec = recurrent_epilogue();
      w.scan = scan_update(dA32, h->buf.E, u.alpha, nullptr, tile / 16);
      if (rec_stream) *rec_stream = st;
      return launch_window_update<T>(h, w, tile, Mrows, st);
    }
  }
  const bool serial = !nce && scan_ids(h, Tn, u) && short_output_update(h, Tn);
  hipStream_t es = serial ? st : h->side;
  // E[w] -= lr * sum_{m: x[m] = w} dA[m]: on the side stream, behind the sort helpers already queued there (joined at
  // the end of this function).
  auto embedding_update = [&]() -> int {
  {
    StageTimer tm(h, RNNLM_STAGE_EMB, es);
    // plain: rows of dA, width H.  Compressed: rows of dx, width P, added on top of the output-side update the
    // same matrix has just received (training: in the master; gradient export: in the caller's buffer), and
    // the compute copy of the tied matrix follows.
    const float *rows = c.P > 0 ? at<float>(h, h->L.dX32) : dA32;
    const float *src = (c.P > 0 && !u.refresh_copies) ? u.E : h->buf.E;
    const float e_alpha = (c.P > 0 && !u.refresh_copies) ? 1.0f : u.alpha;
    T *Ec = (c.P > 0 && u.refresh_copies) ? Wo_c : nullptr;
    const int W = h->D, Wp = h->Dp;
    const bool scan = scan_ids(h, Tn, u);
    const dim3 threads(64 * RUN_WAVES);
    if (scan) {
      const ScanUpdate<T> su = scan_update(rows, src, e_alpha, Ec, RUN_WAVES);
      hipLaunchKernelGGL((W % 4 == 0 ? scatter_scan_kernel<true, T> : scatter_scan_kernel<false, T>),
                         dim3(su.M, blocks_for(W, su.blocks * RUN_COLS)), threads, 0, es, su);
    } else {
      hipLaunchKernelGGL((W % 4 == 0 ? scatter_runs_kernel<true, T> : scatter_runs_kernel<false, T>),
                         dim3(blocks_for(Tn * c.B, RUN_WAVES), blocks_for(W, RUN_COLS)), threads, 0, es, rows, Wp, W, c.B, Bp,
                         xp, perm, seg, p_nseg(h), src, u.E, e_alpha, u.lr, u.e_compact_ld, Ec, Wp);
    }
    HIP_TRY(hipGetLastError());
  }
    return RNNLM_OK;
  };
  // U[i][j] -= lr * sum_m dA[m][i] Hprev[m][j], contracted transposed (tile rows = j, tile columns = i)
  auto recurrent_update = [&](hipStream_t rs) -> int {
  {
    StageTimer tm(h, RNNLM_STAGE_REC_W, rs);
    const EpiSgdT<T> epi = recurrent_epilogue();
    if (big_rec) {
      if constexpr (sizeof(T) == 2)
        HIP_TRY((big_gemm<2, 4, KROW, KROW, true>(rs, Hs_c, Hp, dA_c, Hp, Hp, Hp, rowTerms, 1, epi)));
    } else {
      const long n = round_up(c.H, 64);  // (the epilogue writes valid entries only)
      HIP_TRY((mid_gemm<T, KROW, KROW>(rs, Hs_c, Hp, dA_c, Hp, n, n, rowTerms, 1, epi)));
    }
  }
    return RNNLM_OK;
  };
  // Plain architecture with the normalised criterion: the embedding update and the recurrent weight update need
  // nothing from the output weight update: started on the side stream BEFORE it, they run on the compute units
  // that its last, partly empty round of tiles leaves idle (window time -2 % at H = 2048, -1.3 % at H = 1024).  At
  // H = 4096 the recurrent update is a full round of 256 tiles by itself and keeps its place after the output
  // weight update; the embedding update goes first there as well.
  // Under the noise-contrastive criterion they run next to the update of the touched rows, which is latency-bound (V =
  // 64000, H = 1024, 128x20, 1024 noise words, rmsprop: with the decay and the steps of E and U on that stream as well
  // 319 -> 265 us).
  const bool early_side = c.P == 0;
  const bool early_rec = early_side && (nce || (long)(Hp / BIG) * (Hp / BIG) < 256);
  if (rec_stream) *rec_stream = early_rec ? es : st;
  // An event between the fork and the output update's launch (its stage is timed) lets the embedding update start first,
  // whose workgroups do not fit next to the large update's and keep it from some compute units until they are through.  At
  // the widest layers those compute units then lack in 24 rounds of tiles (V = 100000, H = 4096, 256x32: update 5.72 ms instead
  // of 5.28, window 17.6 instead of 17.2), so the stage opens before the fork there.  With few rounds the timed window is
  // shorter with the embedding update in front (128x20, V = 64000, H = 1024 and V = 100000, H = 2048: 1.2 % each).
  const bool opened = early_side && !early_rec && !serial;
  if (opened) StageTimer(h, RNNLM_STAGE_OUT_BWD_W, st, true, false);
  if (early_side) {
    int rc = serial ? RNNLM_OK : side_fork(h, 0, st);
    if (rc) return rc;
    rc = embedding_update();
    if (rc) return rc;
    if (early_rec) {
      rc = recurrent_update(es);
      if (rc) return rc;
    }
  }
  if (nce) {
    int rc = nce_update<T>(h, Tn, *nce, u, st);
    if (rc) return rc;
  } else {
    {
    // Wo[v][j] -= lr * sum_m dz[v][m] Hs[m][j]; compressed architecture: the output-side update of the tied matrix,
    // E[v][p] -= lr * sum_m dz[v][m] p[m][p].  bf16 compressed on large tiles: contracted transposed (tile rows = p, tile
    // columns = v).
    // Everything else in the matrix's own orientation (tile rows = v, tile columns = j), whose update epilogue touches two
    // 128-byte lines per wave instruction instead of 32 (fp32, V = 64000, H = 1024, 1280 positions: 893 -> 841 us).
    StageTimer tm(h, RNNLM_STAGE_OUT_BWD_W, st, !opened);
    const T *feat = c.P > 0 ? at<T>(h, h->L.P_c) : Hs_c + (long)Bp * Hp;
    EpiSgd<T> epi;
    aim(epi);
    if constexpr (sizeof(T) == 4) {
      const long Dn = f32_extent(h->D, Vp, Mrows, 1), K = round_up(Mrows, 32);
      const F32Plan plan = f32_plan(Vp, Dn, Mrows, 1);
      if (split_reaches(ROWK, ldz, plan.tile, 64)) {
        HIP_TRY((f32_gemm<ROWK, KROW>(st, ZT, ldz, feat, h->Dp, Vp, Dn, K, plan, epi, -4)));
      } else if (Dn % 128 == 0) {  // handles of millions of positions
        HIP_TRY((launch_gemm<T, 128, 128, 2, 2, ROWK, KROW>(st, ZT, ldz, feat, h->Dp, Vp, Dn, K, 1, epi, -4)));
      } else {
        HIP_TRY((launch_gemm<T, 64, 64, 2, 2, ROWK, KROW>(st, ZT, ldz, feat, h->Dp, Vp, Dn, K, 1, epi, -4)));
      }
    } else if (const long Dn = bf16_extent(OUT_UPDATE, h->D, Vp, rowTerms);
               bf16_tile(OUT_UPDATE, Vp, Dn, rowTerms) != BIG) {
      HIP_TRY((bf16_small_gemm<ROWK, KROW>(st, ZT, ldz, feat, h->Dp, Vp, Dn, rowTerms, bf16_tile(OUT_UPDATE, Vp, Dn, rowTerms), 1,
                                           epi, -4)));
    } else if (c.P == 0) {
      // Tiles are walked in bands of 4 (wide matrices: 8) tile columns, so that the 32 tiles an XCD works on at a time
      // share few operand panels in its L2 (8 x 4 or 4 x 8 instead of 2 x 16: 4 % faster on the widest configuration).
      // dz is the K-contiguous operand: up to 8 tile columns its tiles travel as whole cache lines (64-deep blocks,
      // gemm_ring64.h: 8-9 % faster at H = 1024 and 2048); the widest layer runs at the chip's power limit, where the
      // symmetric ring measured 0.5 % better
      if (Hp / BIG >= 16) {
        HIP_TRY((big_gemm<2, 4, ROWK, KROW, true>(st, ZT, ldz, feat, Hp, Vp, Hp, rowTerms, 1, epi, -8)));
      } else {
        HIP_TRY((launch_gemm_ring64<BIG, BIG, 2, 4>(st, ZT, ldz, feat, Hp, Vp, Hp, rowTerms, 1, epi, -4)));
      }
    } else {
      EpiSgdT<T> et;
      aim(et);
      if ((long)(h->Dp / BIG) * (Vp / BIG) < 128) {  // a narrow layer above the state: smaller tiles fill the chip
        HIP_TRY((launch_gemm_dma4<bf16_t, 128, BIG, 2, 4, KROW, ROWK>(st, feat, h->Dp, ZT, ldz, h->Dp, Vp, rowTerms, 1, et, -4)));
      } else {
        HIP_TRY((big_gemm<2, 4, KROW, ROWK, true>(st, feat, h->Dp, ZT, ldz, h->Dp, Vp, rowTerms, 1, et, -2)));
      }
    }
    }
    if (c.P > 0) {
      // through the layer below the state: dx[m][p] = sum_i da[m][i] A[i][p] (before A is updated)
      StageTimer tm(h, RNNLM_STAGE_PROJ, st);
      EpiPartial epi;
      epi.part = at<float>(h, h->L.dX32);
      epi.ld = h->Pp;
      epi.split_stride = 0;
      HIP_TRY((mid_gemm<T, ROWK, KROW>(st, dA_c, Hp, at<T>(h, h->L.A_c), h->Pp, Mp, h->Pp, terms<T>(c.H), 1, epi)));
    }
  }
  if (!early_side) {
    int rc = serial ? RNNLM_OK : side_fork(h, 0, st);  // the side stream waits for everything queued so far
    if (rc) return rc;
    rc = embedding_update();
    if (rc) return rc;
  }
  bool rec_done = early_rec;
  if (c.P > 0) {
    StageTimer tm(h, RNNLM_STAGE_PROJ, st);
    // C[p][j] -= lr * sum_m dp[m][p] h[m][j], contracted transposed (tile rows = j, tile columns = p)
    EpiSgdT<T> ec;
    ec.W = h->buf.C;
    ec.out = u.C;
    ec.Wc = u.refresh_copies ? at<T>(h, h->L.C_c) : nullptr;
    ec.ldw = c.H;
    ec.ldc = Hp;
    ec.R = c.P;
    ec.C = c.H;
    ec.alpha = u.alpha;
    ec.lr = u.lr;
    // A[i][p] -= lr * sum_m da[m][i] x[m][p], contracted transposed (tile rows = p, tile columns = i)
    EpiSgdT<T> ea;
    ea.W = h->buf.A;
    ea.out = u.A;
    ea.Wc = u.refresh_copies ? at<T>(h, h->L.A_c) : nullptr;
    ea.ldw = c.P;
    ea.ldc = h->Pp;
    ea.R = c.H;
    ea.C = c.P;
    ea.alpha = u.alpha;
    ea.lr = u.lr;
    const T *Hs1 = Hs_c + (long)Bp * Hp, *dP_c = at<T>(h, h->L.dP_c), *Xp_c = at<T>(h, h->L.Xp_c);
    bool grouped = false;
    if constexpr (sizeof(T) == 2) {
      // (epilogues write valid entries only: extents are padded to whole tiles, no further)
      const long Hn = round_up(c.H, 64), Pn = round_up(c.P, 64);
      UpdateGroup<EpiSgdT<T>> group;
      grouped = dma4_shape<T, 64, 64, KROW, KROW>(group.g[0], Hs1, Hp, dP_c, h->Pp, Hn, Pn, rowTerms, 1, 4) == hipSuccess &&
                dma4_shape<T, 64, 64, KROW, KROW>(group.g[1], Xp_c, h->Pp, dA_c, Hp, Pn, Hn, rowTerms, 1, 4) == hipSuccess &&
                dma4_shape<T, 64, 64, KROW, KROW>(group.g[2], Hs_c, Hp, dA_c, Hp, Hn, Hn, rowTerms, 1, 4) == hipSuccess;
      if (grouped) {
        group.epi[0] = ec;
        group.epi[1] = ea;
        group.epi[2] = recurrent_epilogue();
        group.first[0] = 0;
        for (int q = 0; q < GROUP_MAX; ++q) group.first[q + 1] = group.first[q] + group.g[q].perXcd * NUM_XCD;
        rec_done = !big_rec && !timed(h, {RNNLM_STAGE_PROJ, RNNLM_STAGE_REC_W});
        hipLaunchKernelGGL((update_group_kernel<KROW, KROW, EpiSgdT<T>>), dim3(group.first[rec_done ? 3 : 2]), dim3(256), 0, st,
                           group);
        HIP_TRY(hipGetLastError());
      }
    }
    if (!grouped) {
      HIP_TRY((mid_gemm<T, KROW, KROW>(st, Hs1, Hp, dP_c, h->Pp, Hp, h->Pp, rowTerms, 1, ec)));
      HIP_TRY((mid_gemm<T, KROW, KROW>(st, Xp_c, h->Pp, dA_c, Hp, h->Pp, Hp, rowTerms, 1, ea)));
    }
  }

  if (!rec_done) {
    int rc = recurrent_update(st);
    if (rc) return rc;
  }
  // wait for the embedding update running on the side stream
  return serial ? RNNLM_OK : side_join(h, 0, st);
}

template <typename T>
int window_call(rnnlm_t *h, const int32_t *x, const int32_t *y, int Tn, float *logp, double *sum_logp,
                const UpdateTargets *u, bool advance_state, hipStream_t st, const NceCall *nce = nullptr,
                hipStream_t *rec_stream = nullptr) {
  const bool want_sum = sum_logp || u;
  const WindowSum ws = {sum_logp ? sum_logp : p_sum(h), nullptr, p_flags(h), u ? p_counter(h) : nullptr};
  int rc = forward_window<T>(h, x, y, Tn, logp, advance_state, nce == nullptr, st, u != nullptr,
                             u && !scan_ids(h, Tn, *u), false, want_sum && !nce ? &ws : nullptr);
  if (rc) return rc;
  if (nce) {  // per-position losses take the place of the log-probabilities
    rc = nce_forward<T>(h, Tn, *nce, want_sum ? &ws : nullptr, st);
    if (rc) return rc;
  }
  if (u) rc = backward_window<T>(h, Tn, *u, nce, st, rec_stream, logp, ws);
  return rc;
}

template <typename T>
int score_call(rnnlm_t *h, const int32_t *x, const int32_t *y, int Tn, float lnZ, float *score, hipStream_t st) {
  int rc = forward_window<T>(h, x, y, Tn, nullptr, true, false, st, false, false, true);
  if (rc) return rc;
  const int Mrows = Tn * h->Bp;
  StageTimer tm(h, RNNLM_STAGE_NCE_SCORE, st);
  // what the output layer reads: the states, or (compressed architecture) the layer above them
  const T *feat = h->cfg.P > 0 ? at<T>(h, h->L.P_c) : at<T>(h, h->L.Hs_c) + (long)h->Bp * h->Hp;
  // the per-position scratch of the log-probability path holds the padded result
  hipLaunchKernelGGL(nce_target_score_kernel<T>, dim3(blocks_for(Mrows, 4)), dim3(256), 0, st, feat,
                     at<T>(h, h->L.Wo_c), h->Dp, at<int32_t>(h, h->L.yp), h->buf.b, (const float *)nullptr, lnZ, Mrows,
                     h->cfg.B, h->Bp, at<float>(h, h->L.zy), score);
  HIP_TRY(hipGetLastError());
  return RNNLM_OK;
}

// Forward pass, then the scores of C candidate words per position (no targets: y = nullptr).
template <typename T>
int shortlist_call(rnnlm_t *h, const int32_t *x, const int32_t *cand, int C, int Tn, float lnZ, float *score,
                   hipStream_t st) {
  int rc = forward_window<T>(h, x, nullptr, Tn, nullptr, true, false, st, false, false, true);
  if (rc) return rc;
  StageTimer tm(h, RNNLM_STAGE_NCE_SCORE, st);
  const T *feat = h->cfg.P > 0 ? at<T>(h, h->L.P_c) : at<T>(h, h->L.Hs_c) + (long)h->Bp * h->Hp;
  const long total = (long)Tn * h->cfg.B * C;
  hipLaunchKernelGGL(score_candidates_kernel<T>, dim3(blocks_for(total, 4)), dim3(256), 0, st, feat,
                     at<T>(h, h->L.Wo_c), h->Dp, cand, C, h->cfg.V, h->buf.b, lnZ, total, h->cfg.B, h->Bp, p_flags(h),
                     score);
  HIP_TRY(hipGetLastError());
  return RNNLM_OK;
}

template <typename T>
int quantize_call(rnnlm_t *h, const rnnlm_quantized &q, hipStream_t st) {
  const rnnlm_config &c = h->cfg;
  hipLaunchKernelGGL(quantize_rows_kernel<T>, dim3(c.V), dim3(256), 0, st, h->buf.E, c.P, q.qE, q.sE,
                     reinterpret_cast<T *>(h->ws + h->L.Wo_c), h->Pp);
  hipLaunchKernelGGL(quantize_rows_kernel<T>, dim3(c.H), dim3(256), 0, st, h->buf.A, c.P, q.qA, q.sA,
                     reinterpret_cast<T *>(h->ws + h->L.A_c), h->Pp);
  hipLaunchKernelGGL(quantize_rows_kernel<T>, dim3(c.H), dim3(256), 0, st, h->buf.U, c.H, q.qU, q.sU,
                     reinterpret_cast<T *>(h->ws + h->L.U_c), h->Hp);
  hipLaunchKernelGGL(quantize_rows_kernel<T>, dim3(c.P), dim3(256), 0, st, h->buf.C, c.H, q.qC, q.sC,
                     reinterpret_cast<T *>(h->ws + h->L.C_c), h->Hp);
  hipLaunchKernelGGL(transpose_kernel<T>, dim3(h->Hp / 32, h->Hp / 32), dim3(256), 0, st,
                     reinterpret_cast<T *>(h->ws + h->L.U_c), h->Hp, reinterpret_cast<T *>(h->ws + h->L.UT_c));
  HIP_TRY(hipGetLastError());
  return RNNLM_OK;
}

bool window_args_ok(rnnlm_t *h, const int32_t *x, const int32_t *y, int T) {
  return h && x && y && T >= 1 && T <= h->cfg.T_max;
}

// The statistics' decay depends on nothing in the window: it starts on the side stream with it (joined with that stream's
// other work at the end of the backward pass).  Short windows spend their time in the host's calls: there neither the
// decay nor the steps overlap anything, which saves a pair of events each.  With and without the overlap, bf16: softmax, V
// = 1000, H = 64, one position 160 and 138 us, 1024 positions 167 and 157, 2048 positions 175 and 180 (V = 20000, H = 1024,
// 128 positions, not short: 229 and 232); noise-contrastive, V = 10000, H = 512, 256 positions 213 and 182, V = 64000,
// H = 1024, 1280 positions 205 and 187, 2560 positions 249 and 253.
bool rms_overlaps(rnnlm_t *h, int Tn, bool nce) {
  return (long)Tn * h->cfg.B > 1024 || !(nce || short_output_update(h, Tn));
}
int rms_decay(rnnlm_t *h, float *r0, float *r1, float *r2, float rho, bool overlap, hipStream_t st) {
  int rc = overlap ? side_fork(h, 0, st) : RNNLM_OK;
  if (rc) return rc;
  hipLaunchKernelGGL(rms_decay_kernel, dim3(blocks_for(h->cfg.V, 256), r1 ? 3 : 1), dim3(256), 0, overlap ? h->side : st,
                     r0, r1, r2, (long)h->cfg.V, rho);
  HIP_TRY(hipGetLastError());
  return RNNLM_OK;
}
// Steps of the embedding rows and of the recurrent matrix, on streams that are ordered behind their gradients: next to the
// steps of the output layer, the stream that formed the gradient (the side stream; backward_window says which one formed
// the recurrent one), otherwise the caller's.
template <typename T>
int rms_apply_inner(rnnlm_t *h, int Tn, const rnnlm_rmsprop_state &state, float rho, float lr, float eps,
                    hipStream_t emb_stream, hipStream_t rec_stream) {
  const rnnlm_config &c = h->cfg;
  hipLaunchKernelGGL(rms_row_apply_kernel<T>, dim3(Tn * c.B), dim3(256), 0, emb_stream, at<float>(h, h->L.dHs32), (long)h->Hp,
                     at<int32_t>(h, h->L.xp), at<int32_t>(h, h->L.perm), at<int32_t>(h, h->L.seg), p_nseg(h), c.B, h->Bp,
                     c.H, h->Hp, h->buf.E, (T *)nullptr, state.rE, rho, lr, eps, nullptr, nullptr, nullptr);
  const unsigned tiles = blocks_for(c.H, 32);
  hipLaunchKernelGGL(rms_square_apply_kernel<T>, dim3(tiles, tiles), dim3(256), 0, rec_stream, at<float>(h, h->L.gU), c.H,
                     h->buf.U, at<T>(h, h->L.U_c), at<T>(h, h->L.UT_c), h->Hp, state.rU, rho, lr, eps);
  HIP_TRY(hipGetLastError());
  return RNNLM_OK;
}
template <typename T>
int rms_apply(rnnlm_t *h, int Tn, const rnnlm_rmsprop_state &state, float rho, float lr, float eps, hipStream_t st,
              hipStream_t rec_stream) {
  const rnnlm_config &c = h->cfg;
  StageTimer tm(h, RNNLM_STAGE_RMSPROP, st);
  const bool overlap = rms_overlaps(h, Tn, false);
  int rc = rms_apply_inner<T>(h, Tn, state, rho, lr, eps, overlap ? h->side : st, overlap ? rec_stream : st);
  if (rc) return rc;
  hipLaunchKernelGGL(rms_row_apply_kernel<T>, dim3(c.V), dim3(256), 0, st, at<float>(h, h->L.gWo), (long)c.H, nullptr,
                     nullptr, nullptr, nullptr, c.B, h->Bp, c.H, h->Hp, h->buf.Wo, at<T>(h, h->L.Wo_c), state.rWo, rho, lr,
                     eps, nullptr, nullptr, nullptr);
  hipLaunchKernelGGL(rms_elem_apply_kernel, dim3(blocks_for(c.V, 256)), dim3(256), 0, st, at<float>(h, h->L.gb), c.V,
                     h->buf.b, state.rb, rho, lr, eps);
  HIP_TRY(hipGetLastError());
  return overlap ? side_join(h, 0, st) : RNNLM_OK;
}
template <typename T>
int rms_apply_nce(rnnlm_t *h, int Tn, int K, const rnnlm_rmsprop_state &state, float rho, float lr, float eps,
                  hipStream_t st, hipStream_t rec_stream) {
  const rnnlm_config &c = h->cfg;
  StageTimer tm(h, RNNLM_STAGE_RMSPROP, st);
  const bool overlap = rms_overlaps(h, Tn, true);
  int rc = rms_apply_inner<T>(h, Tn, state, rho, lr, eps, overlap ? h->side : st, overlap ? rec_stream : st);
  if (rc) return rc;
  const int nent = K + Tn * c.B;
  const int32_t *ids = at<int32_t>(h, h->L.ids), *perm2 = at<int32_t>(h, h->L.perm2), *seg2 = at<int32_t>(h, h->L.seg2);
  // the sort helpers' key indexing key[(i / B) * Bp + i % B] with B = Bp = 1 reads the compact id list
  hipLaunchKernelGGL(rms_row_apply_kernel<T>, dim3(nent), dim3(256), 0, st, at<float>(h, h->L.gN), (long)h->Hp, ids, perm2,
                     seg2, p_nseg2(h), 1, 1, c.H, h->Hp, h->buf.Wo, at<T>(h, h->L.Wo_c), state.rWo, rho, lr, eps,
                     at<float>(h, h->L.gbN), h->buf.b, state.rb);
  HIP_TRY(hipGetLastError());
  return overlap ? side_join(h, 0, st) : RNNLM_OK;
}
// Evaluation of a whole text: windows follow one another in each stream, and a forward pass writes no logits, so the space
// of the logits holds the positions of many windows and the handle runs them as one.  What that saves, per window: the
// launches between two recurrences and their start (some 20 us), and a last, partly empty round of tiles (V = 64000, H = 1024,
// 64x20, eight windows: 1250 tiles each on 256 compute units, 10000 together).  The layout is the handle's own again when
// this goes out of scope.
struct LongWindows {
  rnnlm_t *h;
  const WsLayout L;
  const int MpMax;
  long windows = 1;  // how many windows of T positions a call takes
  LongWindows(rnnlm_t *h_, int T, long most) : h(h_), L(h_->L), MpMax(h_->MpMax) {
    // (the other recurrent forms leave padding to what the workspace is initialised with)
    if (!persistent_ok(h)) return;
    const long per = (long)T * h->cfg.B;
    long W = std::min(most, std::max(1L, std::min((1L << 24) / per, 4096L / T)));
    while (W > 1 && !carve(W * T, most % W * T)) W = W > 2 ? W * 7 / 8 : 1;
    windows = W;
    if (W == 1) {
      h->L = L;
      h->MpMax = MpMax;
    }
  }
  ~LongWindows() {
    h->L = L;
    h->MpMax = MpMax;
  }
  // T positions a stream, and `last` in the call for what is left over
  bool carve(long T, long last) {
    const rnnlm_config &c = h->cfg;
    const size_t es = c.precision == RNNLM_FP32 ? 4 : 2;
    const long Mmax = round_up(T * h->Bp, PAD_M);
    auto stats = [&](long M) {
      const long Mp = window_rows(c, M);
      const long parts = es == 4 ? h->Vp / f32_plan(h->Vp, Mp, h->D, 1).tile : stat_parts(h->Vp, Mp, terms<bf16_t>(h->D));
      return (size_t)parts * Mp * 8;
    };
    size_t o = L.ZT;
    auto take = [&](size_t &at, size_t bytes) {
      at = o;
      o = align256(o + bytes);
    };
    WsLayout &n = h->L;
    take(n.Hs_c, (size_t)(Mmax + h->Bp + 64) * h->Hp * es);
    take(n.X32, (size_t)Mmax * h->Hp * 4);
    take(n.stat, std::max(stats(T * h->Bp), last > 0 ? stats(last * h->Bp) : 0));
    for (size_t *at : {&n.lse, &n.zy, &n.logp_int, &n.xp, &n.yp, &n.xtmp, &n.ytmp}) take(*at, (size_t)Mmax * 4);
    if (c.P > 0) {
      take(n.Xp_c, (size_t)Mmax * h->Pp * es);
      take(n.P_c, (size_t)Mmax * h->Pp * es);
    }
    h->MpMax = (int)Mmax;
    return o <= L.dA_c;  // (what follows the logits in the workspace)
  }
};
}  // namespace

extern "C" {

size_t rnnlm_workspace_bytes(const rnnlm_config *cfg) {
  if (!cfg_ok(cfg)) return 0;
  int Hp, Vp, Bp, MpMax, KpMax;
  WsLayout L;
  make_layout(*cfg, Hp, Vp, Bp, MpMax, KpMax, L);
  return L.total;
}

int rnnlm_init(const rnnlm_config *cfg, const rnnlm_buffers *buf, rnnlm_t **out) {
  if (!out) return RNNLM_ERR_ARG;
  *out = nullptr;
  if (!cfg_ok(cfg) || !buf) return RNNLM_ERR_ARG;
  if (!buf->E || !buf->U || !buf->b || !buf->h_state || !buf->workspace) return RNNLM_ERR_ARG;
  if (cfg->P > 0 ? (buf->Wo || !buf->A || !buf->C) : (!buf->Wo || buf->A || buf->C)) return RNNLM_ERR_ARG;
  if (reinterpret_cast<uintptr_t>(buf->workspace) & 255) return RNNLM_ERR_ARG;
  if ((reinterpret_cast<uintptr_t>(buf->E) | reinterpret_cast<uintptr_t>(buf->U) |
       reinterpret_cast<uintptr_t>(buf->Wo) | reinterpret_cast<uintptr_t>(buf->b) |
       reinterpret_cast<uintptr_t>(buf->h_state) | reinterpret_cast<uintptr_t>(buf->A) |
       reinterpret_cast<uintptr_t>(buf->C)) & 15)
    return RNNLM_ERR_ARG;
  rnnlm_t *h = new (std::nothrow) rnnlm_t;
  if (!h) return RNNLM_ERR_NOMEM;
  h->cfg = *cfg;
  h->buf = *buf;
  make_layout(*cfg, h->Hp, h->Vp, h->Bp, h->MpMax, h->KpMax, h->L);
  h->plan = recurrent_plan(*cfg);
  h->Pp = (int)round_up(cfg->P, PAD_H);
  h->D = cfg->P > 0 ? cfg->P : cfg->H;
  h->Dp = cfg->P > 0 ? h->Pp : h->Hp;
  if (buf->workspace_bytes < h->L.total) {
    delete h;
    return RNNLM_ERR_ARG;
  }
  h->ws = static_cast<char *>(buf->workspace);
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || cfg->device >= ndev || hipSetDevice(cfg->device) != hipSuccess) {
    delete h;
    return RNNLM_ERR_HIP;
  }
  int rc = RNNLM_OK;
  if (hipMemsetAsync(h->ws, 0, h->L.total, nullptr) != hipSuccess ||
      hipMemsetAsync(buf->h_state, 0, sizeof(float) * (size_t)cfg->B * cfg->H, nullptr) != hipSuccess)
    rc = RNNLM_ERR_HIP;
  if (rc == RNNLM_OK)
    rc = (cfg->precision == RNNLM_FP32) ? sync_copies<float>(h, nullptr) : sync_copies<bf16_t>(h, nullptr);
  if (rc == RNNLM_OK && hipDeviceSynchronize() != hipSuccess) rc = RNNLM_ERR_HIP;
  if (rc == RNNLM_OK) {
    // where do the workgroups of a grid land?  (uses the start of the not-yet-used embedding rows)
    constexpr int N = 64 * NUM_XCD;
    int32_t *dev = at<int32_t>(h, h->L.X32);
    int32_t host[N];
    hipLaunchKernelGGL(xcd_probe_kernel, dim3(N), dim3(64), 0, nullptr, dev);
    if (hipMemcpy(host, dev, sizeof(host), hipMemcpyDeviceToHost) != hipSuccess ||
        hipMemsetAsync(dev, 0, sizeof(host), nullptr) != hipSuccess || hipDeviceSynchronize() != hipSuccess) {
      rc = RNNLM_ERR_HIP;
    } else {
      // round-robin from whatever XCD the dispatcher had reached: block i on XCD (first + i) mod 8.  The start
      // rotates from launch to launch (it continues where the previous grid ended); what the XCD-local kernels
      // need is only that a grid of 8 n workgroups puts exactly n on every XCD, which any rotation gives.
      bool rr = host[0] >= 0 && host[0] < NUM_XCD;
      for (int i = 0; i < N; ++i) rr = rr && host[i] == (host[0] + i) % NUM_XCD;
      h->xcd_local = rr;
    }
  }
  if (rc == RNNLM_OK) {
    bool ok = hipStreamCreateWithFlags(&h->side, hipStreamNonBlocking) == hipSuccess;
    for (int i = 0; i < 2 && ok; ++i)
      ok = hipEventCreateWithFlags(&h->ev_fork[i], hipEventDisableTiming) == hipSuccess &&
           hipEventCreateWithFlags(&h->ev_join[i], hipEventDisableTiming) == hipSuccess;
    if (!ok) rc = RNNLM_ERR_HIP;
  }
  if (rc != RNNLM_OK) {
    rnnlm_free(h);
    return rc;
  }
  *out = h;
  return RNNLM_OK;
}

void rnnlm_free(rnnlm_t *h) {
  if (!h) return;
  for (EventPair &e : h->prof_pool) {
    (void)hipEventDestroy(e.start);
    (void)hipEventDestroy(e.stop);
  }
  for (int i = 0; i < 2; ++i) {
    if (h->ev_fork[i]) (void)hipEventDestroy(h->ev_fork[i]);
    if (h->ev_join[i]) (void)hipEventDestroy(h->ev_join[i]);
  }
  if (h->side) {
    (void)hipStreamSynchronize(h->side);
    (void)hipStreamDestroy(h->side);
  }
  delete h;
}

int rnnlm_stream_chunk(rnnlm_t *h, const int32_t *tok, int64_t N, int64_t k, int32_t T, int32_t *x, int32_t *y,
                       void *stream) {
  if (!h || !tok || !x || !y || N < 2 || T < 1 || T > h->cfg.T_max) return RNNLM_ERR_ARG;
  const long L = (long)((N - 1) / h->cfg.B);
  if (k < 0 || k >= L / T) return RNNLM_ERR_ARG;
  hipLaunchKernelGGL(stream_chunk_kernel, dim3(blocks_for((long)T * h->cfg.B, 256)), dim3(256), 0, (hipStream_t)stream,
                     tok, L, (long)k, T, h->cfg.B, x, y);
  HIP_TRY(hipGetLastError());
  return RNNLM_OK;
}

int rnnlm_forward_logprob(rnnlm_t *h, const int32_t *x, const int32_t *y, int32_t T, float *logp, void *stream) {
  if (!window_args_ok(h, x, y, T) || !logp) return RNNLM_ERR_ARG;
  hipStream_t st = (hipStream_t)stream;
  return (h->cfg.precision == RNNLM_FP32) ? window_call<float>(h, x, y, T, logp, nullptr, nullptr, true, st)
                                          : window_call<bf16_t>(h, x, y, T, logp, nullptr, nullptr, true, st);
}

int rnnlm_train_chunk(rnnlm_t *h, const int32_t *x, const int32_t *y, int32_t T, float lr, float *logp,
                      double *sum_logp, void *stream) {
  if (!window_args_ok(h, x, y, T) || !(lr == lr)) return RNNLM_ERR_ARG;
  hipStream_t st = (hipStream_t)stream;
  UpdateTargets u{h->buf.E, h->buf.U, h->buf.Wo, h->buf.b, 1.0f, lr, true, true};
  u.A = h->buf.A;
  u.C = h->buf.C;
  return (h->cfg.precision == RNNLM_FP32) ? window_call<float>(h, x, y, T, logp, sum_logp, &u, true, st)
                                          : window_call<bf16_t>(h, x, y, T, logp, sum_logp, &u, true, st);
}

int rnnlm_grad_chunk(rnnlm_t *h, const int32_t *x, const int32_t *y, int32_t T, float *dE, float *dU, float *dWo,
                     float *db, float *logp, void *stream) {
  if (!window_args_ok(h, x, y, T) || !dE || !dU || !dWo || !db || h->cfg.P > 0) return RNNLM_ERR_ARG;
  if ((reinterpret_cast<uintptr_t>(dE) | reinterpret_cast<uintptr_t>(dU) | reinterpret_cast<uintptr_t>(dWo) |
       reinterpret_cast<uintptr_t>(db)) & 15)
    return RNNLM_ERR_ARG;  // the update epilogues use 16-byte accesses
  hipStream_t st = (hipStream_t)stream;
  const long nE = (long)h->cfg.V * h->cfg.H;
  hipLaunchKernelGGL(fill_kernel<float>, dim3(std::min<long>(blocks_for(nE, 256), 65535)), dim3(256), 0, st, dE, nE,
                     0.0f);
  HIP_TRY(hipGetLastError());
  UpdateTargets u{dE, dU, dWo, db, 0.0f, -1.0f, false, false};
  return (h->cfg.precision == RNNLM_FP32) ? window_call<float>(h, x, y, T, logp, nullptr, &u, false, st)
                                          : window_call<bf16_t>(h, x, y, T, logp, nullptr, &u, false, st);
}

int rnnlm_grad_chunk_compressed(rnnlm_t *h, const int32_t *x, const int32_t *y, int32_t T, float *dE, float *dA,
                                float *dU, float *dC, float *db, float *logp, void *stream) {
  if (!window_args_ok(h, x, y, T) || !dE || !dA || !dU || !dC || !db || h->cfg.P <= 0) return RNNLM_ERR_ARG;
  if ((reinterpret_cast<uintptr_t>(dE) | reinterpret_cast<uintptr_t>(dA) | reinterpret_cast<uintptr_t>(dU) |
       reinterpret_cast<uintptr_t>(dC) | reinterpret_cast<uintptr_t>(db)) & 15)
    return RNNLM_ERR_ARG;
  hipStream_t st = (hipStream_t)stream;
  // every entry of dE is written by the output-side contraction; the input rows are then added on top
  UpdateTargets u{dE, dU, nullptr, db, 0.0f, -1.0f, false, false};
  u.A = dA;
  u.C = dC;
  return (h->cfg.precision == RNNLM_FP32) ? window_call<float>(h, x, y, T, logp, nullptr, &u, false, st)
                                          : window_call<bf16_t>(h, x, y, T, logp, nullptr, &u, false, st);
}

int rnnlm_quantize_weights(rnnlm_t *h, const rnnlm_quantized *q, void *stream) {
  if (!h || !q || h->cfg.P <= 0) return RNNLM_ERR_ARG;
  if (!q->qE || !q->sE || !q->qA || !q->sA || !q->qU || !q->sU || !q->qC || !q->sC) return RNNLM_ERR_ARG;
  return (h->cfg.precision == RNNLM_FP32) ? quantize_call<float>(h, *q, (hipStream_t)stream)
                                          : quantize_call<bf16_t>(h, *q, (hipStream_t)stream);
}

namespace {
bool nce_args_ok(rnnlm_t *h, const int32_t *noise, int32_t K, const float *lnq, float lnZ) {
  return h && noise && lnq && K >= 1 && K <= h->cfg.K_max && (lnZ == lnZ);
}
}  // namespace

int rnnlm_nce_train_chunk(rnnlm_t *h, const int32_t *x, const int32_t *y, int32_t T, const int32_t *noise, int32_t K,
                          const float *lnq, float lnZ, float lr, float *J, double *sum_J, void *stream) {
  if (!window_args_ok(h, x, y, T) || !nce_args_ok(h, noise, K, lnq, lnZ) || !(lr == lr)) return RNNLM_ERR_ARG;
  hipStream_t st = (hipStream_t)stream;
  UpdateTargets u{h->buf.E, h->buf.U, h->buf.Wo, h->buf.b, 1.0f, lr, true, true};
  NceCall n{noise, K, lnq, lnZ, J, true};
  return (h->cfg.precision == RNNLM_FP32) ? window_call<float>(h, x, y, T, nullptr, sum_J, &u, true, st, &n)
                                          : window_call<bf16_t>(h, x, y, T, nullptr, sum_J, &u, true, st, &n);
}

int rnnlm_nce_grad_chunk(rnnlm_t *h, const int32_t *x, const int32_t *y, int32_t T, const int32_t *noise, int32_t K,
                         const float *lnq, float lnZ, float *dE, float *dU, float *dWo, float *db, float *J,
                         void *stream) {
  if (!window_args_ok(h, x, y, T) || !nce_args_ok(h, noise, K, lnq, lnZ) || !dE || !dU || !dWo || !db)
    return RNNLM_ERR_ARG;
  if ((reinterpret_cast<uintptr_t>(dE) | reinterpret_cast<uintptr_t>(dU) | reinterpret_cast<uintptr_t>(dWo) |
       reinterpret_cast<uintptr_t>(db)) & 15)
    return RNNLM_ERR_ARG;
  hipStream_t st = (hipStream_t)stream;
  const long nE = (long)h->cfg.V * h->cfg.H;
  const unsigned fb = (unsigned)std::min<long>(blocks_for(nE, 256), 65535);
  hipLaunchKernelGGL(fill_kernel<float>, dim3(fb), dim3(256), 0, st, dE, nE, 0.0f);
  hipLaunchKernelGGL(fill_kernel<float>, dim3(fb), dim3(256), 0, st, dWo, nE, 0.0f);
  hipLaunchKernelGGL(fill_kernel<float>, dim3(blocks_for(h->cfg.V, 256)), dim3(256), 0, st, db, (long)h->cfg.V, 0.0f);
  HIP_TRY(hipGetLastError());
  UpdateTargets u{dE, dU, dWo, db, 0.0f, -1.0f, false, false};
  NceCall n{noise, K, lnq, lnZ, J, true};
  return (h->cfg.precision == RNNLM_FP32) ? window_call<float>(h, x, y, T, nullptr, nullptr, &u, false, st, &n)
                                          : window_call<bf16_t>(h, x, y, T, nullptr, nullptr, &u, false, st, &n);
}

int rnnlm_forward_score(rnnlm_t *h, const int32_t *x, const int32_t *y, int32_t T, float lnZ, float *score,
                        void *stream) {
  if (!window_args_ok(h, x, y, T) || !score || !(lnZ == lnZ)) return RNNLM_ERR_ARG;
  hipStream_t st = (hipStream_t)stream;
  return (h->cfg.precision == RNNLM_FP32) ? score_call<float>(h, x, y, T, lnZ, score, st)
                                          : score_call<bf16_t>(h, x, y, T, lnZ, score, st);
}

int rnnlm_forward_score_shortlist(rnnlm_t *h, const int32_t *x, const int32_t *cand, int32_t C, int32_t T, float lnZ,
                                  float *score, void *stream) {
  if (!h || !x || !cand || !score || T < 1 || T > h->cfg.T_max || C < 1 || C > 65536 || !(lnZ == lnZ))
    return RNNLM_ERR_ARG;
  hipStream_t st = (hipStream_t)stream;
  return (h->cfg.precision == RNNLM_FP32) ? shortlist_call<float>(h, x, cand, C, T, lnZ, score, st)
                                          : shortlist_call<bf16_t>(h, x, cand, C, T, lnZ, score, st);
}

namespace {
bool rms_args_ok(rnnlm_t *h, float lr, float rho, float eps, const rnnlm_rmsprop_state *s) {
  if (!h || !h->cfg.rmsprop || !s || !s->rE || !s->rU || !s->rWo || !s->rb) return false;
  return (lr == lr) && rho >= 0.0f && rho <= 1.0f && eps >= 0.0f;
}
}  // namespace

int rnnlm_train_chunk_rmsprop(rnnlm_t *h, const int32_t *x, const int32_t *y, int32_t T, float lr, float rho,
                              float eps, const rnnlm_rmsprop_state *state, float *logp, double *sum_logp,
                              void *stream) {
  if (!window_args_ok(h, x, y, T) || !rms_args_ok(h, lr, rho, eps, state)) return RNNLM_ERR_ARG;
  hipStream_t st = (hipStream_t)stream;
  // gradients through the plain step's kernels, update epilogues redirected (out = 0*W + 1*g); the
  // embedding rows go to a compact buffer (one row per distinct input word): the hidden-state gradient
  // buffer, which is free once back-propagation through time is done
  float *gWo = reinterpret_cast<float *>(h->ws + h->L.gWo), *gU = reinterpret_cast<float *>(h->ws + h->L.gU),
        *gb = reinterpret_cast<float *>(h->ws + h->L.gb), *gE = reinterpret_cast<float *>(h->ws + h->L.dHs32);
  UpdateTargets u{gE, gU, gWo, gb, 0.0f, -1.0f, false, true, h->Hp};
  const bool f32 = h->cfg.precision == RNNLM_FP32;
  int rc = rms_decay(h, state->rE, nullptr, nullptr, rho, rms_overlaps(h, T, false), st);
  if (rc) return rc;
  hipStream_t rec = nullptr;
  rc = f32 ? window_call<float>(h, x, y, T, logp, sum_logp, &u, true, st, nullptr, &rec)
           : window_call<bf16_t>(h, x, y, T, logp, sum_logp, &u, true, st, nullptr, &rec);
  if (rc) return rc;
  return f32 ? rms_apply<float>(h, T, *state, rho, lr, eps, st, rec)
             : rms_apply<bf16_t>(h, T, *state, rho, lr, eps, st, rec);
}

int rnnlm_nce_train_chunk_rmsprop(rnnlm_t *h, const int32_t *x, const int32_t *y, int32_t T, const int32_t *noise,
                                  int32_t K, const float *lnq, float lnZ, float lr, float rho, float eps,
                                  const rnnlm_rmsprop_state *state, float *J, double *sum_J, void *stream) {
  if (!window_args_ok(h, x, y, T) || !nce_args_ok(h, noise, K, lnq, lnZ) || !rms_args_ok(h, lr, rho, eps, state))
    return RNNLM_ERR_ARG;
  hipStream_t st = (hipStream_t)stream;
  float *gU = reinterpret_cast<float *>(h->ws + h->L.gU), *gE = reinterpret_cast<float *>(h->ws + h->L.dHs32),
        *gN = reinterpret_cast<float *>(h->ws + h->L.gN), *gbN = reinterpret_cast<float *>(h->ws + h->L.gbN);
  // gradients through the plain step's kernels; the touched rows of Wo / entries of b and the embedding rows
  // go to compact one-row-per-word buffers
  UpdateTargets u{gE, gU, gN, gbN, 0.0f, -1.0f, false, true, h->Hp, h->Hp};
  NceCall n{noise, K, lnq, lnZ, J, true};
  const bool f32 = h->cfg.precision == RNNLM_FP32;
  int rc = rms_decay(h, state->rE, state->rWo, state->rb, rho, rms_overlaps(h, T, true), st);
  if (rc) return rc;
  hipStream_t rec = nullptr;
  rc = f32 ? window_call<float>(h, x, y, T, nullptr, sum_J, &u, true, st, &n, &rec)
           : window_call<bf16_t>(h, x, y, T, nullptr, sum_J, &u, true, st, &n, &rec);
  if (rc) return rc;
  return f32 ? rms_apply_nce<float>(h, T, K, *state, rho, lr, eps, st, rec)
             : rms_apply_nce<bf16_t>(h, T, K, *state, rho, lr, eps, st, rec);
}

int rnnlm_reset_state(rnnlm_t *h, void *stream) {
  if (!h) return RNNLM_ERR_ARG;
  const long n = (long)h->cfg.B * h->cfg.H;
  hipLaunchKernelGGL(fill_kernel<float>, dim3(blocks_for(n, 256)), dim3(256), 0, (hipStream_t)stream, h->buf.h_state, n,
                     0.0f);
  HIP_TRY(hipGetLastError());
  return RNNLM_OK;
}

int rnnlm_sync_compute_copies(rnnlm_t *h, void *stream) {
  if (!h) return RNNLM_ERR_ARG;
  return (h->cfg.precision == RNNLM_FP32) ? sync_copies<float>(h, (hipStream_t)stream)
                                          : sync_copies<bf16_t>(h, (hipStream_t)stream);
}

int rnnlm_check(rnnlm_t *h, void *stream) {
  if (!h) return RNNLM_ERR_ARG;
  hipStream_t st = (hipStream_t)stream;
  int32_t flags[3] = {0, 0, 0};
  HIP_TRY(hipMemcpyAsync(flags, p_flags(h), sizeof(flags), hipMemcpyDeviceToHost, st));
  hipLaunchKernelGGL(fill_kernel<int32_t>, dim3(1), dim3(64), 0, st, p_flags(h), 3L, 0);
  HIP_TRY(hipStreamSynchronize(st));
  if (flags[2]) return RNNLM_ERR_TIMEOUT;
  if (flags[0]) return RNNLM_ERR_TOKEN_RANGE;
  if (flags[1]) return RNNLM_ERR_NONFINITE;
  return RNNLM_OK;
}

int rnnlm_perplexity(rnnlm_t *h, const int32_t *tok, int64_t N, int32_t T, double *ppl, int64_t *scored,
                     void *stream) {
  if (!h || !tok || !ppl || N < 2 || T < 1 || T > h->cfg.T_max) return RNNLM_ERR_ARG;
  hipStream_t st = (hipStream_t)stream;
  const int B = h->cfg.B;
  const long L = (long)((N - 1) / B);
  const long nchunks = L / T;
  if (nchunks < 1) return RNNLM_ERR_ARG;
  int rc = rnnlm_reset_state(h, stream);
  if (rc) return rc;
  hipLaunchKernelGGL(fill_kernel<double>, dim3(1), dim3(64), 0, st, p_running(h), 1L, 0.0);
  {
    const LongWindows many(h, T, nchunks);
    int32_t *xt = at<int32_t>(h, h->L.xtmp), *yt = at<int32_t>(h, h->L.ytmp);
    for (long k = 0; k < nchunks; k += many.windows) {
      const int Tn = (int)std::min(many.windows, nchunks - k) * T;
      hipLaunchKernelGGL(stream_chunk_kernel, dim3(blocks_for((long)Tn * B, 256)), dim3(256), 0, st, tok + k * T, L, 0L, Tn, B,
                         xt, yt);
      const long M = (long)Tn * h->Bp, pad = (window_plan(h, M).Mp - M) * h->Hp;
      if (many.windows > 1 && pad > 0) {  // what was there may be anything: rows of states past the positions are operands
        const size_t es = h->cfg.precision == RNNLM_FP32 ? 4 : 2;
        const long n = pad * (long)es / 4;
        hipLaunchKernelGGL(fill_kernel<uint32_t>, dim3(std::min<long>(blocks_for(n, 256), 1024)), dim3(256), 0, st,
                           reinterpret_cast<uint32_t *>(h->ws + h->L.Hs_c + (M + h->Bp) * h->Hp * es), n, 0u);
      }
      const WindowSum ws = {nullptr, p_running(h), p_flags(h), nullptr};
      rc = (h->cfg.precision == RNNLM_FP32)
               ? forward_window<float>(h, xt, yt, Tn, nullptr, true, true, st, false, false, false, &ws)
               : forward_window<bf16_t>(h, xt, yt, Tn, nullptr, true, true, st, false, false, false, &ws);
      if (rc) return rc;
    }
  }
  HIP_TRY(hipGetLastError());
  double total = 0.0;
  HIP_TRY(hipMemcpyAsync(&total, p_running(h), sizeof(double), hipMemcpyDeviceToHost, st));
  rc = rnnlm_check(h, stream);
  if (rc) return rc;
  const long n = nchunks * (long)B * T;
  *ppl = exp(-total / (double)n);
  if (scored) *scored = n;
  if (!(total == total) || total - total != 0.0) return RNNLM_ERR_NONFINITE;
  return RNNLM_OK;
}

int rnnlm_sort_segments(rnnlm_t *h, const int32_t *x, int32_t T, int32_t *perm, int32_t *seg_start, int32_t *nseg,
                        void *stream) {
  if (!h || !x || !perm || !seg_start || !nseg || T < 1 || T > h->cfg.T_max) return RNNLM_ERR_ARG;
  hipStream_t st = (hipStream_t)stream;
  const int Mp = (int)round_up((long)T * h->Bp, PAD_M);
  const int prep_blocks = (int)blocks_for(Mp, 256);
  PrepWindow<float> pw = {};
  pw.x = x;
  pw.Tn = T;
  pw.B = h->cfg.B;
  pw.Bp = h->Bp;
  pw.Mp = Mp;
  pw.V = h->cfg.V;
  pw.xp = at<int32_t>(h, h->L.xp);
  pw.lse = at<float>(h, h->L.lse);
  pw.flags = p_flags(h);
  pw.prep_blocks = prep_blocks;
  hipLaunchKernelGGL(prep_tokens_kernel<float>, dim3(prep_blocks), dim3(256), 0, st, pw);
  HIP_TRY(hipGetLastError());
  return sort_segments<float>(h, T, perm, seg_start, nseg, st);
}

// ---- the entry point that allocates nothing ----------------------------------------------------------------
namespace {
constexpr int STATIC_MAX_POSITIONS = 65536;  // padded window positions the static scratch holds
struct StaticScratch {
  int32_t xp[STATIC_MAX_POSITIONS];  // padded, range-checked ids
  float lse[STATIC_MAX_POSITIONS];   // the token-preparation kernel marks padded positions here
  int32_t flags[64];                 // [0]: an id was out of range
};
constexpr int STATIC_MAX_DEVICES = 64;
}  // namespace
// One copy per GPU, held until the process ends.  In host code this name is only a handle for
// hipGetSymbolAddress: kernels get the address that call returns for the current device.
static __device__ __align__(256) unsigned char scratch[sizeof(StaticScratch)];
namespace {
std::mutex static_mutex;
StaticScratch *static_ptr[STATIC_MAX_DEVICES] = {nullptr};

// Address of the current device's copy of the scratch array (asked once per device, with that device current).
int static_scratch(StaticScratch **out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return RNNLM_ERR_HIP;
  if (dev < 0 || dev >= STATIC_MAX_DEVICES) return RNNLM_ERR_ARG;
  std::lock_guard<std::mutex> lock(static_mutex);
  if (!static_ptr[dev]) {
    void *p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return RNNLM_ERR_HIP;
    static_ptr[dev] = static_cast<StaticScratch *>(p);
  }
  *out = static_ptr[dev];
  return RNNLM_OK;
}

// Hands the range flag to the caller (when asked for) and clears it for the next call.
__global__ void static_flag_kernel(int32_t *flags, int32_t *range_flag) {
  if (threadIdx.x == 0) {
    if (range_flag) *range_flag = flags[0] ? 1 : 0;
    flags[0] = 0;
  }
}
}  // namespace

int rnnlm_sort_segments_static(const int32_t *x, int32_t T, int32_t B, int32_t V, int32_t *perm, int32_t *seg_start,
                               int32_t *nseg, int32_t *range_flag, void *stream) {
  if (!x || !perm || !seg_start || !nseg || T < 1 || B < 1 || V < 1) return RNNLM_ERR_ARG;
  const long Bp = round_up(B, PAD_B);
  const long Mp = round_up((long)T * Bp, PAD_M);
  if (Mp > STATIC_MAX_POSITIONS) return RNNLM_ERR_ARG;  // beyond what the static scratch holds
  StaticScratch *sc = nullptr;
  int rc = static_scratch(&sc);
  if (rc) return rc;
  hipStream_t st = (hipStream_t)stream;
  const int M = T * B;
  const int prep_blocks = (int)blocks_for(Mp, 256);
  // the array keeps the previous call's contents: the flag starts at zero, the ids of all Mp positions are rewritten
  hipLaunchKernelGGL(fill_kernel<int32_t>, dim3(1), dim3(64), 0, st, sc->flags, 64L, 0);
  PrepWindow<float> pw = {};
  pw.x = x;
  pw.Tn = T;
  pw.B = B;
  pw.Bp = (int)Bp;
  pw.Mp = (int)Mp;
  pw.V = V;
  pw.xp = sc->xp;
  pw.lse = sc->lse;
  pw.flags = sc->flags;
  pw.prep_blocks = prep_blocks;
  hipLaunchKernelGGL(prep_tokens_kernel<float>, dim3(prep_blocks), dim3(256), 0, st, pw);
  hipLaunchKernelGGL(rank_sort_kernel, dim3(blocks_for(M, 64)), dim3(1024), 0, st, sc->xp, M, B, (int)Bp, perm);
  hipLaunchKernelGGL(segment_kernel, dim3(1), dim3(1024), 0, st, sc->xp, perm, M, B, (int)Bp, seg_start, nseg);
  hipLaunchKernelGGL(static_flag_kernel, dim3(1), dim3(64), 0, st, sc->flags, range_flag);
  HIP_TRY(hipGetLastError());
  return RNNLM_OK;
}

int rnnlm_set_barrier_spin_limit(rnnlm_t *h, uint32_t polls) {
  if (!h || polls == 0) return RNNLM_ERR_ARG;
  h->spin_limit = polls;
  return RNNLM_OK;
}

int rnnlm_set_recurrent_exchange(rnnlm_t *h, int32_t mode) {
  if (!h) return RNNLM_ERR_ARG;
  if (mode != RNNLM_EXCHANGE_AUTO && mode != RNNLM_EXCHANGE_CHIP_WIDE && mode != RNNLM_EXCHANGE_XCD_LOCAL)
    return RNNLM_ERR_ARG;
  // the XCD-local exchange needs the placement the probe at init looks for and at most one block of 32 streams per XCD
  if (mode == RNNLM_EXCHANGE_XCD_LOCAL && !(h->xcd_local && round_up(h->cfg.B, PAD_B) / 32 <= NUM_XCD)) return RNNLM_ERR_ARG;
  h->exchange_mode = mode;
  return RNNLM_OK;
}

int rnnlm_measure_peaks(rnnlm_t *h, double *mfma_bf16_random_tflops, double *mfma_bf16_constant_tflops,
                        double *copy_gbs, void *stream) {
  if (!h || !mfma_bf16_random_tflops || !mfma_bf16_constant_tflops || !copy_gbs) return RNNLM_ERR_ARG;
  hipStream_t st = (hipStream_t)stream;
  hipEvent_t e0, e1;
  HIP_TRY(hipEventCreate(&e0));
  HIP_TRY(hipEventCreate(&e1));
  // scratch: the logits buffer (rewritten by the next window's forward pass before anything reads it)
  const size_t es = (h->cfg.precision == RNNLM_FP32) ? 4 : 2;
  char *scratch = h->ws + h->L.ZT;
  const size_t avail = (size_t)h->Vp * h->MpMax * es;
  int rc = RNNLM_OK;
  auto timed = [&](auto launch, double &ms_out) {
    launch();  // warm-up
    if (hipEventRecord(e0, st) != hipSuccess) rc = RNNLM_ERR_HIP;
    launch();
    if (hipEventRecord(e1, st) != hipSuccess || hipEventSynchronize(e1) != hipSuccess) rc = RNNLM_ERR_HIP;
    float ms = 0.0f;
    if (hipEventElapsedTime(&ms, e0, e1) != hipSuccess) rc = RNNLM_ERR_HIP;
    ms_out = ms;
  };
  const int iters = 50000;
  const double mfma_flops = 256.0 * 8 * iters * 8 * 32.0 * 32 * 16 * 2;
  double ms = 0.0;
  *mfma_bf16_random_tflops = *mfma_bf16_constant_tflops = *copy_gbs = 0.0;
  if (avail >= 256 * 512 * sizeof(float)) {
    float *out = reinterpret_cast<float *>(scratch);
    timed([&] { hipLaunchKernelGGL(mfma_rate_kernel<true>, dim3(256), dim3(512), 0, st, out, iters); }, ms);
    if (rc == RNNLM_OK && ms > 0) *mfma_bf16_random_tflops = mfma_flops / ms / 1e9;
    timed([&] { hipLaunchKernelGGL(mfma_rate_kernel<false>, dim3(256), dim3(512), 0, st, out, iters); }, ms);
    if (rc == RNNLM_OK && ms > 0) *mfma_bf16_constant_tflops = mfma_flops / ms / 1e9;
  }
  const size_t half = (avail / 2) & ~(size_t)255;
  if (half >= (8u << 20)) {
    const long n16 = (long)(half / 16);
    timed([&] {
      hipLaunchKernelGGL(copy_kernel, dim3(256 * 32), dim3(256), 0, st, reinterpret_cast<const u32x4_t *>(scratch),
                         reinterpret_cast<u32x4_t *>(scratch + half), n16);
    }, ms);
    if (rc == RNNLM_OK && ms > 0) *copy_gbs = 2.0 * half / ms / 1e6;  // read + write
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (rc == RNNLM_OK && hipGetLastError() != hipSuccess) rc = RNNLM_ERR_HIP;
  return rc;
}

int rnnlm_profile_enable(rnnlm_t *h, uint32_t stage_mask) {
  if (!h || stage_mask >= (1u << RNNLM_STAGE_COUNT)) return RNNLM_ERR_ARG;
  h->prof_mask = stage_mask;
  return RNNLM_OK;
}

int rnnlm_profile_read(rnnlm_t *h, int32_t stage, double *total_ms, int64_t *executions) {
  if (!h || stage < 0 || stage >= RNNLM_STAGE_COUNT || !total_ms || !executions) return RNNLM_ERR_ARG;
  for (size_t i = 0; i < h->prof_used; ++i) {
    EventPair &e = h->prof_pool[i];
    HIP_TRY(hipEventSynchronize(e.stop));
    float ms = 0.0f;
    HIP_TRY(hipEventElapsedTime(&ms, e.start, e.stop));
    h->prof_ms[e.stage] += ms;
    h->prof_n[e.stage] += 1;
  }
  h->prof_used = 0;
  *total_ms = h->prof_ms[stage];
  *executions = h->prof_n[stage];
  h->prof_ms[stage] = 0.0;
  h->prof_n[stage] = 0;
  return RNNLM_OK;
}

const char *rnnlm_status_string(int status) {
  switch (status) {
    case RNNLM_OK: return "ok";
    case RNNLM_ERR_ARG: return "invalid argument";
    case RNNLM_ERR_TOKEN_RANGE: return "token id out of range";
    case RNNLM_ERR_NONFINITE: return "non-finite log-probability sum";
    case RNNLM_ERR_HIP: return "HIP runtime error";
    case RNNLM_ERR_NOMEM: return "host allocation failed";
    case RNNLM_ERR_TIMEOUT: return "grid barrier wait expired";
    default: return "unknown status";
  }
}

}  // extern "C"
