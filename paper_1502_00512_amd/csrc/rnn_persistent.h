// Persistent recurrent kernel: all T dependent timesteps of a window in ONE launch, with the state-to-state matrix
// held in registers for the whole window (Sec. 4.2 marshals the state-to-state work into one large matrix product; on
// this hardware the serial chain is latency-bound instead, so the matrix stays on chip and only the B x H state
// travels between steps).
//
// Decomposition: workgroup (group, ub) owns R <= 32 streams x 16 UT hidden units.  Its NWAVE waves split the
// contraction dimension in whole blocks of 32 values; each keeps its share of its units' rows of U (forward; backward:
// of U^T) as MFMA operand fragments in registers, loads the matching part of the previous step's state straight from
// the L2 into operand fragments, and the NWAVE partial tiles are summed through LDS.
//
// Exchange without a barrier.  The step is a chain of latencies (2.6 us at H = 1024 with a counter barrier: state copy
// and contraction 1.0, barrier 0.8, partial sums 0.2, elementwise part, store and its acknowledgement 0.45), so the
// data is its own flag: a word of the exchange buffer that its step has not written holds UNWRITTEN (all bits set, which
// the kernel itself never stores), and a wave reloads its fragments until no word of them is UNWRITTEN.  A word is
// written by one store of one lane, so it is either old or new.  Store, acknowledgement, arrival, poll and load become
// store and load, and a wave waits only for the units it contracts over.
//
// The exchange buffer is a ring of RING = 4 steps' states in operand order: the fragment of 16 streams x 32 values is
// one contiguous kilobyte (fp32: two), lane l's 16 bytes at 16 l.  (Loaded from the row-major state instead, adjacent
// lanes ask for different rows and the vector L1 looks every lane up by itself: 2.0 us per step at 128 streams.)
// At step t a thread sets its words of step t - 2 back to UNWRITTEN.  It may: the barrier inside step t follows the
// arrival of every workgroup's step t - 1, each of which had read step t - 2 before.  The reset is in place before step
// t + 2 is stored there and polled: the wave waits for its own stores at its next poll, before it stores step t + 1, and
// a reader polls for a wave's step t + 2 only after it has that wave's step t + 1.
//
// Measured (bf16, per step, forward / backward): H = 1024, one stream 0.93 / 0.94 us, 128 streams 1.24 / 0.97 (with the
// counter barrier 2.4 / 2.8), 256 streams 1.8 / 1.6; H = 2048, 128 streams 2.6 / 2.5 (4.5 / 5.9); fp32, H = 1024, 128
// streams 3.2 / 2.8 (9.2 / 10.4).  What is left is latency: an L2 round trip and a half for the wait, the contraction,
// one LDS exchange and the elementwise part.
#pragma once
#include <type_traits>

#include "common.h"
#include "gemm.h"
#include "gemm_dma.h"
#include "kernels.h"

namespace rnnlm_dev {

struct RnnPersistArgs {
  const void *W;      // forward: U_c [Hp][Hp]; backward: UT_c [Hp][Hp] (row n holds the k-contiguous operand)
  void *Hs;           // hidden-state slots [(T+1)][Bp][Hp] (slot 0 = carried state)
  const float *X;     // forward: gathered embeddings [T][Bp][Hp]; backward: dHs [T][Bp][Hp]
  float *dA32;        // backward: [T][Bp][Hp]
  void *dAc;          // backward: [T][Bp][Hp] compute type
  float *h_state;     // forward: [B][H] or nullptr
  unsigned *counter;  // SYNC_WORDS barrier / ticket counters, zero at launch (see sync_word)
  int32_t *flags;     // flags[2] raised when a wait expires
  int T, B, H, Bp, Hp;
  unsigned spin_limit;
  // rnn_persistent_kernel: streams per group, groups, workgroups per group, 32-wide blocks of the contraction and how
  // many of them a wave takes; xcd: one group per XCD (see below)
  int R, groups, nwg, nkb, ks, xcd;
  void *ring;  // exchange buffer: [RING][groups][RT][nkb] fragments
};

// Where the exchanged words travel.  The workgroups that exchange state with one another are exactly those of one
// group of streams.
// XCD-local mode: such a group runs on ONE accelerator die (XCD) and shares its L2; plain stores (the vector L1 is
// write-through) and loads with the agent-scope policy, which bypass the L1, need nothing beyond that L2.  Placement
// does not rely on the dispatch order: every workgroup reads the id of the XCD it runs on, groups are bound to XCDs
// (group x <-> XCD x), and a per-XCD ticket counter hands out the unit blocks; surplus workgroups and those on XCDs
// without a group exit at once.  The host enables this mode only after a probe launch has shown that an 8*n grid lands
// n workgroups on each XCD.
// Chip-wide mode: stores with agent-scope relaxed atomics, which carry the agent-scope cache policy on the access
// itself, and the same loads.
// The values and the order of every sum are the same in both modes and for any R.
__device__ inline int xcc_id() { return __builtin_amdgcn_s_getreg((3 << 11) | 20) & 15; }  // HW_REG_XCC_ID[3:0]

// Release half of a step barrier, executed by every wave: a workgroup-scope release fence only drains the
// LDS/scalar counter on this target, so the wave also waits until each of its vector-memory stores has been
// acknowledged (vmcnt counts stores as well as loads here); only then may the workgroup signal its arrival.
__device__ inline void wait_own_stores() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
}

__device__ inline void coherent_store64(void *p, unsigned long long v) {
  __hip_atomic_store(reinterpret_cast<unsigned long long *>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// 4 consecutive values, agent-scope accesses.
template <typename T>
__device__ inline void store4(T *p, const f32x4_t &v);
template <>
__device__ inline void store4<bf16_t>(bf16_t *p, const f32x4_t &v) {
  union {
    unsigned long long q;
    bf16x4_t h;
  } u;
#pragma unroll
  for (int e = 0; e < 4; ++e) u.h[e] = (bf16_t)v[e];
  coherent_store64(p, u.q);
}

// V consecutive values as the words of the exchanged state.  A word never equals UNWRITTEN: one whose value would
// (NaNs with every bit set) becomes another NaN.
template <typename T, int V>
struct StateWords {
  static constexpr int N = V * (int)sizeof(T) / 4;
  unsigned w[N];
  __device__ inline void pack(const float (&v)[V]) {
    if constexpr (sizeof(T) == 4) {
#pragma unroll
      for (int e = 0; e < N; ++e) w[e] = min(__builtin_bit_cast(unsigned, v[e]), UNWRITTEN - 1u);
    } else {
      typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
#pragma unroll
      for (int e = 0; e < N; ++e) {
        bf16x2_t h;
        h[0] = (bf16_t)v[2 * e];
        h[1] = (bf16_t)v[2 * e + 1];
        w[e] = min(__builtin_bit_cast(unsigned, h), UNWRITTEN - 1u);
      }
    }
  }
  __device__ inline void store(unsigned *q, bool plain) const {
    if (plain) {
      if constexpr (N == 1) {
        *q = w[0];
      } else {
        typedef unsigned words_t __attribute__((ext_vector_type(N)));
        words_t t;
#pragma unroll
        for (int e = 0; e < N; ++e) t[e] = w[e];
        *reinterpret_cast<words_t *>(q) = t;
      }
    } else {
#pragma unroll
      for (int e = 0; e < N; ++e) __hip_atomic_store(q + e, w[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
};

// Operand fragment of one 16-row block and one 32-wide block of k: lane l holds row l % 16 and k = 8 (l / 16) .. +7.
template <typename T>
struct StepFrag {
  static constexpr int LOADS = 8 * (int)sizeof(T) / 16;  // 16-byte pieces
  u32x4_t q[LOADS];
};
// acc[0] and acc[1] are two accumulation chains of one 16 x 16 tile (consecutive MFMAs do not wait for one another).
// fp32: the e-th 16x16x4 instruction contracts k = e, 8 + e, 16 + e and 24 + e.
__device__ inline void mma_block(f32x4_t (&acc)[2], int kk, const StepFrag<bf16_t> &a, const StepFrag<bf16_t> &b) {
  acc[kk & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a.q[0]),
                                                        __builtin_bit_cast(bf16x8_t, b.q[0]), acc[kk & 1], 0, 0, 0);
}
__device__ inline void mma_block(f32x4_t (&acc)[2], int, const StepFrag<float> &a, const StepFrag<float> &b) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const f32x4_t av = __builtin_bit_cast(f32x4_t, a.q[i]), bv = __builtin_bit_cast(f32x4_t, b.q[i]);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[e], bv[e], acc[e & 1], 0, 0, 0);
  }
}

// Exchange buffer of one direction: [RING][groups][RT][nkb][LOADS] pieces of a kilobyte.  Piece i of the fragment of
// (16 streams, 32 units) holds, for lane l, the units 8 (l / 16) + i * 16 / sizeof(T) .. of stream l % 16.
// (RING, UNWRITTEN and the first contents: prep_tokens_kernel.)

// BACKWARD = false: h_t = sigmoid(X_t + h_{t-1} U^T) for t = 0..T-1.  BACKWARD = true: dA_t = (dHs_t + dA_{t+1} U) *
// h_t * (1 - h_t) for t = T-1..0.
// KS = blocks of 32 contraction values a wave has registers for (it takes a.ks of them); RT = 16-row blocks of streams.
// Four waves and 32 units up to 1024 units; eight waves and 64 units (bf16) up to 2048: at most 32 workgroups per group,
// one per compute unit of an XCD.
// The host guarantees that the grid is small enough to be co-resident; every wait is bounded: on expiry flags[2] is
// raised, the wave waits no more and the kernel runs to its end.
// Two handles' kernels are certain to fit the device together where a wave takes at most 168 of the 512 registers a SIMD
// lane has (three waves): one of 200 can start, next to a wave of another kernel that ends later, where neither side of
// it has room for a second, and then both handles' waits expired.  rnn_pairs: the forms held to that (no form is slower
// for it: fp32, H = 512, 256 streams, a 20-step scoring call 82.5 us, before 83.5).
template <typename T, int KS, int NWAVE, int RT>
constexpr bool rnn_pairs() {
  return NWAVE == 4 && (sizeof(T) == 2 ? RT == 1 || KS <= 6 : KS <= 4);
}
template <typename T, int KS, int NWAVE, int UT, int RT, bool BACKWARD>
__global__ void __launch_bounds__(64 * NWAVE, (rnn_pairs<T, KS, NWAVE, RT>() ? 3 : 1)) rnn_persistent_kernel(const RnnPersistArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int ES = sizeof(T);
  constexpr int V = RT * UT * 4 / NWAVE;  // consecutive units per thread in the elementwise part
  constexpr int TPS = UT * 16 / V;        // threads per stream there
  constexpr int LOADS = StepFrag<T>::LOADS;
  constexpr int TILE = 256;               // floats of a partial 16 x 16 tile
  __shared__ __attribute__((aligned(16))) float red[2][NWAVE * RT * UT * TILE];
  __shared__ int s_ticket;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int group, ub;
  if (a.xcd) {
    group = xcc_id();
    if (group >= a.groups) return;  // no group lives on this XCD
    if (tid == 0)
      s_ticket = (int)__hip_atomic_fetch_add(a.counter + sync_word(2, group), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    ub = __builtin_amdgcn_readfirstlane(s_ticket);
    if (ub >= a.nwg) return;  // surplus workgroup
  } else {
    group = blockIdx.x % a.groups;
    ub = blockIdx.x / a.groups;
  }
  const int Hp = a.Hp;
  const long slot = (long)a.Bp * Hp;
  const int kb0 = wave * a.ks;                          // first block of this wave
  const int nk = min(a.ks, a.nkb - kb0);                // its blocks (not positive: none)
  const int lr = lane & 15, lk = (lane >> 4) * 8;

  // this wave's slice of the matrix, resident in registers for all T steps
  StepFrag<T> w[UT][KS];
#pragma unroll
  for (int u = 0; u < UT; ++u) {
    const T *Wp = static_cast<const T *>(a.W) + (long)(ub * (UT * 16) + u * 16 + lr) * Hp + kb0 * 32 + lk;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk)
#pragma unroll
      for (int i = 0; i < LOADS; ++i)
        w[u][kk].q[i] = kk < nk ? *reinterpret_cast<const u32x4_t *>(Wp + kk * 32 + i * (16 / ES)) : u32x4_t{0u, 0u, 0u, 0u};
  }
  const int row0 = group * a.R;
  const int nrow = min(a.R, a.B - row0);
  // this lane's 16 bytes of a piece; rows past the group's streams repeat its last one (their products are unused)
  char *const ring = static_cast<char *>(a.ring) + (long)group * (RT * LOADS * 1024) * a.nkb;
  const long ring_slot = (long)a.groups * (RT * LOADS * 1024) * a.nkb;
  int voff[RT];
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    const int er = min(r * 16 + lr, nrow - 1);
    voff[r] = (er >> 4) * a.nkb * (LOADS * 1024) + ((lane & 48) + (er & 15)) * 16;
  }
  // elementwise part: this thread's stream and its V consecutive units
  const int es = tid / TPS, eu = (tid % TPS) * V;
  const int erow = row0 + es, ecol = ub * (UT * 16) + eu;
  const bool row_ok = es < nrow;
  const long ebase = (long)erow * Hp + ecol, ebase_in = (long)(row_ok ? erow : row0) * Hp + ecol;
  const int red_at = ((es >> 4) * UT + (eu >> 4)) * TILE + ((((eu >> 2) & 3) << 4) + ((es & 15) ^ (eu & 12))) * 4 + (eu & 3);
  const int ring_at = (((es >> 4) * a.nkb + (ecol >> 5)) * LOADS + (ES == 4 ? (eu >> 2) & 1 : 0)) * 1024 +
                      (((ecol >> 3) & 3) * 16 + (es & 15)) * 16 + (ecol * ES & 15);
  T *Hs = static_cast<T *>(a.Hs);
  T *dAc = static_cast<T *>(a.dAc);
  typedef float fv_t __attribute__((ext_vector_type(V)));
  typedef unsigned hv_t __attribute__((ext_vector_type(StateWords<T, V>::N)));
  struct Operands {  // of one step's elementwise part, as loaded (unpacked at once, they would be waited for at once)
    fv_t x;
    hv_t h;
  };
  auto request = [&](int t, Operands &o) {
    const long at = (long)t * slot + ebase_in;
    o.x = *reinterpret_cast<const fv_t *>(a.X + at);
    if (BACKWARD) o.h = *reinterpret_cast<const hv_t *>(Hs + slot + at);
  };
  // A step's rows of the state (gradient) leave after the next step's wait: in front of it, the wait would be for their
  // acknowledgement as well.
  struct Result {
    StateWords<T, V> words;
    float v[V];
  } last;
  auto flush = [&](int t) {
    if (!row_ok) return;
    const long at = (long)t * slot + ebase;
    last.words.store(reinterpret_cast<unsigned *>((BACKWARD ? dAc : Hs + slot) + at), true);
    if (BACKWARD) {
      fv_t d;
#pragma unroll
      for (int e = 0; e < V; ++e) d[e] = last.v[e];
      *reinterpret_cast<fv_t *>(a.dA32 + at) = d;
    }
  };
  // The same for all lanes: said so, or every access through it becomes a loop over lanes.
  auto uniform = [](char *p) {
    const unsigned long long v = reinterpret_cast<unsigned long long>(p);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
    return reinterpret_cast<char *>(((unsigned long long)hi << 32) | lo);
  };
  int expired = 0;
  // row blocks whose fragments fit the registers at once (fp32, KS = 3 and 4: at two, 174 and 206 registers)
  constexpr int RB = NWAVE == 8 || (ES == 4 && KS >= 3 && KS <= 4) ? 1 : RT;
  StepFrag<T> f[RB][KS];
  auto step_of = [&](auto first, int step_, Operands &now, Operands &next) {
    const int step = __builtin_amdgcn_readfirstlane(step_);
    const int t = BACKWARD ? a.T - 1 - step : step;
    constexpr bool contract = !(BACKWARD && first.value);  // nothing flows into the window's last position
    // partial tiles through LDS: lane l holds units 4 (l / 16) .. +3 of stream l % 16.  Two buffers, one barrier per
    // step: a wave writes a buffer again only after the barrier of the step between, which follows every read of it.
    float *rd = red[step & 1];
    auto hand_over = [&](int r, int u, const f32x4_t &v) {
      *reinterpret_cast<f32x4_t *>(rd + ((wave * RT + r) * UT + u) * TILE +
                                   ((lane & 48) + (lr ^ ((lane >> 4) << 2))) * 4) = v;
    };
    if constexpr (contract) {
      // (a block past this wave's share reads through a resource without extent: zeros, no memory access)
      char *const src = uniform(ring + (long)((step - 1) & (RING - 1)) * ring_slot + kb0 * (LOADS * 1024));
      // (what step 0 reads was written before the launch)
      const unsigned limit = first.value ? 0u : __builtin_amdgcn_readfirstlane(expired ? 0u : a.spin_limit);
#pragma unroll
      for (int r0 = 0; r0 < RT; r0 += RB) {
        f32x4_t acc[RB][UT][2];
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
          for (int u = 0; u < UT; ++u) acc[r][u][0] = acc[r][u][1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        unsigned spins = 0;
        bool missing;
        do {
          asm volatile("" ::: "memory");  // these loads are new ones
#pragma unroll
          for (int kk = 0; kk < KS; ++kk) {
            const __amdgpu_buffer_rsrc_t rs =
                __builtin_amdgcn_make_buffer_rsrc(src, 0, kk < nk ? 0x7fffffff : 0, 0x00020000);
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
              for (int i = 0; i < LOADS; ++i)
                f[r][kk].q[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, voff[r0 + r], (kk * LOADS + i) * 1024, 16 /* sc1 */);
          }
          unsigned m = 0u;
#pragma unroll
          for (int kk = 0; kk < KS; ++kk)
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
              for (int i = 0; i < LOADS; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) m = max(m, f[r][kk].q[i][e]);
          missing = __builtin_amdgcn_ballot_w64(m == UNWRITTEN) != 0;
        } while (missing && ++spins < limit);
        if (missing && limit > 0) {
          expired = 1;
          if (lane == 0) a.flags[2] = 1;
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the reset of the step before is in place as well
        // the next step's operands of the elementwise part: their latency passes behind this step and the next wait
        if (r0 + RB == RT && step + 1 < a.T) request(BACKWARD ? t - 1 : t + 1, next);
        if (r0 + RB == RT && !first.value) flush(BACKWARD ? t + 1 : t - 1);
#pragma unroll
        for (int kk = 0; kk < KS; ++kk)
#pragma unroll
          for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int u = 0; u < UT; ++u) mma_block(acc[r][u], kk, w[u][kk], f[r][kk]);
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
          for (int u = 0; u < UT; ++u) hand_over(r0 + r, u, acc[r][u][0] + acc[r][u][1]);
      }
    } else {
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int u = 0; u < UT; ++u) hand_over(r, u, f32x4_t{0.f, 0.f, 0.f, 0.f});
      if (step + 1 < a.T) {
        __builtin_amdgcn_s_waitcnt(0x0F70);  // as above: step 0's own operands would be waited for together with the next ones
        request(BACKWARD ? t - 1 : t + 1, next);
      }
    }
    __syncthreads();
    float s[V];
#pragma unroll
    for (int e = 0; e < V; ++e) s[e] = rd[red_at + e];
#pragma unroll
    for (int q = 1; q < NWAVE; ++q)
#pragma unroll
      for (int e = 0; e < V; ++e) s[e] += rd[q * (RT * UT * TILE) + red_at + e];
    if (!row_ok) return;
    float(&o)[V] = last.v;
    float now_h[V] = {};
    if (BACKWARD) {
      typedef T tv_t __attribute__((ext_vector_type(V)));
      const tv_t h = __builtin_bit_cast(tv_t, now.h);
#pragma unroll
      for (int e = 0; e < V; ++e) now_h[e] = to_f32(h[e]);
    }
#pragma unroll
    for (int e = 0; e < V; ++e)
      o[e] = BACKWARD ? (now.x[e] + s[e]) * now_h[e] * (1.0f - now_h[e]) : sigmoidf_(s[e] + now.x[e]);
#pragma unroll
    for (int e = 0; e < V; ++e) o[e] = ecol + e < a.H ? o[e] : 0.0f;
    last.words.pack(o);
    if (step + 1 < a.T) last.words.store(reinterpret_cast<unsigned *>(ring + (long)(step & (RING - 1)) * ring_slot + ring_at), a.xcd);
    if (!first.value && step + 2 < a.T) {
      StateWords<T, V> none;
#pragma unroll
      for (int e = 0; e < none.N; ++e) none.w[e] = UNWRITTEN;
      none.store(reinterpret_cast<unsigned *>(ring + (long)((step - 2) & (RING - 1)) * ring_slot + ring_at), a.xcd);
    }
    if (!BACKWARD && a.h_state && step == a.T - 1) {
#pragma unroll
      for (int e = 0; e < V; ++e)
        if (ecol + e < a.H) a.h_state[(long)erow * a.H + ecol + e] = o[e];
    }
  };
  Operands even, odd;
  request(BACKWARD ? a.T - 1 : 0, even);
  step_of(std::true_type{}, 0, even, odd);
  for (int step = 1; step < a.T; step += 2) {
    step_of(std::false_type{}, step, odd, even);
    if (step + 1 < a.T) step_of(std::false_type{}, step + 1, even, odd);
  }
  flush(BACKWARD ? 0 : a.T - 1);
#endif
}

// Records which XCD each workgroup of the launch runs on.
__global__ void xcd_probe_kernel(int32_t *out) {
  if (threadIdx.x == 0) out[blockIdx.x] = xcc_id();
}

}  // namespace rnnlm_dev
