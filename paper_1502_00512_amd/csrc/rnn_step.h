// One timestep of the recurrence in one launch, for layers wider than the persistent kernel takes.
//
// A step of few streams reads the whole state-to-state matrix once and does little with it.  As a contraction split over
// workgroups and a pass that adds up the parts it is two launches, each mostly latency, and the parts' way through the
// caches between them.  Here a workgroup owns 16 units x 16 RT streams and the whole contraction dimension: its eight waves
// share it out, and each wave moves its own pieces (16 rows x 128 bytes of the matrix and of the states) straight from global
// memory into a ring of LDS of its own and reads operand fragments from there.  Nothing in the loop waits for another wave;
// partial tiles are added through LDS at the end and the first RT waves apply the elementwise part.
// (Fragments loaded straight into registers: adjacent lanes ask for different rows, which the vector L1 looks up lane by
// lane, 120 cycles a load; a step of 16 streams at H = 2816 took twice as long.)
#pragma once
#include "gemm_dma4.h"
#include "rnn_persistent.h"

namespace rnnlm_dev {

//
// The same contraction by itself (STEP_STORE, STEP_STORE32): the inserted layers of the compressed architecture over the few
// positions of a scored text (P = 512, H = 1024, 20 positions: 5.2 and 7.2 us on 64x64 tiles, whose workgroups walk 16 and 32
// blocks one after the other; scoring call 43.0 and 37.6).  It writes whole rows: columns past the units become zeros, which
// the contractions that follow read.
enum : int { STEP_FORWARD, STEP_BACKWARD, STEP_STORE, STEP_STORE32 };

struct RnnStepArgs {
  const void *W;      // forward: U_c [Hp][Hp]; backward: UT_c [Hp][Hp] (row n holds the k-contiguous operand)
  const void *state;  // rows [B][lds] that are contracted: previous states, or the gradients of the next position
  const float *X;     // forward: additive input; backward: gradient from the output layer; [B][Hp]
  const void *h;      // backward: states of the position [B][Hp]
  void *out;          // compute type [B][Hp]: new states, or gradients
  float *out32;       // backward: gradients in fp32
  float *h_state;     // forward: [B][H] or nullptr
  int B, H, Hp;       // rows, units, row length of what is written
  int lds;            // row length of the operands (Hp, where they are states)
  int pieces;         // 128-byte pieces of a row that are contracted (0: nothing flows in)
};

template <typename T, int RT, int MODE>
__global__ void __launch_bounds__(512) rnn_step_kernel(const RnnStepArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int ES = sizeof(T), NWAVE = 8;
  constexpr bool BACKWARD = MODE == STEP_BACKWARD, STORE = MODE == STEP_STORE || MODE == STEP_STORE32;
  constexpr int DEPTH = RT == 1 ? 4 : RT == 2 ? 3 : 2;   // pieces of a wave in flight (what the LDS holds)
  constexpr int PIECE = 2048, SLOT = (1 + RT) * PIECE;   // 16 rows x 128 bytes; matrix, then RT row blocks of states
  constexpr int LOADS = 2 * (1 + RT);                    // a piece is two kilobyte loads
  static_assert(DEPTH >= 2 && DEPTH <= 4 && (DEPTH - 1) * LOADS <= 63, "the counted waits below");  // 12, 12 and 10 loads
  static_assert(NWAVE * RT * 1024 <= NWAVE * DEPTH * SLOT, "the partial tiles reuse the ring");
  __shared__ __attribute__((aligned(1024))) char lds[NWAVE * DEPTH * SLOT];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, Hp = a.Hp;
  const int unit0 = blockIdx.x * 16, row0 = blockIdx.y * (16 * RT);

  // elementwise part: wave r of the first RT, stream 16 r + lane % 16, units 4 (lane / 16) .. +3
  const int erow = row0 + wave * 16 + lr, ecol = unit0 + (lane >> 4) * 4;
  const bool mine = wave < RT && erow < a.B;
  f32x4_t x = {0.0f, 0.0f, 0.0f, 0.0f};
  typedef T tv_t __attribute__((ext_vector_type(4)));
  tv_t hv = {};
  if (mine && !STORE) {
    x = *reinterpret_cast<const f32x4_t *>(a.X + (long)erow * Hp + ecol);
    if (BACKWARD) hv = *reinterpret_cast<const tv_t *>(static_cast<const T *>(a.h) + (long)erow * Hp + ecol);
  }

  // this wave's pieces: first .. first + n - 1
  const int pieces = unit0 < a.H ? a.pieces : 0;  // (columns past the units: zeros)
  const int base = pieces / NWAVE, more = pieces % NWAVE;
  const int n = base + (wave < more), first = wave * base + min(wave, more);
  f32x4_t acc[RT][2];
#pragma unroll
  for (int r = 0; r < RT; ++r) acc[r][0] = acc[r][1] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
  if (n > 0) {
    char *const ring = lds + wave * (DEPTH * SLOT);
    // a load takes 8 rows of whole 128-byte lines; chunks are swizzled as in gemm_dma.h (rows of 128 bytes)
    typedef int i32x4_t __attribute__((ext_vector_type(4)));
    auto resource = [](const char *p, long bytes) {
      const unsigned long long b = reinterpret_cast<unsigned long long>(p);
      i32x4_t r;
      r[0] = __builtin_amdgcn_readfirstlane((int)(unsigned)b);
      r[1] = __builtin_amdgcn_readfirstlane((int)(unsigned)((b >> 32) & 0xffffu));
      r[2] = __builtin_amdgcn_readfirstlane((int)(bytes < 0x7fffffffL ? bytes : 0x7fffffffL));
      r[3] = 0x00020000;
      return r;
    };
    const long ld = (long)a.lds * ES;
    const i32x4_t rw = resource(static_cast<const char *>(a.W) + unit0 * ld, 16 * ld);
    const i32x4_t rs = resource(static_cast<const char *>(a.state) + row0 * ld, (a.B - row0) * ld);
    int off[1 + RT][2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = i * 8 + (lane >> 3), chunk = ((lane & 7) ^ rowk_swz(r)) << 4;
      off[0][i] = (int)(r * ld) + chunk + first * 128;
#pragma unroll
      for (int b = 0; b < RT; ++b)  // rows past the streams repeat the last one (their products are unused)
        off[1 + b][i] = (int)(min(b * 16 + r, a.B - 1 - row0) * ld) + chunk + first * 128;
    }
    auto issue = [&](int slot, int piece) {
      char *const at = ring + slot * SLOT;
#pragma unroll
      for (int b = 0; b < 1 + RT; ++b)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const unsigned lds_addr = __builtin_amdgcn_readfirstlane(
              (unsigned)(unsigned long long)(lds_void_ptr)(at + b * PIECE + i * 1024));
          asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                       :
                       : "s"(lds_addr), "v"(off[b][i]), "s"(b == 0 ? rw : rs), "s"(piece * 128)
                       : "memory", "m0");
        }
    };
    const int lrow = lr * 128, swz = rowk_swz(lr);
    // the g-th 16 bytes of this lane's row of a piece
    auto chunk = [&](const char *p, int g) { return *reinterpret_cast<const u32x4_t *>(p + lrow + ((g ^ swz) << 4)); };
#pragma unroll
    for (int q = 0; q < DEPTH; ++q)
      if (q < n) issue(q, q);
    int slot = 0;
#pragma unroll 1
    for (int p = 0; p < n; ++p) {
      // piece p has landed: at most the loads of those after it are outstanding
      const int behind = min(n - 1 - p, DEPTH - 1);
      if (behind == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      else if (behind == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LOADS) : "memory");
      else if constexpr (DEPTH > 2) {
        if (behind == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * LOADS) : "memory");
        else if constexpr (DEPTH > 3) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * LOADS) : "memory");
      }
      const char *const at = ring + slot * SLOT;
      const int g = lane >> 4;
      u32x4_t w[2], f[RT][2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {  // bf16: two blocks of 32 values; fp32: the two halves of one
        const int q = ES == 2 ? 4 * i + g : 2 * g + i;
        w[i] = chunk(at, q);
#pragma unroll
        for (int r = 0; r < RT; ++r) f[r][i] = chunk(at + (1 + r) * PIECE, q);
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // before the slot is filled again
      if (p + DEPTH < n) issue(slot, p + DEPTH);
      slot = slot + 1 == DEPTH ? 0 : slot + 1;
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        if constexpr (ES == 2) {
#pragma unroll
          for (int i = 0; i < 2; ++i) mma_block(acc[r], i, StepFrag<T>{{w[i]}}, StepFrag<T>{{f[r][i]}});
        } else {
          mma_block(acc[r], 0, StepFrag<T>{{w[0], w[1]}}, StepFrag<T>{{f[r][0], f[r][1]}});
        }
      }
    }
  }
  // (a wave's own loads and reads of its ring are through; its partial tiles go where no other wave's loads can land)
  f32x4_t *const red = reinterpret_cast<f32x4_t *>(lds);
  auto part = [&](int w, int r) { return red + w * (DEPTH * SLOT / 16) + r * 64 + lane; };
#pragma unroll
  for (int r = 0; r < RT; ++r) *part(wave, r) = acc[r][0] + acc[r][1];
  __syncthreads();
  if (!mine) return;
  f32x4_t s = *part(0, wave);
#pragma unroll
  for (int q = 1; q < NWAVE; ++q) s += *part(q, wave);
  f32x4_t o;
  tv_t oc;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float h = BACKWARD ? to_f32(hv[e]) : 0.0f;
    o[e] = STORE ? s[e] : BACKWARD ? (x[e] + s[e]) * h * (1.0f - h) : sigmoidf_(s[e] + x[e]);
    if (ecol + e >= a.H) o[e] = 0.0f;
    oc[e] = from_f32<T>(o[e]);
  }
  if (MODE != STEP_STORE32) *reinterpret_cast<tv_t *>(static_cast<T *>(a.out) + (long)erow * Hp + ecol) = oc;
  if (BACKWARD || MODE == STEP_STORE32) *reinterpret_cast<f32x4_t *>(a.out32 + (long)erow * Hp + ecol) = o;
  if (MODE == STEP_FORWARD && a.h_state)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (ecol + e < a.H) a.h_state[(long)erow * a.H + ecol + e] = o[e];
#endif
}

}  // namespace rnnlm_dev
