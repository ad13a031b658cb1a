// Weight updates of a window that share a launch.
#pragma once
#include "gemm_dma4.h"
#include "gemm_split.h"
#include "kernels.h"

namespace rnnlm_dev {

// Contractions of one form (operand layouts, 64x64 tiles, depth) whose outputs are updated matrices.  Each is bound by the
// chain of K blocks that a workgroup walks, with one workgroup or less per compute unit; side by side their chains overlap
// (compressed architecture, H = 1024, P = 512, 128x20: three launches 17 + 17 + 18 us on 128, 128 and 256 workgroups, one
// launch of the 512 some 25; window 348 and 329).
constexpr int GROUP_MAX = 3;
template <class Epi>
struct UpdateGroup {
  GemmShape g[GROUP_MAX];
  Epi epi[GROUP_MAX];
  int first[GROUP_MAX + 1];  // workgroups before each (multiples of 8, so that their XCDs are as in a launch of their own)
};
template <int LA, int LB, class Epi>
__global__ void __launch_bounds__(256) update_group_kernel(const UpdateGroup<Epi> u) {
#if defined(__HIP_DEVICE_COMPILE__)
  __shared__ __attribute__((aligned(1024))) char lds[4][dma4_stage_bytes<64, 64, Epi>()];
  int p = 0;
#pragma unroll
  for (int q = 1; q < GROUP_MAX; ++q) p += (int)blockIdx.x >= u.first[q];
  const GemmShape &g = u.g[p];
  gemm_dma4_items<bf16_t, 64, 64, 2, 2, LA, LB, Epi, false>(g, u.epi[p], blockIdx.x - u.first[p], g.perXcd * NUM_XCD, lds[0],
                                                            lds[1], lds[2], lds[3]);
#endif
}

// All updates of a short window of the plain architecture (output matrix, recurrent matrix, embedding rows) in one launch:
// they need nothing from one another, and as three launches, or two of them on a second stream that is tied in and out with
// events, they took longer to start than to run.  PARTS as in F32Plan (fp32 cores or split operands).  us a window, before and
// now: fp32 V = 1000, H = 64, 4x8 59.8 and 52.8, V = 10000, H = 256, 32x10 148 and 113, V = 5000, H = 1000, 30x30 500 and 472;
// bf16 V = 10000, H = 512, 16x16 95.9 and 87.9, V = 5000, H = 1000, 30x30 192 and 162; where the output update takes most of the
// time no difference (V = 100000, H = 2048, 16x8 873 and 876).
template <typename T>
struct WindowUpdate {
  GemmShape out_g, rec_g;
  EpiSgd<T> out;
  EpiSgdT<T> rec;
  ScanUpdate<T> scan;
  int nRec, nOut;  // workgroups of the recurrent and of the output update; then those of the embedding update
};
template <typename T, int TILE, int PARTS, int LA, int LB, class Epi>
__device__ inline void update_tile(const GemmShape &g, const Epi &epi, int item, char *lds) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (sizeof(T) == 4 && PARTS == 1) {
    gemm_split_item<64, 64, 2, 2, 1, LA, LB, 1, 2, Epi>(g, epi, item, lds);
  } else {
    constexpr int S = dma4_stage_bytes<TILE, TILE, Epi>(), WGM = TILE == 128 ? 4 : 2;
    gemm_dma4_items<T, TILE, TILE, WGM, 2, LA, LB, Epi, false>(g, epi, item, g.perXcd * NUM_XCD, lds, lds + S, lds + 2 * S,
                                                               lds + 3 * S);
  }
#endif
}
template <typename T, int TILE, int PARTS, bool ALIGNED>
__global__ void __launch_bounds__(TILE * 4) window_update_kernel(const WindowUpdate<T> u) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int LOOP = PARTS == 1 ? split_lds_bytes<64, 64, 1, EpiSgd<T>>() : 4 * dma4_stage_bytes<TILE, TILE, EpiSgd<T>>();
  constexpr int BYTES = LOOP > (int)sizeof(ScanShared) ? LOOP : (int)sizeof(ScanShared);
  __shared__ __attribute__((aligned(1024))) char lds[BYTES];
  const int id = blockIdx.x;
  if (id < u.nRec) {
    update_tile<T, TILE, PARTS, KROW, KROW>(u.rec_g, u.rec, id, lds);
  } else if (id < u.nRec + u.nOut) {
    update_tile<T, TILE, PARTS, ROWK, KROW>(u.out_g, u.out, id - u.nRec, lds);
  } else {
    const int k = id - u.nRec - u.nOut;
    scatter_scan<TILE / 16, ALIGNED>(u.scan, *reinterpret_cast<ScanShared *>(lds), k % u.scan.M, k / u.scan.M);
  }
#endif
}

}  // namespace rnnlm_dev
