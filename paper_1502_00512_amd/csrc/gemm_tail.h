// The output layer's large bf16 contraction: whole rounds of 256x256 tiles, what is left over on 128x128 ones.
//
// One persistent workgroup per compute unit walks the large tiles, and a last round that only some compute units have a tile
// for takes nearly as long as a full one.  So the large tiles take as many rows of the output as fill whole rounds, and the
// same workgroups then share out the remaining rows in tiles of a quarter the size.  us a window, all rows on large tiles and
// this: V = 33278, H = 650, 100x9 (520 tiles are 2.03 rounds) 331 and 327; V = 100000, H = 2048, 128x20 (15.3) 3146 and 3130,
// hardly more than two runs differ; V = 40000, H = 500, 120x18 (5.5) 507 and 507; eight evaluated windows of V = 64000, H =
// 1024, 64x20 (39.06) 1333 and 1293.
// (The output update's rest on small tiles: V = 33278, H = 650, 1.5 rounds, 331 and 348; V = 30000, H = 1500, 2.8 rounds, 618 and
// 628; nowhere more than a hundredth faster: its epilogue's memory traffic is what a full round waits for.)
#pragma once
#include "gemm_dma4.h"

namespace rnnlm_dev {

template <int WGM, int WGN, int LB, class Epi>
__global__ void __launch_bounds__(512) gemm_tail_kernel(const GemmShape g, const Epi epi, const GemmShape gt, const Epi epit) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int STAGE = dma_stage_bytes<256, 256, Epi>(), SMALL = dma4_stage_bytes<128, 128, Epi>();
  static_assert(2 * STAGE <= 160 * 1024 && 2 * SMALL <= STAGE, "tile does not fit the 160 KB of LDS");
  __shared__ __attribute__((aligned(1024))) char stage0[STAGE];
  __shared__ __attribute__((aligned(1024))) char stage1[STAGE];
  gemm_dma_items<256, 256, WGM, WGN, ROWK, LB, Epi, true>(g, epi, stage0, stage1);
  for (int item = blockIdx.x; item < gt.perXcd * NUM_XCD; item += gridDim.x) {
    __syncthreads();  // the LDS is free
    gemm_dma4_items<bf16_t, 128, 128, 4, 2, ROWK, LB, Epi, false>(gt, epit, item, gt.perXcd * NUM_XCD, stage0, stage0 + SMALL,
                                                                  stage1, stage1 + SMALL);
  }
#endif  // __HIP_DEVICE_COMPILE__
}

// A operand's first `rows` rows (a multiple of 256) on large tiles, the others on small ones (epit: the epilogue aimed at
// them).  (An output without such a rest is 1 % of a short window faster through gemm_dma_kernel.)
template <int WGM, int WGN, int LB, class Epi>
inline hipError_t launch_gemm_tail(hipStream_t stream, const bf16_t *A, long lda, const bf16_t *B, long ldb, long Mg, long Ng,
                                   long K, long rows, const Epi &epi, const Epi &epit, int band) {
  GemmShape g, gt;
  hipError_t e = dma_shape<256, 256, ROWK, LB>(g, A, lda, B, ldb, rows, Ng, K, 1, band);
  if (e == hipSuccess)
    e = dma4_shape<bf16_t, 128, 128, ROWK, LB>(gt, A + rows * lda, lda, B, ldb, Mg - rows, Ng, K, 1, band);
  if (e != hipSuccess) return e;
  const int items = std::max(g.perXcd, gt.perXcd) * NUM_XCD;
  hipLaunchKernelGGL((gemm_tail_kernel<WGM, WGN, LB, Epi>), dim3(std::min(items, 256)), dim3(512), 0, stream, g, epi, gt, epit);
  return hipGetLastError();
}

}  // namespace rnnlm_dev
