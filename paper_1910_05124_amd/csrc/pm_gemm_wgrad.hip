// Weight-gradient products on 256 x 256 blocks (see pm_gemm_async_api.hpp).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "pm_gemm_async.hpp"
#include "pm_transformer.hpp"

void pm_wgrad_grouped256_launch(hipStream_t st, const PmGemmProb<PmEpiBwdWeight>* probs, const PmXcdSeg* segs,
                                const int32_t* xcd_tiles, int max_segs, int blocks) {
  hipLaunchKernelGGL((pm_gemm_async_grouped_kernel<PmAsync256, PmEpiBwdWeight>), dim3(blocks), dim3(PmAsync256::NT), 0, st, probs, segs, xcd_tiles, max_segs);
}
void pm_wgrad_grouped256_launch(hipStream_t st, const PmGemmProb<PmEpiBwdWeightUpd>* probs, const PmXcdSeg* segs,
                                const int32_t* xcd_tiles, int max_segs, int blocks) {
  hipLaunchKernelGGL((pm_gemm_async_grouped_kernel<PmAsync256, PmEpiBwdWeightUpd>), dim3(blocks), dim3(PmAsync256::NT), 0, st, probs, segs, xcd_tiles, max_segs);
}
