// Data-gradient products (see pm_gemm_async_api.hpp).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "pm_gemm_async.hpp"
#include "pm_transformer.hpp"

// How a product with K >> I, J is cut (pm_gemm_async_ksplit_kernel): as many parts, of at least 512 indices each, as the rule
// finds fastest with the parts' outputs written and read once more at 4 bytes per ps; parts = 1: not at all.
PmKSplit pm_ksplit_plan(int I, int J, int K, int max_parts) {
  PmKSplit plan{1, K};
  if (K < 2048) return plan;
  float best = 3e38f;
  for (int parts = 1; parts <= std::min({8, max_parts, K / 512}); ++parts) {
    const int kpart = (K + 64 * parts - 1) / (64 * parts) * 64;
    if ((K + kpart - 1) / kpart != parts) continue;
    float us = 3e38f;
    pm_async_each([&](auto cfg) { us = std::min(us, pm_async_us<decltype(cfg)>(parts, I, J, kpart, 1)); });
    us += (parts - 1) * 2e-6f * (float)I * (float)J;
    if (us < best) best = us, plan = PmKSplit{parts, kpart};
  }
  return plan;
}

template bool pm_async_try(hipStream_t, const PmGemmProb<PmEpiF32>&, const PmPrefetch*);
template bool pm_async_try(hipStream_t, const PmGemmProb<PmEpiBwdData<bf16_t>>&, const PmPrefetch*);
template bool pm_gemm_kseg3_try(hipStream_t, int, int, int, const bf16_t* const (&)[3], int64_t, const PmWLoc<bf16_t> (&)[3], int64_t, const PmEpiF32&);
template bool pm_gemm_ksplit_try(hipStream_t, const PmGemmProb<PmEpiF32>&, const PmKSplit&, int64_t);
