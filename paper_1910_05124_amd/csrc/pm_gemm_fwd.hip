// Forward products (see pm_gemm_async_api.hpp).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "pm_gemm_async.hpp"
#include "pm_transformer.hpp"

template bool pm_async_try(hipStream_t, const PmGemmProb<PmEpiFwd<bf16_t>>&, const PmPrefetch*);
template bool pm_async_try(hipStream_t, const PmGemmProb<PmEpiFwdRes<bf16_t>>&, const PmPrefetch*);
template bool pm_gemm_multi3_try(hipStream_t, const PmGemmProb<PmEpiFwd<bf16_t>> (&)[3]);
