// Entry points of the attention core (kernels in pm_attn.hip, a translation unit of its own: it is compiled with
// accumulators of the matrix instructions kept in ordinary vector registers, which suits these kernels (the
// softmax arithmetic works on the accumulators between two products) and not the 256 x 256-tile GEMM, whose
// accumulators fill the second register file).
#pragma once
#include <hip/hip_runtime.h>

#include "pm_common.hpp"

// Shapes the core takes: bf16 with 64-wide heads and whole 32-row tiles of any length; otherwise head sizes 4 .. 64
// and sequences of at most 8192 / (head size + 1) rows.
inline bool pm_attn_whole_tiles(int S, int dh) { return dh == 64 && S >= 32 && (S % 32) == 0; }
inline bool pm_attn_short_fits(int S, int dh) {
  return (int64_t)S * (dh + 1) <= 8192 && S <= 1024 && (dh == 4 || dh == 8 || dh == 16 || dh == 32 || dh == 64);
}

// q, k, v, o, dO, dq, dk, dv: [B * S, H * dh], row b * S + s; lse: [B, H, S] fp32 (natural-log units).
// False (nothing launched): shape not taken.
bool pm_attn_fwd_launch(hipStream_t st, int B, int S, int H, int dh, const bf16_t* q, const bf16_t* k, const bf16_t* v, bf16_t* o,
                        float* lse);
bool pm_attn_fwd_launch(hipStream_t st, int B, int S, int H, int dh, const float* q, const float* k, const float* v, float* o,
                        float* lse);
bool pm_attn_bwd_launch(hipStream_t st, int B, int S, int H, int dh, const bf16_t* q, const bf16_t* k, const bf16_t* v,
                        const bf16_t* o, const bf16_t* dO, const float* lse, bf16_t* dq, bf16_t* dk, bf16_t* dv);
bool pm_attn_bwd_launch(hipStream_t st, int B, int S, int H, int dh, const float* q, const float* k, const float* v,
                        const float* o, const float* dO, const float* lse, float* dq, float* dk, float* dv);
