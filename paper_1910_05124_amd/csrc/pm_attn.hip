// Attention core: kernels and their launchers (see pm_attn_api.hpp for why this is a separate translation unit).
#include <hip/hip_runtime.h>

#include <climits>
#include <cmath>
#include <cstdint>

#include "pm_attn_api.hpp"
#include "pm_attn_f32.hpp"
#include "pm_attn_mfma.hpp"

namespace {
// bf16 matrix instructions: whole tiles of 64-wide heads, or (ragged lengths, 32-wide heads) with the probabilities in
// three terms
template <int DH, bool RAGGED, bool SPLIT>
void mfma_fwd(hipStream_t st, int B, int S, int H, const bf16_t* q, const bf16_t* k, const bf16_t* v, bf16_t* o, float* lse) {
  const int qblocks = (S + 127) / 128;
  hipLaunchKernelGGL((pm_attn_mfma_fwd_kernel<DH, RAGGED, SPLIT>), dim3(B * H * qblocks), dim3(256), 0, st, q, k, v, o, lse, S, H,
                     B * H, 1.f / sqrtf((float)DH));
}
template <int DH, bool RAGGED, bool SPLIT>
void mfma_bwd(hipStream_t st, int B, int S, int H, const bf16_t* q, const bf16_t* k, const bf16_t* v, const bf16_t* o,
              const bf16_t* dO, const float* lse, bf16_t* dq, bf16_t* dk, bf16_t* dv) {
  const int qblocks = (S + 127) / 128;
  const float scale = 1.f / sqrtf((float)DH);
  hipLaunchKernelGGL((pm_attn_mfma_dq_kernel<DH, RAGGED, SPLIT>), dim3(B * H * qblocks), dim3(256), 0, st, q, k, v, o, dO, lse, dq,
                     S, H, B * H, scale);
  hipLaunchKernelGGL((pm_attn_mfma_dkv_kernel<DH, RAGGED, SPLIT>), dim3(B * H * qblocks), dim3(256), 0, st, q, k, v, o, dO, lse,
                     dk, dv, S, H, B * H, scale);
}
template <typename T, int DH>
void f32_fwd(hipStream_t st, int B, int S, int H, const T* q, const T* k, const T* v, T* o, float* lse) {
  hipLaunchKernelGGL((pm_attn_f32_fwd_kernel<T, DH>), dim3(B * H * ((S + 15) / 16)), dim3(256), 0, st, q, k, v, o, lse, S, H, B * H,
                     1.f / sqrtf((float)DH));
}
template <typename T, int DH>
void f32_bwd(hipStream_t st, int B, int S, int H, const T* q, const T* k, const T* v, const T* o, const T* dO, const float* lse,
             T* dq, T* dk, T* dv) {
  const dim3 grid(B * H * ((S + 31) / 32)), blk(64);
  const float scale = 1.f / sqrtf((float)DH);
  hipLaunchKernelGGL((pm_attn_f32_dq_kernel<T, DH>), grid, blk, 0, st, q, k, v, o, dO, lse, dq, S, H, B * H, scale);
  hipLaunchKernelGGL((pm_attn_f32_dkv_kernel<T, DH>), grid, blk, 0, st, q, k, v, o, dO, lse, dk, dv, S, H, B * H, scale);
}
}  // namespace

bool pm_attn_fwd_launch(hipStream_t st, int B, int S, int H, int dh, const bf16_t* q, const bf16_t* k, const bf16_t* v, bf16_t* o,
                        float* lse) {
  if (pm_attn_whole_tiles(S, dh)) { mfma_fwd<64, false, false>(st, B, S, H, q, k, v, o, lse); return true; }
  if (!pm_attn_short_fits(S, dh)) return false;
  switch (dh) {
    case 4: f32_fwd<bf16_t, 4>(st, B, S, H, q, k, v, o, lse); break;
    case 8: f32_fwd<bf16_t, 8>(st, B, S, H, q, k, v, o, lse); break;
    case 16: f32_fwd<bf16_t, 16>(st, B, S, H, q, k, v, o, lse); break;
    case 32: mfma_fwd<32, true, true>(st, B, S, H, q, k, v, o, lse); break;
    default: mfma_fwd<64, true, true>(st, B, S, H, q, k, v, o, lse); break;
  }
  return true;
}
bool pm_attn_fwd_launch(hipStream_t st, int B, int S, int H, int dh, const float* q, const float* k, const float* v, float* o,
                        float* lse) {
  if (!pm_attn_short_fits(S, dh)) return false;
  switch (dh) {
    case 4: f32_fwd<float, 4>(st, B, S, H, q, k, v, o, lse); break;
    case 8: f32_fwd<float, 8>(st, B, S, H, q, k, v, o, lse); break;
    case 16: f32_fwd<float, 16>(st, B, S, H, q, k, v, o, lse); break;
    case 32: f32_fwd<float, 32>(st, B, S, H, q, k, v, o, lse); break;
    default: f32_fwd<float, 64>(st, B, S, H, q, k, v, o, lse); break;
  }
  return true;
}
bool pm_attn_bwd_launch(hipStream_t st, int B, int S, int H, int dh, const bf16_t* q, const bf16_t* k, const bf16_t* v,
                        const bf16_t* o, const bf16_t* dO, const float* lse, bf16_t* dq, bf16_t* dk, bf16_t* dv) {
  if (pm_attn_whole_tiles(S, dh)) { mfma_bwd<64, false, false>(st, B, S, H, q, k, v, o, dO, lse, dq, dk, dv); return true; }
  if (!pm_attn_short_fits(S, dh)) return false;
  switch (dh) {
    case 4: f32_bwd<bf16_t, 4>(st, B, S, H, q, k, v, o, dO, lse, dq, dk, dv); break;
    case 8: f32_bwd<bf16_t, 8>(st, B, S, H, q, k, v, o, dO, lse, dq, dk, dv); break;
    case 16: f32_bwd<bf16_t, 16>(st, B, S, H, q, k, v, o, dO, lse, dq, dk, dv); break;
    case 32: mfma_bwd<32, true, true>(st, B, S, H, q, k, v, o, dO, lse, dq, dk, dv); break;
    default: mfma_bwd<64, true, true>(st, B, S, H, q, k, v, o, dO, lse, dq, dk, dv); break;
  }
  return true;
}
bool pm_attn_bwd_launch(hipStream_t st, int B, int S, int H, int dh, const float* q, const float* k, const float* v,
                        const float* o, const float* dO, const float* lse, float* dq, float* dk, float* dv) {
  if (!pm_attn_short_fits(S, dh)) return false;
  switch (dh) {
    case 4: f32_bwd<float, 4>(st, B, S, H, q, k, v, o, dO, lse, dq, dk, dv); break;
    case 8: f32_bwd<float, 8>(st, B, S, H, q, k, v, o, dO, lse, dq, dk, dv); break;
    case 16: f32_bwd<float, 16>(st, B, S, H, q, k, v, o, dO, lse, dq, dk, dv); break;
    case 32: f32_bwd<float, 32>(st, B, S, H, q, k, v, o, dO, lse, dq, dk, dv); break;
    default: f32_bwd<float, 64>(st, B, S, H, q, k, v, o, dO, lse, dq, dk, dv); break;
  }
  return true;
}
