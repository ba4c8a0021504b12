// Attention core: kernels and their launchers (see pm_attn_api.hpp for why this is a separate translation unit).
#include <hip/hip_runtime.h>

#include <climits>
#include <cmath>
#include <cstdint>

#include "pm_attn_api.hpp"
#include "pm_attn_f32.hpp"
#include "pm_attn_mfma.hpp"

namespace {
// Backward passes of up to this many blocks a half go out as one launch (two blocks per compute unit: beyond that the halves fill
// the chip by themselves, and dQ alone has three).  dQ + dK / dV, us: 32 x 128 tokens, 8 heads 10.6 + 10.2 -> 16.2, 8 x 256, 12 heads
// 11.5 + 12.6 -> 17.4, 24 x 100, 5 heads 9.7 + 12.4 -> 14.0, fp32 8 x 64, 8 heads of 32 8.3 + 9.1 -> 10.1.
constexpr unsigned PM_AT_JOIN = 512;

// bf16 matrix instructions: forward whole tiles of 64-wide heads; backward those, or (ragged lengths, 32-wide heads) with
// the probabilities in three terms
void mfma_fwd(hipStream_t st, int B, int S, int H, const bf16_t* q, const bf16_t* k, const bf16_t* v, bf16_t* o, float* lse) {
  const int qblocks = (S + 127) / 128;
  hipLaunchKernelGGL((pm_attn_mfma_fwd_kernel<64>), dim3(B * H * qblocks), dim3(256), 0, st, q, k, v, o, lse, S, H, B * H,
                     1.f / sqrtf(64.f));
}
template <int DH, bool RAGGED, bool SPLIT>
void mfma_bwd(hipStream_t st, int B, int S, int H, const bf16_t* q, const bf16_t* k, const bf16_t* v, const bf16_t* o,
              const bf16_t* dO, const float* lse, bf16_t* dq, bf16_t* dk, bf16_t* dv) {
  const int qblocks = (S + 127) / 128;
  const float scale = 1.f / sqrtf((float)DH);
  const unsigned n = B * H * qblocks;
  if (n <= PM_AT_JOIN) {
    hipLaunchKernelGGL((pm_attn_mfma_bwd_kernel<DH, RAGGED, SPLIT>), dim3(2 * n), dim3(256), 0, st, q, k, v, o, dO, lse, dq, dk, dv, S, H, B * H, scale);
    return;
  }
  hipLaunchKernelGGL((pm_attn_mfma_dq_kernel<DH, RAGGED, SPLIT>), dim3(n), dim3(256), 0, st, q, k, v, o, dO, lse, dq,
                     S, H, B * H, scale);
  hipLaunchKernelGGL((pm_attn_mfma_dkv_kernel<DH, RAGGED, SPLIT>), dim3(n), dim3(256), 0, st, q, k, v, o, dO, lse,
                     dk, dv, S, H, B * H, scale);
}
template <typename T, int DH, bool VEC>
void f32_fwd(hipStream_t st, int B, int S, int H, const T* q, const T* k, const T* v, T* o, float* lse) {
  hipLaunchKernelGGL((pm_attn_f32_fwd_kernel<T, DH, VEC>), dim3(B * H * ((S + 15) / 16)), dim3(256), 0, st, q, k, v, o, lse, S, H,
                     B * H, 1.f / sqrtf((float)DH));
}
template <typename T, int DH, bool VEC>
void f32_bwd(hipStream_t st, int B, int S, int H, const T* q, const T* k, const T* v, const T* o, const T* dO, const float* lse,
             T* dq, T* dk, T* dv) {
  const dim3 grid(B * H * ((S + 31) / 32)), blk(64);
  const float scale = 1.f / sqrtf((float)DH);
  if (grid.x <= PM_AT_JOIN) {
    hipLaunchKernelGGL((pm_attn_f32_bwd_kernel<T, DH, VEC>), dim3(2 * grid.x), blk, 0, st, q, k, v, o, dO, lse, dq, dk, dv, S, H, B * H, scale);
    return;
  }
  hipLaunchKernelGGL((pm_attn_f32_dq_kernel<T, DH, VEC>), grid, blk, 0, st, q, k, v, o, dO, lse, dq, S, H, B * H, scale);
  hipLaunchKernelGGL((pm_attn_f32_dkv_kernel<T, DH, VEC>), grid, blk, 0, st, q, k, v, o, dO, lse, dk, dv, S, H, B * H, scale);
}
// the fp32 kernels of a head size, in bf16 with 8-byte accesses or without
template <typename T, bool VEC, class... P>
void f32_fwd_any(int dh, P... p) {
  switch (dh) {
    case 4: f32_fwd<T, 4, VEC>(p...); break;
    case 8: f32_fwd<T, 8, VEC>(p...); break;
    case 16: f32_fwd<T, 16, VEC>(p...); break;
    case 32: f32_fwd<T, 32, VEC>(p...); break;
    default: f32_fwd<T, 64, VEC>(p...); break;
  }
}
template <typename T, bool VEC, class... P>
void f32_bwd_any(int dh, P... p) {
  switch (dh) {
    case 4: f32_bwd<T, 4, VEC>(p...); break;
    case 8: f32_bwd<T, 8, VEC>(p...); break;
    case 16: f32_bwd<T, 16, VEC>(p...); break;
    default:
      if constexpr (sizeof(T) == 4 || !VEC) {
        if (dh == 32) f32_bwd<T, 32, VEC>(p...);
        else f32_bwd<T, 64, VEC>(p...);
      }
  }
}
template <class... P>
bool aligned(size_t n, P... p) { return ((... | (uintptr_t)p) & (n - 1)) == 0; }
}  // namespace

// Outside whole tiles the forward pass is fp32 arithmetic (see pm_attn_mfma.hpp).  Backward of heads of 32 and 64: the bf16
// kernels read 16 bytes at a time; tensors that start anywhere else go through the fp32 kernels, element by element
// (24 x 100 tokens, 5 heads of 64: 59 us against 20).
bool pm_attn_fwd_launch(hipStream_t st, int B, int S, int H, int dh, const bf16_t* q, const bf16_t* k, const bf16_t* v, bf16_t* o,
                        float* lse) {
  if (pm_attn_whole_tiles(S, dh)) { mfma_fwd(st, B, S, H, q, k, v, o, lse); return true; }
  if (!pm_attn_short_fits(S, dh)) return false;
  if (aligned(8, q, k, v, o)) f32_fwd_any<bf16_t, true>(dh, st, B, S, H, q, k, v, o, lse);
  else f32_fwd_any<bf16_t, false>(dh, st, B, S, H, q, k, v, o, lse);
  return true;
}
bool pm_attn_fwd_launch(hipStream_t st, int B, int S, int H, int dh, const float* q, const float* k, const float* v, float* o,
                        float* lse) {
  if (!pm_attn_short_fits(S, dh)) return false;
  f32_fwd_any<float, true>(dh, st, B, S, H, q, k, v, o, lse);
  return true;
}
bool pm_attn_bwd_launch(hipStream_t st, int B, int S, int H, int dh, const bf16_t* q, const bf16_t* k, const bf16_t* v,
                        const bf16_t* o, const bf16_t* dO, const float* lse, bf16_t* dq, bf16_t* dk, bf16_t* dv) {
  if (pm_attn_whole_tiles(S, dh)) { mfma_bwd<64, false, false>(st, B, S, H, q, k, v, o, dO, lse, dq, dk, dv); return true; }
  if (!pm_attn_short_fits(S, dh)) return false;
  if (!aligned(dh < 32 ? 8 : 16, q, k, v, o, dO, dq, dk, dv)) f32_bwd_any<bf16_t, false>(dh, st, B, S, H, q, k, v, o, dO, lse, dq, dk, dv);
  else if (dh == 32) mfma_bwd<32, true, true>(st, B, S, H, q, k, v, o, dO, lse, dq, dk, dv);
  else if (dh == 64) mfma_bwd<64, true, true>(st, B, S, H, q, k, v, o, dO, lse, dq, dk, dv);
  else f32_bwd_any<bf16_t, true>(dh, st, B, S, H, q, k, v, o, dO, lse, dq, dk, dv);
  return true;
}
bool pm_attn_bwd_launch(hipStream_t st, int B, int S, int H, int dh, const float* q, const float* k, const float* v,
                        const float* o, const float* dO, const float* lse, float* dq, float* dk, float* dv) {
  if (!pm_attn_short_fits(S, dh)) return false;
  f32_bwd_any<float, true>(dh, st, B, S, H, q, k, v, o, dO, lse, dq, dk, dv);
  return true;
}
