// Causal attention core in fp32 arithmetic, for fp32 contexts, for the forward pass of bf16 tensors outside whole
// tiles of 64-wide heads, and for the backward pass of bf16 heads narrower than 32 or off the bf16 kernels' alignment, gfx950.
// T: element type of the tensors in memory; everything inside is fp32.  VEC: see pm_af_ld4.
//
// Order of the sums.  Scores are one chain of fused multiply-adds over the head dimension, the forward pass takes its keys
// one after the other (running maximum and sum, every earlier value scaled when the maximum moves), and a gradient row is one
// chain over its keys or queries in order.  Whole fp32 networks have ReLU units behind this core, whose gradients
// hang on the rounding of a pre-activation next to zero, so the order is part of the result (see pm_gemm_f32.hpp).
//
// Forward: 16 lanes per query row.  A lane holds DH / 16 columns of the row's output; for 16 keys at a time each lane
// computes one key's score, a scan over the lanes gives every key's running maximum (a maximum does not depend on
// the order), so that the two exponentials of a key are computed once, and the 16 keys are then applied in order.
//
// Backward, on v_mfma_f32_32x32x2_f32: the scheme is that of pm_attn_mfma.hpp, a wave owns 32 rows of one index and
// streams 32-row tiles of the other; the score-like products come out transposed, streamed index on the MFMA rows and
// owned index on the columns, so row statistics are per-lane scalars and the probabilities are the second product's
// B operand.  The instruction adds its two products one after the other, lane group 0's first, hence:
//   * scores: step c contracts head-dimension entries 2 c and 2 c + 1.  The tile lies in LDS with the even entries of a row
//     in front of the odd ones, so that a lane reads its share as 16-byte pieces;
//   * second product: accumulator value v of group g is streamed row 8 (v / 4) + 4 g + v % 4, and a step is to contract rows
//     r and r + 1: one lane exchange per two values brings them there.
// One wave per block (the tiles are private, no barrier but the wave's own): a tile costs 64 clocks per contracted pair
// - 2048 + 2048 clocks at DH = 64 - against 256 clocks to fetch it, so sharing tiles between waves would save nothing,
// and these shapes (a few dozen heads, sequences of at most 8192 / (DH + 1) rows) need the blocks to fill the chip.
// A masked row has probability zero, and zero times an infinity or NaN of its is NaN: where a tile with masked rows holds such
// a value, its rows are added by hand (pm_at_add_row), each for the owned rows that see it.
// 24 sequences of 100 tokens, 5 heads of 64 in bf16: forward 496 -> 12 us (8 on the bf16 matrix kernel); 82 x 100 tokens, 16
// heads of 64: 1213 -> 82 us (23).
// 8 sequences of 64 tokens, 8 heads of 32: forward 85 -> 6 us, backward 161 -> 16 us per layer against one thread per row.
#pragma once
#include "pm_common.hpp"
#include "pm_mfma_types.hpp"

template <int DH>
struct PmAf {
  static constexpr int ST = DH + 4;                       // LDS row stride (floats): 16-byte rows, 4 floats apart in the banks
  static constexpr int HALF = DH / 2;
  static constexpr int NDT = (DH + 31) / 32;              // 32-row tiles of the head dimension in the second product
  static constexpr int PIECES = 32 * DH / 4;              // 4-element pieces of a 32-row tile
  static constexpr int PER = (PIECES + 63) / 64;          // pieces per lane
  static constexpr int ELEMS = 32 * ST + 32;              // a narrow head's column reads run past its rows
};
// Four consecutive elements of a tensor that starts anywhere: fp32 tensors are read and written 16 bytes at a time (a
// memory access of that width needs 4-byte alignment), bf16 ones 8 bytes with VEC (8-byte alignment), else element by element.
typedef float pm_f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
template <bool VEC>
__device__ __forceinline__ float4 pm_af_ld4(const float* p) {
  const pm_f32x4_any v = *reinterpret_cast<const pm_f32x4_any*>(p);
  return make_float4(v.x, v.y, v.z, v.w);
}
template <bool VEC>
__device__ __forceinline__ float4 pm_af_ld4(const bf16_t* p) {
  if constexpr (VEC) return pm_ld4(p);
  else return make_float4(ldf(p), ldf(p + 1), ldf(p + 2), ldf(p + 3));
}
template <bool VEC>
__device__ __forceinline__ void pm_af_st4(float* p, float4 x) {
  *reinterpret_cast<pm_f32x4_any*>(p) = pm_f32x4_any{x.x, x.y, x.z, x.w};
}
template <bool VEC>
__device__ __forceinline__ void pm_af_st4(bf16_t* p, float4 x) {
  if constexpr (VEC) {
    pm_st4(p, x);
  } else {
    stf(p, x.x); stf(p + 1, x.y); stf(p + 2, x.z); stf(p + 3, x.w);
  }
}
__device__ __forceinline__ float pm_af_exp(float x) { return __builtin_amdgcn_exp2f(x * 1.44269504f); }

// ---------------------------------------------------------------------------------------------
// forward
// ---------------------------------------------------------------------------------------------
// lane N of each group of 16, to all of them
template <int N>
__device__ __forceinline__ float pm_row_bcast(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x150 + N, 0xf, 0xf, true));
}
// lane l - N of the group of 16, `out` where there is none
template <int N>
__device__ __forceinline__ float pm_row_shr(float x, float out) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(out), __float_as_int(x), 0x110 + N, 0xf, 0xf, false));
}

// Keys N .. 15 of a group, in order: l and acc scaled by the key's correction, then its probability added.  have: keys of
// the group that the row sees (FULL: all).
template <int N, int CPL, bool FULL>
__device__ __forceinline__ void pm_af_keys(float corr, float p, const float* v, int st, int have, float& l, float (&acc)[CPL]) {
  if constexpr (N < 16) {
    const float c = pm_row_bcast<N>(corr), w = pm_row_bcast<N>(p);
    float x[CPL];
#pragma unroll
    for (int e = 0; e < CPL; ++e) x[e] = v[N * st + e];
    const bool on = FULL || N < have;
    l = on ? fmaf(l, c, w) : l;
#pragma unroll
    for (int e = 0; e < CPL; ++e) acc[e] = on ? fmaf(acc[e], c, w * x[e]) : acc[e];
    pm_af_keys<N + 1, CPL, FULL>(corr, p, v, st, have, l, acc);
  }
}

// blockIdx.x = block of 16 query rows * BH + (sequence, head); wave w takes rows 4 w .. 4 w + 3, lanes 16 r .. 16 r + 15 row r
template <typename T, int DH, bool VEC>
__global__ __launch_bounds__(256) void pm_attn_f32_fwd_kernel(const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
                                                              T* __restrict__ o, float* __restrict__ lse, int S, int H, int BH,
                                                              float scale) {
  constexpr int ST = DH + 4, CPL = DH >= 16 ? DH / 16 : 1, PIECES = 32 * DH / 4, PER = (PIECES + 255) / 256;
  __shared__ __attribute__((aligned(16))) float sK[32 * ST], sV[32 * ST + 16];       // narrow heads: lanes without a column read on
  const int blocks = (S + 15) / 16;
  const int bh = blockIdx.x % BH, qb = blocks - 1 - blockIdx.x / BH;                 // long blocks first
  const int b = bh / H, h = bh % H, d = H * DH, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, t = lane & 15;
  const int64_t base = (int64_t)b * S * d + (int64_t)h * DH;
  const int w0 = qb * 16 + wave * 4, row = w0 + (lane >> 4), i = row < S ? row : S - 1;
  float qi[DH];
#pragma unroll
  for (int c = 0; c < DH; c += 4) {
    const float4 x = pm_af_ld4<VEC>(q + base + (int64_t)i * d + c);
    qi[c] = x.x * scale; qi[c + 1] = x.y * scale; qi[c + 2] = x.z * scale; qi[c + 3] = x.w * scale;
  }
  float4 rk[PER], rv[PER];
  auto fetch = [&](int tile) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int c = ((int)threadIdx.x + 256 * j) % PIECES;           // (fewer pieces than threads: fetched more than once)
      int r = tile * 32 + c / (DH / 4);
      r = r < S ? r : S - 1;
      const int64_t at = base + (int64_t)r * d + (c % (DH / 4)) * 4;
      rk[j] = pm_af_ld4<VEC>(k + at);
      rv[j] = pm_af_ld4<VEC>(v + at);
    }
  };
  auto park = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int c = ((int)threadIdx.x + 256 * j) % PIECES, at = (c / (DH / 4)) * ST + (c % (DH / 4)) * 4;
      *reinterpret_cast<float4*>(sK + at) = rk[j];
      *reinterpret_cast<float4*>(sV + at) = rv[j];
    }
  };
  const int last = (qb * 16 + 15 < S ? qb * 16 + 15 : S - 1);        // last key that a row of the block sees
  float m = -3.0e38f, l = 0.f, acc[CPL] = {};
  fetch(0);
  for (int tile = 0; tile <= last >> 5; ++tile) {
    park();
    __syncthreads();
    if (tile < last >> 5) fetch(tile + 1);                           // on its way while this one is used
    for (int jj = 0; jj < 32; jj += 16) {
      const int j0 = tile * 32 + jj;
      if (j0 > w0 + 3) break;                                        // uniform over the wave
      float s = 0.f;
      const float* kr = sK + (jj + t) * ST;
#pragma unroll
      for (int c = 0; c < DH; c += 4) {
        const float4 x = *reinterpret_cast<const float4*>(kr + c);
        s = fmaf(qi[c], x.x, s);
        s = fmaf(qi[c + 1], x.y, s);
        s = fmaf(qi[c + 2], x.z, s);
        s = fmaf(qi[c + 3], x.w, s);
      }
      // running maximum behind each key; keys that the row does not see leave it alone
      const float none = -__builtin_inff();
      float mx = j0 + t <= i ? s : none;
      mx = fmaxf(mx, pm_row_shr<1>(mx, none));
      mx = fmaxf(mx, pm_row_shr<2>(mx, none));
      mx = fmaxf(mx, pm_row_shr<4>(mx, none));
      mx = fmaxf(mx, pm_row_shr<8>(mx, none));
      const float mt = fmaxf(m, mx), mb = pm_row_shr<1>(mt, m);      // behind and before this lane's key
      const float corr = pm_af_exp(mb - mt), p = pm_af_exp(s - mt);
      m = pm_row_bcast<15>(mt);
      const float* vc = sV + jj * ST + t * CPL;
      if (j0 + 15 <= w0) pm_af_keys<0, CPL, true>(corr, p, vc, ST, 16, l, acc);
      else pm_af_keys<0, CPL, false>(corr, p, vc, ST, i - j0 + 1, l, acc);
    }
    __syncthreads();
  }
  if (row >= S) return;
  const float inv = 1.f / l;
  if (t * CPL < DH) {
    T* out = o + base + (int64_t)row * d + t * CPL;
#pragma unroll
    for (int e = 0; e < CPL; ++e) stf(out + e, acc[e] * inv);
  }
  if (t == 0) lse[((int64_t)b * H + h) * S + row] = m + __logf(l);
}

// ---------------------------------------------------------------------------------------------
// rows by hand, for tiles whose masked rows hold an infinity or NaN (also used by pm_attn_mfma.hpp)
// ---------------------------------------------------------------------------------------------
template <typename T, int DH>
__device__ __forceinline__ float pm_at_dot(const T* a, const T* b) {
  float s = 0.f;
#pragma unroll 4
  for (int c = 0; c < DH; ++c) s = fmaf(ldf(a + c), ldf(b + c), s);
  return s;
}
// acc [head dimension][owned row] += w * row, in the lanes whose owned row sees it
template <typename T, int DH>
__device__ __forceinline__ void pm_at_add_row(pm_f32x16* acc, const T* row, float w, bool sees, int lane) {
#pragma unroll
  for (int dt = 0; dt < (DH + 31) / 32; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int c = dt * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
      if (c < DH && sees) acc[dt][e] = fmaf(w, ldf(row + c), acc[dt][e]);
    }
}

// ---------------------------------------------------------------------------------------------
// backward
// ---------------------------------------------------------------------------------------------
// 32 rows of X (row stride d, rows past the end re-read the last one): registers first, LDS later
template <typename T, int DH, bool VEC>
__device__ __forceinline__ void pm_af_load(const T* X, int64_t d, int r0, int S, int lane, float4* r) {
  using A = PmAf<DH>;
#pragma unroll
  for (int j = 0; j < A::PER; ++j) {
    const int c = (lane + 64 * j) % A::PIECES;            // (fewer pieces than lanes: fetched more than once)
    int row = r0 + c / (DH / 4);
    row = row < S ? row : S - 1;
    r[j] = pm_af_ld4<VEC>(X + (int64_t)row * d + (c % (DH / 4)) * 4);
  }
}
// whether any lane's pieces hold a value that is not finite
template <int N>
__device__ __forceinline__ bool pm_af_odd(const float4* r) {
  uint32_t top = 0;                                          // an exponent of all ones carries into the sign
  auto carry = [](float f) { return (__float_as_uint(f) & 0x7f800000u) + 0x00800000u; };
#pragma unroll
  for (int j = 0; j < N; ++j) top |= carry(r[j].x) | carry(r[j].y) | carry(r[j].z) | carry(r[j].w);
  return __builtin_amdgcn_ballot_w64((top & 0x80000000u) != 0) != 0;
}
// head-dimension entry c of a row in LDS: the even ones, then the odd ones
template <int DH>
__device__ __forceinline__ constexpr int pm_af_pos(int c) { return (c & 1) * PmAf<DH>::HALF + (c >> 1); }
template <int DH>
__device__ __forceinline__ void pm_af_park(float* s, int lane, const float4* r) {
  using A = PmAf<DH>;
#pragma unroll
  for (int j = 0; j < A::PER; ++j) {
    const int c = (lane + 64 * j) % A::PIECES;
    float* p = s + (c / (DH / 4)) * A::ST + (c % (DH / 4)) * 2;
    *reinterpret_cast<float2*>(p) = make_float2(r[j].x, r[j].z);
    *reinterpret_cast<float2*>(p + A::HALF) = make_float2(r[j].y, r[j].w);
  }
}
// this lane's entries 2 c + g of a row of X
template <typename T, int DH, bool VEC>
__device__ __forceinline__ void pm_af_own(const T* X, int64_t d, int row, int g, float* x) {
#pragma unroll
  for (int c = 0; c < DH; c += 4) {
    const float4 v = pm_af_ld4<VEC>(X + (int64_t)row * d + c);
    x[c / 2] = g ? v.y : v.x;
    x[c / 2 + 1] = g ? v.w : v.z;
  }
}
// out^T [streamed row][owned row] = tile rows . owned rows
template <int DH>
__device__ __forceinline__ pm_f32x16 pm_af_scores(const float* s, const float* own, int lane) {
  using A = PmAf<DH>;
  pm_f32x16 acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
  const float* p = s + (lane & 31) * A::ST + (lane >> 5) * A::HALF;
#pragma unroll
  for (int c = 0; c < A::HALF; ++c) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(p[c], own[c], acc, 0, 0, 0);
  return acc;
}
// acc[dt] [head dimension][owned row] += tile^T . x, streamed rows in order
template <int DH>
__device__ __forceinline__ void pm_af_second(pm_f32x16* acc, const float* s, const float* x, int lane) {
  using A = PmAf<DH>;
  const float* p = s + (lane >> 5) * A::ST + pm_af_pos<DH>(lane & 31);
  auto step = [&](int r, float w) __attribute__((always_inline)) {              // rows r and r + 1
#pragma unroll
    for (int dt = 0; dt < A::NDT; ++dt)
      acc[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(p[r * A::ST + dt * 16], w, acc[dt], 0, 0, 0);
  };
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    // values 4 a .. 4 a + 3: rows 8 a .. 8 a + 3 in group 0, 8 a + 4 .. 8 a + 7 in group 1
    const auto w0 = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[4 * a]), __float_as_uint(x[4 * a + 1]), false, false);
    const auto w1 = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[4 * a + 2]), __float_as_uint(x[4 * a + 3]), false, false);
    step(8 * a, __uint_as_float(w0[0]));
    step(8 * a + 2, __uint_as_float(w1[0]));
    step(8 * a + 4, __uint_as_float(w0[1]));
    step(8 * a + 6, __uint_as_float(w1[1]));
  }
}
template <typename T, int DH, bool VEC>
__device__ __forceinline__ void pm_af_store(T* out_row, const pm_f32x16* acc, int lane) {
#pragma unroll
  for (int dt = 0; dt < PmAf<DH>::NDT; ++dt)
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const int c = dt * 32 + 8 * a + 4 * (lane >> 5);
      if (c < DH) pm_af_st4<VEC>(out_row + c, make_float4(acc[dt][4 * a], acc[dt][4 * a + 1], acc[dt][4 * a + 2], acc[dt][4 * a + 3]));
    }
}

// blockIdx.x = block of 32 owned rows * BH + (sequence, head)
template <typename T, int DH, bool VEC>
__device__ __forceinline__ void pm_attn_f32_dq_block(float* smem, int block, const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
                                                     const T* __restrict__ o, const T* __restrict__ dO,
                                                     const float* __restrict__ lse, T* __restrict__ dq, int S, int H, int BH,
                                                     float scale) {
  using A = PmAf<DH>;
  float *sK = smem, *sV = smem + A::ELEMS;
  const int bh = block % BH, qb = (S + 31) / 32 - 1 - block / BH;                // long blocks first
  const int b = bh / H, h = bh % H, d = H * DH, lane = threadIdx.x, ql = lane & 31, g = lane >> 5;
  const int64_t base = (int64_t)b * S * d + (int64_t)h * DH;
  const int q0 = qb * 32, qi = q0 + ql, qr = qi < S ? qi : S - 1;
  float own[A::HALF], od[A::HALF], D = 0.f;
#pragma unroll
  for (int c = 0; c < DH; c += 4) {
    const float4 x = pm_af_ld4<VEC>(dO + base + (int64_t)qr * d + c), y = pm_af_ld4<VEC>(o + base + (int64_t)qr * d + c);
    D = fmaf(x.x, y.x, D);
    D = fmaf(x.y, y.y, D);
    D = fmaf(x.z, y.z, D);
    D = fmaf(x.w, y.w, D);
    od[c / 2] = g ? x.y : x.x;
    od[c / 2 + 1] = g ? x.w : x.z;
  }
  pm_af_own<T, DH, VEC>(q + base, d, qr, g, own);
  const float L = lse[((int64_t)b * H + h) * S + qr];
  pm_f32x16 acc[A::NDT];
#pragma unroll
  for (int dt = 0; dt < A::NDT; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[dt][e] = 0.f;
  float4 rk[A::PER], rv[A::PER];
  pm_af_load<T, DH, VEC>(k + base, d, 0, S, lane, rk);
  pm_af_load<T, DH, VEC>(v + base, d, 0, S, lane, rv);
  for (int jt = 0; jt <= qb; ++jt) {
    pm_af_park<DH>(sK, lane, rk);
    pm_af_park<DH>(sV, lane, rv);
    const bool odd = jt == qb && pm_af_odd<A::PER>(rk);
    __syncthreads();
    if (jt < qb) {                                 // the next tile is on its way while this one is multiplied
      pm_af_load<T, DH, VEC>(k + base, d, (jt + 1) * 32, S, lane, rk);
      pm_af_load<T, DH, VEC>(v + base, d, (jt + 1) * 32, S, lane, rv);
    }
    const pm_f32x16 s = pm_af_scores<DH>(sK, own, lane), dp = pm_af_scores<DH>(sV, od, lane);
    float ds[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const float p = pm_af_exp(fmaf(s[e], scale, -L));
      ds[e] = p * (dp[e] - D) * scale;
      if (jt == qb && jt * 32 + 8 * (e >> 2) + 4 * g + (e & 3) > qi) ds[e] = 0.f;      // causal mask (keys past the end too)
    }
    if (odd) {
#pragma unroll 1
      for (int j = q0; j < S && j < q0 + 32; ++j) {
        const int64_t rj = base + (int64_t)j * d, ri = base + (int64_t)qr * d;
        const float pj = pm_af_exp(fmaf(pm_at_dot<T, DH>(q + ri, k + rj), scale, -L));
        pm_at_add_row<T, DH>(acc, k + rj, pj * (pm_at_dot<T, DH>(dO + ri, v + rj) - D) * scale, j <= qi, lane);
      }
    } else {
      pm_af_second<DH>(acc, sK, ds, lane);
    }
    __syncthreads();
  }
  if (qi < S) pm_af_store<T, DH, VEC>(dq + base + (int64_t)qi * d, acc, lane);
}

template <int DH>
constexpr int PM_AF_BWD_LDS = 2 * PmAf<DH>::ELEMS + 32 * PmAf<DH>::ST + 64;      // floats of LDS of a block of either kernel
template <typename T, int DH, bool VEC>
__device__ __forceinline__ void pm_attn_f32_dkv_block(float* smem, int block, const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
                                                      const T* __restrict__ o, const T* __restrict__ dO,
                                                      const float* __restrict__ lse, T* __restrict__ dk, T* __restrict__ dv,
                                                      int S, int H, int BH, float scale) {
  using A = PmAf<DH>;
  float *sQ = smem, *sO = sQ + A::ELEMS, *sX = sO + A::ELEMS, *sL = sX + 32 * A::ST, *sD = sL + 32;
  const int bh = block % BH, kb = block / BH;                                    // long blocks (early keys) first
  const int b = bh / H, h = bh % H, d = H * DH, lane = threadIdx.x, kl = lane & 31, g = lane >> 5;
  const int64_t base = (int64_t)b * S * d + (int64_t)h * DH;
  const int ki = kb * 32 + kl, kr = ki < S ? ki : S - 1;
  float ok[A::HALF], ov[A::HALF];
  pm_af_own<T, DH, VEC>(k + base, d, kr, g, ok);
  pm_af_own<T, DH, VEC>(v + base, d, kr, g, ov);
  pm_f32x16 ak[A::NDT], av[A::NDT];
#pragma unroll
  for (int dt = 0; dt < A::NDT; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      ak[dt][e] = 0.f;
      av[dt][e] = 0.f;
    }
  const int n_tiles = (S + 31) / 32;
  float4 rq[A::PER], rd[A::PER], ro[A::PER];
  float L = 0.f;
  auto load = [&](int it) __attribute__((always_inline)) {
    pm_af_load<T, DH, VEC>(q + base, d, it * 32, S, lane, rq);
    pm_af_load<T, DH, VEC>(dO + base, d, it * 32, S, lane, rd);
    pm_af_load<T, DH, VEC>(o + base, d, it * 32, S, lane, ro);
    const int row = it * 32 + kl;
    L = lse[((int64_t)b * H + h) * S + (row < S ? row : S - 1)];
  };
  load(kb);
  for (int it = kb; it < n_tiles; ++it) {
    pm_af_park<DH>(sQ, lane, rq);
    pm_af_park<DH>(sO, lane, rd);
    pm_af_park<DH>(sX, lane, ro);
    const bool odd = (it == kb || it * 32 + 32 > S) && (pm_af_odd<A::PER>(rq) | pm_af_odd<A::PER>(rd));
    if (lane < 32) sL[lane] = L;
    __syncthreads();
    if (it + 1 < n_tiles) load(it + 1);
    {                                              // D of row kl: both lane groups compute it
      const float *x = sO + kl * A::ST, *y = sX + kl * A::ST;
      float D = 0.f;
#pragma unroll
      for (int c = 0; c < A::HALF; ++c) {
        D = fmaf(x[c], y[c], D);
        D = fmaf(x[A::HALF + c], y[A::HALF + c], D);
      }
      if (lane < 32) sD[lane] = D;
    }
    const pm_f32x16 s = pm_af_scores<DH>(sQ, ok, lane), dp = pm_af_scores<DH>(sO, ov, lane);
    __syncthreads();
    float p[16], ds[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int r = 8 * (e >> 2) + 4 * g + (e & 3), qi = it * 32 + r;
      p[e] = pm_af_exp(fmaf(s[e], scale, -sL[r]));
      ds[e] = p[e] * (dp[e] - sD[r]) * scale;
      if (qi < ki || qi >= S) p[e] = ds[e] = 0.f;
    }
    if (odd) {
#pragma unroll 1
      for (int i = it * 32; i < S && i < it * 32 + 32; ++i) {
        const int64_t ri = base + (int64_t)i * d, rj = base + (int64_t)kr * d;
        const float pi = pm_af_exp(fmaf(pm_at_dot<T, DH>(q + ri, k + rj), scale, -sL[i - it * 32]));
        const float di = pi * (pm_at_dot<T, DH>(dO + ri, v + rj) - sD[i - it * 32]) * scale;
        pm_at_add_row<T, DH>(av, dO + ri, pi, i >= ki, lane);
        pm_at_add_row<T, DH>(ak, q + ri, di, i >= ki, lane);
      }
    } else {
      pm_af_second<DH>(av, sO, p, lane);
      pm_af_second<DH>(ak, sQ, ds, lane);
    }
    __syncthreads();
  }
  if (ki < S) {
    pm_af_store<T, DH, VEC>(dk + base + (int64_t)ki * d, ak, lane);
    pm_af_store<T, DH, VEC>(dv + base + (int64_t)ki * d, av, lane);
  }
}

// As launches of their own, and as one with the dK / dV blocks first (see pm_attn_mfma_bwd_kernel).
template <typename T, int DH, bool VEC>
__global__ __launch_bounds__(64) void pm_attn_f32_dq_kernel(const T* q, const T* k, const T* v, const T* o, const T* dO, const float* lse, T* dq,
                                                            int S, int H, int BH, float scale) {
  __shared__ __attribute__((aligned(16))) float smem[2 * PmAf<DH>::ELEMS];
  pm_attn_f32_dq_block<T, DH, VEC>(smem, blockIdx.x, q, k, v, o, dO, lse, dq, S, H, BH, scale);
}
template <typename T, int DH, bool VEC>
__global__ __launch_bounds__(64) void pm_attn_f32_dkv_kernel(const T* q, const T* k, const T* v, const T* o, const T* dO, const float* lse, T* dk, T* dv,
                                                             int S, int H, int BH, float scale) {
  __shared__ __attribute__((aligned(16))) float smem[PM_AF_BWD_LDS<DH>];
  pm_attn_f32_dkv_block<T, DH, VEC>(smem, blockIdx.x, q, k, v, o, dO, lse, dk, dv, S, H, BH, scale);
}
template <typename T, int DH, bool VEC>
__global__ __launch_bounds__(64) void pm_attn_f32_bwd_kernel(const T* q, const T* k, const T* v, const T* o, const T* dO, const float* lse, T* dq, T* dk, T* dv,
                                                             int S, int H, int BH, float scale) {
  __shared__ __attribute__((aligned(16))) float smem[PM_AF_BWD_LDS<DH>];
  const int n = gridDim.x / 2;
  if ((int)blockIdx.x < n) pm_attn_f32_dkv_block<T, DH, VEC>(smem, blockIdx.x, q, k, v, o, dO, lse, dk, dv, S, H, BH, scale);
  else pm_attn_f32_dq_block<T, DH, VEC>(smem, blockIdx.x - n, q, k, v, o, dO, lse, dq, S, H, BH, scale);
}
