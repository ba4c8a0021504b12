// Causal attention core in fp32 arithmetic on v_mfma_f32_32x32x2_f32, for fp32 contexts and for bf16 tensors with
// heads narrower than 32, gfx950.  T: element type of the tensors in memory; everything inside is fp32.
//
// The scheme is that of pm_attn_mfma.hpp: a wave owns 32 rows of one index and streams 32-row tiles of the other; the
// score-like products come out transposed, streamed index on the MFMA rows and owned index on the columns, so row
// statistics are per-lane scalars and the probabilities are the second product's B operand without leaving their
// lane.  The fp32 instruction contracts two indices at a time, lane group g = lane / 32 holding one of them, and the
// order of a contraction is free as long as both operands agree, hence:
//   * scores: group g holds head-dimension entries g DH / 2 .. + DH / 2 - 1 of its row, step c contracts the c-th of each
//     half: both operands are read as 16-byte pieces;
//   * second product: accumulator value v of group g is streamed row 8 (v / 4) + 4 g + v % 4, so step v contracts exactly
//     the two rows that the groups' values v stand for; the A operand is read column-wise from the tile in LDS.
// One wave per block (the tiles are private, no barrier but the wave's own): a tile costs 64 clocks per contracted pair
// - 2048 + 2048 clocks at DH = 64 - against 256 clocks to fetch it, so sharing tiles between waves would save nothing,
// and these shapes (a few dozen heads, sequences of at most 8192 / (DH + 1) rows) need the blocks to fill the chip.
// 8 sequences of 64 tokens, 8 heads of 32: forward 85 -> 5 us, backward 161 -> 15 us per layer against one thread per row.
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

// 32 rows of X (row stride d, rows past the end re-read the last one): registers first, LDS later
template <typename T, int DH>
__device__ __forceinline__ void pm_af_load(const T* X, int64_t d, int r0, int S, int lane, float4* r) {
  using A = PmAf<DH>;
#pragma unroll
  for (int j = 0; j < A::PER; ++j) {
    const int c = (lane + 64 * j) % A::PIECES;            // (fewer pieces than lanes: fetched more than once)
    int row = r0 + c / (DH / 4);
    row = row < S ? row : S - 1;
    r[j] = pm_ld4(X + (int64_t)row * d + (c % (DH / 4)) * 4);
  }
}
template <int DH>
__device__ __forceinline__ void pm_af_park(float* s, int lane, const float4* r) {
  using A = PmAf<DH>;
#pragma unroll
  for (int j = 0; j < A::PER; ++j) {
    const int c = (lane + 64 * j) % A::PIECES;
    *reinterpret_cast<float4*>(s + (c / (DH / 4)) * A::ST + (c % (DH / 4)) * 4) = r[j];
  }
}
// this lane's half of a row of X
template <typename T, int DH>
__device__ __forceinline__ void pm_af_own(const T* X, int64_t d, int row, int g, float* x) {
  const T* p = X + (int64_t)row * d + g * PmAf<DH>::HALF;
#pragma unroll
  for (int c = 0; c < PmAf<DH>::HALF; ++c) x[c] = ldf(p + c);
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
// acc[dt] [head dimension][owned row] += tile^T . x
template <int DH>
__device__ __forceinline__ void pm_af_second(pm_f32x16* acc, const float* s, const float* x, int lane) {
  using A = PmAf<DH>;
  const float* p = s + 4 * (lane >> 5) * A::ST + (lane & 31);
#pragma unroll
  for (int v = 0; v < 16; ++v)
#pragma unroll
    for (int dt = 0; dt < A::NDT; ++dt)
      acc[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(p[(8 * (v >> 2) + (v & 3)) * A::ST + dt * 32], x[v], acc[dt], 0, 0, 0);
}
template <typename T, int DH>
__device__ __forceinline__ void pm_af_store(T* out_row, const pm_f32x16* acc, float mul, int lane) {
#pragma unroll
  for (int dt = 0; dt < PmAf<DH>::NDT; ++dt)
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const int c = dt * 32 + 8 * a + 4 * (lane >> 5);
      if (c < DH)
        pm_st4(out_row + c, make_float4(acc[dt][4 * a] * mul, acc[dt][4 * a + 1] * mul, acc[dt][4 * a + 2] * mul, acc[dt][4 * a + 3] * mul));
    }
}

// blockIdx.x = block of 32 owned rows * BH + (sequence, head)
template <typename T, int DH>
__global__ __launch_bounds__(64) void pm_attn_f32_fwd_kernel(const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
                                                             T* __restrict__ o, float* __restrict__ lse, int S, int H, int BH,
                                                             float scale) {
  using A = PmAf<DH>;
  __shared__ __attribute__((aligned(16))) float sK[A::ELEMS], sV[A::ELEMS];
  const int bh = blockIdx.x % BH, qb = (S + 31) / 32 - 1 - blockIdx.x / BH;      // long blocks first
  const int b = bh / H, h = bh % H, d = H * DH, lane = threadIdx.x, ql = lane & 31, g = lane >> 5;
  const int64_t base = (int64_t)b * S * d + (int64_t)h * DH;
  const int q0 = qb * 32, qi = q0 + ql, qr = qi < S ? qi : S - 1;
  float own[A::HALF];
  pm_af_own<T, DH>(q + base, d, qr, g, own);
  pm_f32x16 acc[A::NDT];
#pragma unroll
  for (int dt = 0; dt < A::NDT; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[dt][e] = 0.f;
  float m = -3.0e38f, lsum = 0.f;
  float4 rk[A::PER], rv[A::PER];
  pm_af_load<T, DH>(k + base, d, 0, S, lane, rk);
  pm_af_load<T, DH>(v + base, d, 0, S, lane, rv);
  const float c2 = scale * 1.44269504f;            // scores in base-2 units
  for (int jt = 0; jt <= qb; ++jt) {
    pm_af_park<DH>(sK, lane, rk);
    pm_af_park<DH>(sV, lane, rv);
    __syncthreads();
    if (jt < qb) {                                 // the next tile is on its way while this one is multiplied
      pm_af_load<T, DH>(k + base, d, (jt + 1) * 32, S, lane, rk);
      pm_af_load<T, DH>(v + base, d, (jt + 1) * 32, S, lane, rv);
    }
    const pm_f32x16 s = pm_af_scores<DH>(sK, own, lane);
    float p[16], mx = -3.0e38f;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      p[e] = s[e] * c2;
      if (jt == qb && jt * 32 + 8 * (e >> 2) + 4 * g + (e & 3) > qi) p[e] = -3.0e38f;      // causal mask (keys past the end too)
      mx = fmaxf(mx, p[e]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mn = fmaxf(m, mx), corr = __builtin_amdgcn_exp2f(m - mn);
    float ps = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      p[e] = __builtin_amdgcn_exp2f(p[e] - mn);
      ps += p[e];
    }
    lsum = lsum * corr + ps;
#pragma unroll
    for (int dt = 0; dt < A::NDT; ++dt)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[dt][e] *= corr;
    m = mn;
    pm_af_second<DH>(acc, sV, p, lane);
    __syncthreads();
  }
  lsum += __shfl_xor(lsum, 32, 64);
  if (qi >= S) return;
  pm_af_store<T, DH>(o + base + (int64_t)qi * d, acc, 1.f / lsum, lane);
  if (g == 0) lse[((int64_t)b * H + h) * S + qi] = m * 0.693147181f + __logf(lsum);
}

template <typename T, int DH>
__global__ __launch_bounds__(64) void pm_attn_f32_dq_kernel(const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
                                                            const T* __restrict__ o, const T* __restrict__ dO,
                                                            const float* __restrict__ lse, T* __restrict__ dq, int S, int H, int BH,
                                                            float scale) {
  using A = PmAf<DH>;
  __shared__ __attribute__((aligned(16))) float sK[A::ELEMS], sV[A::ELEMS];
  const int bh = blockIdx.x % BH, qb = (S + 31) / 32 - 1 - blockIdx.x / BH;
  const int b = bh / H, h = bh % H, d = H * DH, lane = threadIdx.x, ql = lane & 31, g = lane >> 5;
  const int64_t base = (int64_t)b * S * d + (int64_t)h * DH;
  const int q0 = qb * 32, qi = q0 + ql, qr = qi < S ? qi : S - 1;
  float own[A::HALF], od[A::HALF], D = 0.f;
  pm_af_own<T, DH>(o + base, d, qr, g, own);
  pm_af_own<T, DH>(dO + base, d, qr, g, od);
#pragma unroll
  for (int c = 0; c < A::HALF; ++c) D += own[c] * od[c];
  D += __shfl_xor(D, 32, 64);
  pm_af_own<T, DH>(q + base, d, qr, g, own);
  const float c2 = scale * 1.44269504f, l2 = lse[((int64_t)b * H + h) * S + qr] * 1.44269504f;
  pm_f32x16 acc[A::NDT];
#pragma unroll
  for (int dt = 0; dt < A::NDT; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[dt][e] = 0.f;
  float4 rk[A::PER], rv[A::PER];
  pm_af_load<T, DH>(k + base, d, 0, S, lane, rk);
  pm_af_load<T, DH>(v + base, d, 0, S, lane, rv);
  for (int jt = 0; jt <= qb; ++jt) {
    pm_af_park<DH>(sK, lane, rk);
    pm_af_park<DH>(sV, lane, rv);
    __syncthreads();
    if (jt < qb) {
      pm_af_load<T, DH>(k + base, d, (jt + 1) * 32, S, lane, rk);
      pm_af_load<T, DH>(v + base, d, (jt + 1) * 32, S, lane, rv);
    }
    const pm_f32x16 s = pm_af_scores<DH>(sK, own, lane), dp = pm_af_scores<DH>(sV, od, lane);
    float ds[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      ds[e] = __builtin_amdgcn_exp2f(fmaf(s[e], c2, -l2)) * (dp[e] - D);       // the factor 1 / sqrt(dh) goes into the store
      if (jt == qb && jt * 32 + 8 * (e >> 2) + 4 * g + (e & 3) > qi) ds[e] = 0.f;
    }
    pm_af_second<DH>(acc, sK, ds, lane);
    __syncthreads();
  }
  if (qi < S) pm_af_store<T, DH>(dq + base + (int64_t)qi * d, acc, scale, lane);
}

template <typename T, int DH>
__global__ __launch_bounds__(64) void pm_attn_f32_dkv_kernel(const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
                                                             const T* __restrict__ o, const T* __restrict__ dO,
                                                             const float* __restrict__ lse, T* __restrict__ dk, T* __restrict__ dv,
                                                             int S, int H, int BH, float scale) {
  using A = PmAf<DH>;
  __shared__ __attribute__((aligned(16))) float sQ[A::ELEMS], sO[A::ELEMS], sL[32], sD[32];
  const int bh = blockIdx.x % BH, kb = blockIdx.x / BH;                          // long blocks (early keys) first
  const int b = bh / H, h = bh % H, d = H * DH, lane = threadIdx.x, kl = lane & 31, g = lane >> 5;
  const int64_t base = (int64_t)b * S * d + (int64_t)h * DH;
  const int ki = kb * 32 + kl, kr = ki < S ? ki : S - 1;
  float ok[A::HALF], ov[A::HALF];
  pm_af_own<T, DH>(k + base, d, kr, g, ok);
  pm_af_own<T, DH>(v + base, d, kr, g, ov);
  pm_f32x16 ak[A::NDT], av[A::NDT];
#pragma unroll
  for (int dt = 0; dt < A::NDT; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      ak[dt][e] = 0.f;
      av[dt][e] = 0.f;
    }
  const int n_tiles = (S + 31) / 32;
  const float c2 = scale * 1.44269504f;
  float4 rq[A::PER], rd[A::PER], ro[A::PER];
  float L = 0.f;
  auto load = [&](int it) __attribute__((always_inline)) {
    pm_af_load<T, DH>(q + base, d, it * 32, S, lane, rq);
    pm_af_load<T, DH>(dO + base, d, it * 32, S, lane, rd);
    pm_af_load<T, DH>(o + base, d, it * 32, S, lane, ro);
    const int row = it * 32 + kl;
    L = lse[((int64_t)b * H + h) * S + (row < S ? row : S - 1)] * 1.44269504f;
  };
  load(kb);
  for (int it = kb; it < n_tiles; ++it) {
    pm_af_park<DH>(sQ, lane, rq);
    pm_af_park<DH>(sO, lane, rd);
    // D of the tile's rows: the DH / 4 lanes that hold a row's pieces are neighbours
#pragma unroll
    for (int j = 0; j < A::PER; ++j) {
      float part = rd[j].x * ro[j].x + rd[j].y * ro[j].y + rd[j].z * ro[j].z + rd[j].w * ro[j].w;
#pragma unroll
      for (int m = 1; m < DH / 4; m <<= 1) part += __shfl_xor(part, m, 64);
      const int c = (lane + 64 * j) % A::PIECES;
      if (c % (DH / 4) == 0) sD[c / (DH / 4)] = part;
    }
    if (lane < 32) sL[lane] = L;
    __syncthreads();
    if (it + 1 < n_tiles) load(it + 1);
    const pm_f32x16 s = pm_af_scores<DH>(sQ, ok, lane), dp = pm_af_scores<DH>(sO, ov, lane);
    float p[16], ds[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int r = 8 * (e >> 2) + 4 * g + (e & 3), qi = it * 32 + r;
      p[e] = __builtin_amdgcn_exp2f(fmaf(s[e], c2, -sL[r]));
      if (qi < ki || qi >= S) p[e] = 0.f;
      ds[e] = p[e] * (dp[e] - sD[r]);
    }
    pm_af_second<DH>(av, sO, p, lane);
    pm_af_second<DH>(ak, sQ, ds, lane);
    __syncthreads();
  }
  if (ki < S) {
    pm_af_store<T, DH>(dk + base + (int64_t)ki * d, ak, scale, lane);
    pm_af_store<T, DH>(dv + base + (int64_t)ki * d, av, 1.f, lane);
  }
}
