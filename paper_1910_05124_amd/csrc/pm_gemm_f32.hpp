// fp32 products of the stages on the fp32 matrix instruction (gfx950).
//
//   C[i, j] = sum_k A(i, k) * B(j, k),   v_mfma_f32_16x16x4_f32 (fp32 operands, fp32 accumulation).
//
// Operands are "KC" (contraction index contiguous) or "RC" (row index contiguous) as in pm_gemm_mfma.hpp.  The networks
// trained in fp32 are small: a product has 10^5 .. 10^9 multiply-adds, and what bounds it is the latency of its first loads
// and of its chain of additions, not the matrix rate.  So the operands go from memory to the matrix instruction's
// registers without a stop in LDS (no barrier in the main loop), several 16-deep pieces of the contraction in flight ahead
// of those being multiplied.  A dependent 16 x 16 x 4 step takes 12.9 ns from registers, 3.2 ns per index; here an
// index costs 7 ns (100 x 4096 x 33: 31 us), a third of it the lane exchanges below (21 us without them), the rest loads.
// Staged through LDS, 32 x 32 outputs and 128 indices at a time, it was slower: 6.5 -> 7.7 us on 100 x 512 x 512, 31 -> 43.
//
// Order of the sums.  Every output is ONE chain of fused multiply-adds over k = 0, 1, 2, ... starting at zero: the
// instruction adds its four products to the accumulator one after the other, each addition rounded (checked bit for bit
// against fmaf chains, with wide exponents and denormal products).  A network with ReLU units turns a difference of one
// rounding in a pre-activation next to zero into a gradient that differs in the third digit, so the order is part of
// what a caller can rely on: splitting the contraction over waves or permuting it inside a piece made a 2-layer Transformer
// 256 wide differ by 5e-6 .. 1e-4 in its gradients on some inputs (4 of 24 seeds in a simulation), and is left out.  For the same reason a bias
// gradient adds rows m, m + 4, m + 8, ... in four chains and the chains in order.
//
// One lane of a 16 x 16 x 4 step s holds row lane % 16 and contraction index 4 s + lane / 16 of each operand.  A KC
// operand is one 16-byte load per lane and 16-deep piece (lane group g takes indices 4 g .. 4 g + 3) and four lane
// exchanges that transpose the 4 x 4 registers x lane groups; an RC operand with two 16-row tiles per wave gives tile t
// the rows 2 m + t, so that a lane loads its two rows with one 8-byte access.
//
// Measured (us per launch; before: 16 x 16 outputs per 256-thread block on vector FMAs through LDS): 100 x 512 x 512
// forward 21.9 -> 7.4, data gradient 20.6 -> 8.5 (4.6 and 4.3 with the contraction over eight waves); 512 x 1024 x 256 with
// the residual 25.5 -> 12.1.  More than four pieces ahead gained nothing.  The weight gradients of a step and their bias
// gradients were two launches per unit and are one now: 120 -> 16 us on the 9 units of that first network (8 of them 512
// wide), 615 -> 35 us on a 2-layer Transformer 256 wide with 512 tokens.
#pragma once
#include "pm_common.hpp"
#include "pm_elem.hpp"

typedef float pm_f32x4 __attribute__((ext_vector_type(4)));

// T x T matrix tiles of 16 x 16 per wave, WI x WJ waves over the block's outputs, U pieces in flight ahead
template <int T_, int WI_, int WJ_, int U_>
struct PmF32Cfg {
  static constexpr int T = T_, WI = WI_, WJ = WJ_, U = U_, NT = WI_ * WJ_ * 64;
  static constexpr int BI = WI_ * T_ * 16, BJ = WJ_ * T_ * 16, RS = BJ + 4;       // RS: padded row of the output tile
  static constexpr int lds_floats = BI * RS;
};

template <class Epi>
struct PmF32Prob {
  int I, J, K;
  const float* A;
  int64_t lda;
  PmWLoc<float> B;
  int64_t ldb;
  Epi epi;
};

// One wave's share of an operand: T tiles of 16 rows from row r0 on.  V: whole 16-byte (KC) / 8-byte (RC) accesses are
// allowed.  Rows beyond the extent R repeat the last one (their results are not stored).
template <int T, bool KC, bool V>
struct PmF32Operand {
  const float* p[T];
  int64_t ld;
  int g;
  __device__ __forceinline__ void init(const float* X, int64_t ld_, int r0, int R, int lane) {
    const int m = lane & 15;
    ld = ld_;
    g = lane >> 4;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      int row = KC ? r0 + 16 * t + m : r0 + T * m + t;
      // (a vector access of an RC operand starts at an even row and R is even then: both rows are inside or neither)
      if (row >= R) row = (!KC && V) ? R - T + t : R - 1;
      p[t] = KC ? X + (int64_t)row * ld : X + row;
    }
  }
  // the 16-deep piece at k0, all of it inside the contraction: x[s][t] = row t's value of index k0 + 4 s + lane / 16.
  // (KC with vector accesses: what arrives is index k0 + 4 (lane / 16) + s, see arrange)
  __device__ __forceinline__ void load(int k0, float (&x)[4][T]) const {
    if constexpr (KC && V) {
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const float4 v = *reinterpret_cast<const float4*>(p[t] + k0 + 4 * g);
        x[0][t] = v.x; x[1][t] = v.y; x[2][t] = v.z; x[3][t] = v.w;
      }
    } else {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int64_t o = KC ? (int64_t)(k0 + 4 * s + g) : (int64_t)(k0 + 4 * s + g) * ld;
        if constexpr (V && T == 2) {
          const float2 v = *reinterpret_cast<const float2*>(p[0] + o);
          x[s][0] = v.x; x[s][1] = v.y;
        } else {
#pragma unroll
          for (int t = 0; t < T; ++t) x[s][t] = p[t][o];
        }
      }
    }
  }
  // after the load has arrived: registers s x lane groups g transposed, so that register s holds index 4 s + g
  __device__ __forceinline__ void arrange(float (&x)[4][T]) const {
    if constexpr (KC && V) {
#pragma unroll
      for (int t = 0; t < T; ++t) {
        auto bits = [](float f) { return __float_as_uint(f); };
        const auto a = __builtin_amdgcn_permlane32_swap(bits(x[0][t]), bits(x[2][t]), false, false);
        const auto b = __builtin_amdgcn_permlane32_swap(bits(x[1][t]), bits(x[3][t]), false, false);
        const auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
        const auto d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
        x[0][t] = __uint_as_float(c[0]); x[1][t] = __uint_as_float(c[1]);
        x[2][t] = __uint_as_float(d[0]); x[3][t] = __uint_as_float(d[1]);
      }
    }
  }
  // the piece that crosses the end of the contraction, arranged already: zeros beyond it
  __device__ __forceinline__ void load_tail(int k0, int K, float (&x)[4][T]) const {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int k = k0 + 4 * s + g;
      const int64_t o = KC ? (int64_t)(k < K ? k : K - 1) : (int64_t)(k < K ? k : K - 1) * ld;
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const float v = p[t][o];
        x[s][t] = k < K ? v : 0.f;
      }
    }
  }
};

template <class Cfg, bool AKC, bool BKC, bool V, class Epi>
__device__ __forceinline__ void pm_gemm_f32_body(const PmF32Prob<Epi>& pr, Epi epi, int bx, int by, float* smem) {
  constexpr int T = Cfg::T, WJ = Cfg::WJ, BI = Cfg::BI, BJ = Cfg::BJ, RS = Cfg::RS, NT = Cfg::NT, U = Cfg::U;
  const int I = pr.I, J = pr.J, K = pr.K;
  const int i0 = by * BI, j0 = bx * BJ;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int wj = wave % WJ, wi = wave / WJ;
  PmF32Operand<T, AKC, V> oa;
  PmF32Operand<T, BKC, V> ob;
  oa.init(pr.A, pr.lda, i0 + wi * 16 * T, I, lane);
  ob.init(pr.B.get(), pr.ldb, j0 + wj * 16 * T, J, lane);

  pm_f32x4 acc[T][T];
#pragma unroll
  for (int a = 0; a < T; ++a)
#pragma unroll
    for (int b = 0; b < T; ++b) acc[a][b] = pm_f32x4{0.f, 0.f, 0.f, 0.f};
  float cs[T] = {};
  const bool do_colsum = Epi::kColSumA && !AKC && bx == 0 && wj == 0 && epi.wants_colsum();
  auto mul = [&](const float (&xa)[4][T], const float (&xb)[4][T]) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int a = 0; a < T; ++a)
#pragma unroll
        for (int b = 0; b < T; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[s][a], xb[s][b], acc[a][b], 0, 0, 0);
    if (Epi::kColSumA && !AKC) {
      if (do_colsum) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int a = 0; a < T; ++a) cs[a] += xa[s][a];
      }
    }
  };
  auto piece = [&](float (&xa)[4][T], float (&xb)[4][T]) __attribute__((always_inline)) {
    oa.arrange(xa);
    ob.arrange(xb);
    mul(xa, xb);
  };
  // whole pieces, U at a time with the next U on their way; the first group takes what is no multiple of U, and the
  // piece that crosses the end is requested before the last group is multiplied
  struct Group { float a[U][4][T], b[U][4][T]; };
  const int whole = K >> 4;
  const bool tail = K & 15;
  float ta[4][T], tb[4][T];
  Group x, y;
  int n = whole % U;
  if (n == 0 && whole > 0) n = U;
  const int first = n;
  auto load = [&](Group& q) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      oa.load((n + u) * 16, q.a[u]);
      ob.load((n + u) * 16, q.b[u]);
    }
    n += U;
    __builtin_amdgcn_sched_barrier(0);          // keep the requests ahead of the products
  };
  auto load_tail = [&]() __attribute__((always_inline)) {
    if (tail) {
      oa.load_tail(whole * 16, K, ta);
      ob.load_tail(whole * 16, K, tb);
    }
  };
  auto group = [&](Group& q, int have) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (u < have) piece(q.a[u], q.b[u]);
  };
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (u < first) {
      oa.load(u * 16, x.a[u]);
      ob.load(u * 16, x.b[u]);
    }
  if (n == whole) {
    load_tail();
    group(x, first);
  } else {
    load(y);
    group(x, first);
    while (n + U < whole) {                     // two groups at a time: the registers trade places
      load(x);
      group(y, U);
      load(y);
      group(x, U);
    }
    if (n < whole) {
      load(x);
      group(y, U);
      load_tail();
      group(x, U);
    } else {
      load_tail();
      group(y, U);
    }
  }
  if (tail) mul(ta, tb);

  if (Epi::kColSumA && !AKC) {
    if (do_colsum) {
#pragma unroll
      for (int a = 0; a < T; ++a) {
        // lane group g holds the chain of rows m = g mod 4; the four chains in order
        const float s1 = __shfl(cs[a], (lane & 15) + 16, 64), s2 = __shfl(cs[a], (lane & 15) + 32, 64), s3 = __shfl(cs[a], (lane & 15) + 48, 64);
        const int i = i0 + wi * 16 * T + T * lane + a;
        if (lane < 16 && i < I) epi.colsum(i, ((cs[a] + s1) + s2) + s3);
      }
    }
  }
  // accumulator layout of the 16 x 16 tile: value v of lane l is row 4 (l / 16) + v, column l % 16; through LDS so that
  // the stores are consecutive
#pragma unroll
  for (int a = 0; a < T; ++a)
#pragma unroll
    for (int b = 0; b < T; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = (lane >> 4) * 4 + v, c = lane & 15;
        const int li = wi * 16 * T + (AKC ? 16 * a + r : T * r + a), lj = wj * 16 * T + (BKC ? 16 * b + c : T * c + b);
        smem[li * RS + lj] = acc[a][b][v];
      }
  __syncthreads();
  epi.begin();
#pragma unroll
  for (int q = 0; q < BI * BJ / NT; ++q) {
    const int e = q * NT + threadIdx.x;
    const int li = e / BJ, lj = e % BJ, i = i0 + li, j = j0 + lj;
    if (i < I && j < J) epi(i, j, smem[li * RS + lj]);
  }
}

template <class Cfg, bool V, class Epi>
__global__ __launch_bounds__(Cfg::NT) void pm_gemm_f32_kernel(PmF32Prob<Epi> pr) {
  __shared__ float smem[Cfg::lds_floats];
  pm_gemm_f32_body<Cfg, Epi::kAKC, Epi::kBKC, V, Epi>(pr, pr.epi, blockIdx.x, blockIdx.y, smem);
}

// A table of problems in one launch: block b works on the problem p with first[p] <= b < first[p + 1].
template <class Cfg, bool V, class Epi>
__global__ __launch_bounds__(Cfg::NT) void pm_gemm_f32_grouped_kernel(const PmF32Prob<Epi>* __restrict__ probs, const int32_t* __restrict__ first, int np) {
  __shared__ float smem[Cfg::lds_floats];
  int lo = 0, hi = np - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (first[mid] <= (int)blockIdx.x) lo = mid; else hi = mid - 1;
  }
  const PmF32Prob<Epi> pr = probs[lo];
  const int id = (int)blockIdx.x - first[lo], tj = (pr.J + Cfg::BJ - 1) / Cfg::BJ;
  pm_gemm_f32_body<Cfg, Epi::kAKC, Epi::kBKC, V, Epi>(pr, pr.epi, id % tj, id / tj, smem);
}

// A wave tile of 16 x 16 takes 8 clocks per contraction index, one of 32 x 32 32 clocks with half the operand traffic per
// product: small tiles, and so more waves with shorter chains, up to two 64 x 64 blocks per compute unit.  Blocks of
// four such waves (which share operand lines in the first-level cache) once there is one for each compute unit.
using PmF32Small = PmF32Cfg<1, 1, 1, 4>;
using PmF32Mid = PmF32Cfg<1, 2, 2, 4>;
using PmF32Large = PmF32Cfg<2, 2, 2, 2>;
inline int64_t pm_f32_tiles(int I, int J, int b) { return (int64_t)((I + b - 1) / b) * ((J + b - 1) / b); }
// outputs per block edge for a launch with that many 32 x 32 and 64 x 64 tiles in total
inline int pm_f32_pick(int64_t tiles32, int64_t tiles64) { return tiles64 >= 512 ? 64 : tiles32 >= 256 ? 32 : 16; }

// Whether the operands allow the vector accesses.
template <class Epi>
inline bool pm_f32_vector(const PmF32Prob<Epi>& pr) {
  auto one = [&](bool kc, const void* X, int64_t stride, int64_t ld, int R) {
    return kc ? pr.K % 4 == 0 && ld % 4 == 0 && stride % 4 == 0 && ((uintptr_t)X & 15) == 0
              : R % 2 == 0 && ld % 2 == 0 && stride % 2 == 0 && ((uintptr_t)X & 7) == 0;
  };
  return one(Epi::kAKC, pr.A, 0, pr.lda, pr.I) && one(Epi::kBKC, pr.B.base, pr.B.stride, pr.ldb, pr.J);
}

template <class Epi>
inline void pm_gemm_f32_launch(hipStream_t st, const PmF32Prob<Epi>& pr) {
  auto go = [&](auto cfg) {
    using Cfg = decltype(cfg);
    const dim3 grid((pr.J + Cfg::BJ - 1) / Cfg::BJ, (pr.I + Cfg::BI - 1) / Cfg::BI);
    if (pm_f32_vector(pr)) hipLaunchKernelGGL((pm_gemm_f32_kernel<Cfg, true, Epi>), grid, dim3(Cfg::NT), 0, st, pr);
    else hipLaunchKernelGGL((pm_gemm_f32_kernel<Cfg, false, Epi>), grid, dim3(Cfg::NT), 0, st, pr);
  };
  switch (pm_f32_pick(pm_f32_tiles(pr.I, pr.J, 32), pm_f32_tiles(pr.I, pr.J, 64))) {
    case 64: go(PmF32Large()); break;
    case 32: go(PmF32Mid()); break;
    default: go(PmF32Small()); break;
  }
}

template <class Epi>
inline void pm_gemm_f32_grouped_launch(hipStream_t st, int block, bool vector, const PmF32Prob<Epi>* probs, const int32_t* first, int np, int tiles) {
  auto go = [&](auto cfg) {
    using Cfg = decltype(cfg);
    if (vector) hipLaunchKernelGGL((pm_gemm_f32_grouped_kernel<Cfg, true, Epi>), dim3(tiles), dim3(Cfg::NT), 0, st, probs, first, np);
    else hipLaunchKernelGGL((pm_gemm_f32_grouped_kernel<Cfg, false, Epi>), dim3(tiles), dim3(Cfg::NT), 0, st, probs, first, np);
  };
  switch (block) {
    case 64: go(PmF32Large()); break;
    case 32: go(PmF32Mid()); break;
    default: go(PmF32Small()); break;
  }
}
