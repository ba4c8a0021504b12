// 3x3 convolution stages (zero padding 1, stride 1 or 2) with a folded per-channel affine, ReLU and
// parameter-free residual shortcuts, for the ResNet-shaped stages of the training step.  gfx950.
//
// Activations are NHWC in the compute dtype T; pixel index p = (b * H + y) * W + x.  A convolution
// unit's parameters lie in one ring slot: W [C_out][tap = 3 dy + dx][C_in], then scale [C_out],
// shift [C_out].  forward:  z = conv(x, W_fwd);  a = scale_fwd * z + shift_fwd (+ shortcut);  y = relu(a).
// backward (two weight sets, Sec. 2.1): da = dy * [y > 0];  d scale = sum da * z;  d shift = sum da;
// dz = da * scale_bkwd;  dW = correlation of dz with the stored input;  d input = transposed convolution
// of dz with W_bkwd (+ da of the block's second convolution through the shortcut).
//
// The convolutions are implicit GEMMs on v_mfma_f32_32x32x16_bf16 (bf16, channel counts multiples
// of 16): no patch matrix is ever written.  Every product is computed transposed, channels on the
// MFMA rows and pixels on the MFMA columns, so a lane owns one pixel and 4 consecutive channels per
// accumulator group: the gathered operand (8 consecutive channels of one input pixel of one tap) is
// a single 16-byte global load, and results leave as 8-byte pieces of NHWC rows.
//   forward   out^T [co][pixel]    = sum_{tap, ci} W[co][tap][ci] x[pixel + tap][ci]
//   data      dx^T  [ci][in pixel] = sum_{tap, co} W[co][tap][ci] dz[pixel - tap][co]   (W transposed once per step)
//   weight    dW    [co][tap, ci]  = sum_{pixel}   dz[pixel][co] x[pixel + tap][ci]     (both operands via LDS transpose loads)
// These layers are bound by the latency of their loads and launches, not by the MFMA rate (channel counts of
// 16 .. 64 give 70 - 300 flop per byte of activation traffic): what counts is that a wave's loads are in flight
// together and that a step has few launches in a row.  fp32 contexts and channel counts beyond 64 or no multiple
// of 16 use the plain kernels below.
#pragma once
#include <type_traits>
#include "pm_common.hpp"
#include "pm_mfma_types.hpp"

struct PmConvGeom {
  int B, H, W, Cin, Cout, stride, Ho, Wo;   // input H x W, output Ho x Wo
};

// Shortcut added to a block's second convolution: the block input (Hs x Ws x Cs), subsampled by
// `stride` with the new channels zero.  src == nullptr: none.
template <typename T>
struct PmShortcut {
  const T* src;
  int Hs, Ws, Cs, stride;
  __device__ __forceinline__ float at(int b, int oy, int ox, int c) const {
    if (!src || c >= Cs) return 0.f;
    return ldf(src + (((int64_t)b * Hs + oy * stride) * Ws + ox * stride) * Cs + c);
  }
};

// Gradient that reaches a block's input through its shortcut: da of the block's second convolution
// (Ho x Wo x Co) placed on every stride-th input pixel, first Cin channels.
template <typename T>
struct PmShortcutBwd {
  const T* da;
  int Ho, Wo, Co, stride;
  __device__ __forceinline__ float at(int b, int iy, int ix, int c) const {
    if (!da) return 0.f;
    if (stride == 2 && ((iy | ix) & 1)) return 0.f;
    return ldf(da + (((int64_t)b * Ho + iy / stride) * Wo + ix / stride) * Co + c);
  }
};

// ---------------------------------------------------------------------------------------------
// plain kernels (any T, any channel counts)
// ---------------------------------------------------------------------------------------------
// NCHW fp32 image batch -> NHWC compute dtype
template <typename T>
__global__ __launch_bounds__(256) void pm_image_stage_kernel(const float* __restrict__ x, T* __restrict__ out, int B, int C,
                                                             int H, int W) {
  const int64_t total = (int64_t)B * H * W * C;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const int c = (int)(i % C);
    const int64_t p = i / C;
    const int xw = (int)(p % W), yh = (int)((p / W) % H), b = (int)(p / ((int64_t)W * H));
    stf(out + i, x[(((int64_t)b * C + c) * H + yh) * W + xw]);
  }
}

// The same for bf16 images of fewer than 16 channels whose convolution takes the matrix path: pixels of 16 channels,
// the missing ones zero.  The blocks from pix_blocks on pad the convolution's kernel tensor likewise
// ([co][tap][C] -> [co][tap][16]) and copy its scale and shift behind it.
__global__ __launch_bounds__(256) void pm_image_stage16_kernel(const float* __restrict__ x, bf16_t* __restrict__ out, int B, int C,
                                                               int HW, int pix_blocks, PmWLoc<bf16_t> wloc,
                                                               bf16_t* __restrict__ wpad, int Cout) {
  if ((int)blockIdx.x >= pix_blocks) {
    const bf16_t* w = wloc.get();
    const int n = Cout * 9 * 16, first = ((int)blockIdx.x - pix_blocks) * 256 + threadIdx.x, step = ((int)gridDim.x - pix_blocks) * 256;
    for (int i = first; i < n + 2 * Cout; i += step) {
      const int c = i & 15;
      wpad[i] = i >= n ? w[Cout * 9 * C + i - n] : c < C ? w[(i >> 4) * C + c] : (bf16_t)0;
    }
    return;
  }
  const int64_t total = (int64_t)B * HW;
  for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < total; p += (int64_t)pix_blocks * 256) {
    const int64_t b = p / HW, at = p - b * HW;
    float v[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) v[c] = c < C ? x[(b * C + c) * HW + at] : 0.f;
    pm_st8(out + p * 16, v);
    pm_st8(out + p * 16 + 8, v + 8);
  }
}
constexpr int PM_IMAGE_PAD_BLOCKS = 4;
// x == nullptr: the kernel tensor only
inline void pm_image_stage16_launch(hipStream_t st, const float* x, bf16_t* out, int B, int C, int HW, PmWLoc<bf16_t> w, bf16_t* wpad,
                                    int Cout) {
  const int pb = x ? (int)std::min<int64_t>(2048, ((int64_t)B * HW + 255) / 256) : 0;
  hipLaunchKernelGGL(pm_image_stage16_kernel, dim3((unsigned)(pb + PM_IMAGE_PAD_BLOCKS)), dim3(256), 0, st, x, out, B, C, HW, pb, w,
                     wpad, Cout);
}

template <typename T>
__global__ __launch_bounds__(256) void pm_conv_fwd_plain_kernel(PmConvGeom g, const T* __restrict__ x, PmWLoc<T> wloc,
                                                                PmShortcut<T> sc, T* __restrict__ z, T* __restrict__ y) {
  const T* Wt = wloc.get();
  const T* scale = Wt + (int64_t)g.Cout * 9 * g.Cin;
  const T* shift = scale + g.Cout;
  const int64_t total = (int64_t)g.B * g.Ho * g.Wo * g.Cout;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const int co = (int)(i % g.Cout);
    const int64_t p = i / g.Cout;
    const int ox = (int)(p % g.Wo), oy = (int)((p / g.Wo) % g.Ho), b = (int)(p / ((int64_t)g.Wo * g.Ho));
    float acc = 0.f;
    for (int dy = 0; dy < 3; ++dy) {
      const int iy = oy * g.stride + dy - 1;
      if (iy < 0 || iy >= g.H) continue;
      for (int dx = 0; dx < 3; ++dx) {
        const int ix = ox * g.stride + dx - 1;
        if (ix < 0 || ix >= g.W) continue;
        const T* xr = x + (((int64_t)b * g.H + iy) * g.W + ix) * g.Cin;
        const T* wr = Wt + ((int64_t)co * 9 + dy * 3 + dx) * g.Cin;
        for (int ci = 0; ci < g.Cin; ++ci) acc += ldf(xr + ci) * ldf(wr + ci);
      }
    }
    const float a = ldf(scale + co) * acc + ldf(shift + co) + sc.at(b, oy, ox, co);
    stf(z + i, acc);
    stf(y + i, a > 0.f ? a : 0.f);
  }
}

// Forward of the image layer (3 input channels, 16 output channels; fp32, and bf16 at the stand-alone entry): one thread per output pixel
// computes all 16 channels from the 27 inputs of its window, with the kernel tensor, scale and shift
// held in LDS as fp32 (every lane reads the same entry: a broadcast); outputs go out as 16-byte pieces.
// The one-thread-per-output-element kernel above spends 61 us on the 128 x 32 x 32 images of the
// ResNet workload (2-byte loads, a 27-element stride between the lanes' weights), this one a few.
template <typename T>
__global__ __launch_bounds__(256) void pm_conv_fwd_thin_kernel(PmConvGeom g, const T* __restrict__ x, PmWLoc<T> wloc,
                                                               PmShortcut<T> sc, T* __restrict__ z, T* __restrict__ y) {
  constexpr int CO = 16, CI = 3, NW = CO * 9 * CI;
  __shared__ float sw[NW + 2 * CO];                   // W [CO][9][CI], then scale [CO], shift [CO] (as in memory)
  const T* Wt = wloc.get();
  for (int i = threadIdx.x; i < NW + 2 * CO; i += blockDim.x) sw[i] = ldf(Wt + i);
  __syncthreads();
  const int64_t npix = (int64_t)g.B * g.Ho * g.Wo;
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < npix; p += (int64_t)gridDim.x * blockDim.x) {
    const int ox = (int)(p % g.Wo), oy = (int)((p / g.Wo) % g.Ho), b = (int)(p / ((int64_t)g.Wo * g.Ho));
    float acc[CO];
#pragma unroll
    for (int co = 0; co < CO; ++co) acc[co] = 0.f;
#pragma unroll
    for (int dy = 0; dy < 3; ++dy) {
      const int iy = oy * g.stride + dy - 1;
      if (iy < 0 || iy >= g.H) continue;
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) {
        const int ix = ox * g.stride + dx - 1;
        if (ix < 0 || ix >= g.W) continue;
        const T* xr = x + (((int64_t)b * g.H + iy) * g.W + ix) * CI;
        const float x0 = ldf(xr), x1 = ldf(xr + 1), x2 = ldf(xr + 2);
        const float* w = sw + (dy * 3 + dx) * CI;
#pragma unroll
        for (int co = 0; co < CO; ++co) {             // same order of additions as the plain kernel
          acc[co] = fmaf(x0, w[co * 9 * CI], acc[co]);
          acc[co] = fmaf(x1, w[co * 9 * CI + 1], acc[co]);
          acc[co] = fmaf(x2, w[co * 9 * CI + 2], acc[co]);
        }
      }
    }
    float a[CO];
#pragma unroll
    for (int co = 0; co < CO; ++co) {
      const float v = sw[NW + co] * acc[co] + sw[NW + CO + co] + sc.at(b, oy, ox, co);
      a[co] = v > 0.f ? v : 0.f;
    }
    pm_st8(z + p * CO, acc);
    pm_st8(z + p * CO + 8, acc + 8);
    pm_st8(y + p * CO, a);
    pm_st8(y + p * CO + 8, a + 8);
  }
}

template <typename T>
__global__ __launch_bounds__(256) void pm_conv_dgrad_plain_kernel(PmConvGeom g, const T* __restrict__ dz, PmWLoc<T> wloc,
                                                                  PmShortcutBwd<T> sb, T* __restrict__ dx) {
  const T* Wt = wloc.get();
  const int64_t total = (int64_t)g.B * g.H * g.W * g.Cin;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const int ci = (int)(i % g.Cin);
    const int64_t p = i / g.Cin;
    const int ix = (int)(p % g.W), iy = (int)((p / g.W) % g.H), b = (int)(p / ((int64_t)g.W * g.H));
    float acc = 0.f;
    for (int dy = 0; dy < 3; ++dy) {
      const int ny = iy + 1 - dy;
      if (ny < 0 || ny % g.stride) continue;
      const int oy = ny / g.stride;
      if (oy >= g.Ho) continue;
      for (int dxx = 0; dxx < 3; ++dxx) {
        const int nx = ix + 1 - dxx;
        if (nx < 0 || nx % g.stride) continue;
        const int ox = nx / g.stride;
        if (ox >= g.Wo) continue;
        const T* dr = dz + (((int64_t)b * g.Ho + oy) * g.Wo + ox) * g.Cout;
        const T* wr = Wt + (int64_t)(dy * 3 + dxx) * g.Cin + ci;
        for (int co = 0; co < g.Cout; ++co) acc += ldf(dr + co) * ldf(wr + (int64_t)co * 9 * g.Cin);
      }
    }
    stf(dx + i, acc + sb.at(b, iy, ix, ci));
  }
}

// one block per weight element (co, tap, ci): sum over all output pixels
template <typename T>
__global__ __launch_bounds__(256) void pm_conv_wgrad_plain_kernel(PmConvGeom g, const T* __restrict__ dz,
                                                                  const T* __restrict__ x, float* __restrict__ dW,
                                                                  int accumulate) {
  const int e = blockIdx.x;
  const int ci = e % g.Cin, tap = (e / g.Cin) % 9, co = e / (9 * g.Cin);
  const int dy = tap / 3, dxx = tap % 3;
  const int64_t npix = (int64_t)g.B * g.Ho * g.Wo;
  float acc = 0.f;
  for (int64_t p = threadIdx.x; p < npix; p += blockDim.x) {
    const int ox = (int)(p % g.Wo), oy = (int)((p / g.Wo) % g.Ho), b = (int)(p / ((int64_t)g.Wo * g.Ho));
    const int iy = oy * g.stride + dy - 1, ix = ox * g.stride + dxx - 1;
    if (iy < 0 || iy >= g.H || ix < 0 || ix >= g.W) continue;
    acc += ldf(dz + p * g.Cout + co) * ldf(x + (((int64_t)b * g.H + iy) * g.W + ix) * g.Cin + ci);
  }
  acc = pm_wave_sum(acc);
  __shared__ float part[4];
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    const float s = part[0] + part[1] + part[2] + part[3];
    dW[e] = accumulate ? dW[e] + s : s;
  }
}

// weight gradient of a convolution with very few input channels (the 3-channel input layer), any T.
// grid (pixel groups, 9 taps); a thread walks pixels of its group and keeps the CO x CI outer-product
// sums of its pixels in registers; wave shuffles, then LDS across the four waves; the block writes
// its partial of the tap to scratch [group][co][tap][ci] for pm_conv_reduce_kernel.
template <typename T, int CO, int CI>
__global__ __launch_bounds__(256) void pm_conv_wgrad_thin_kernel(PmConvGeom g, const T* __restrict__ dz,
                                                                 const T* __restrict__ x, float* __restrict__ part) {
  const int tap = blockIdx.y, dy = tap / 3 - 1, dx = tap % 3 - 1;
  const int npix = g.B * g.Ho * g.Wo;
  float acc[CO][CI];
#pragma unroll
  for (int a = 0; a < CO; ++a)
#pragma unroll
    for (int b = 0; b < CI; ++b) acc[a][b] = 0.f;
  for (int p = blockIdx.x * 256 + threadIdx.x; p < npix; p += gridDim.x * 256) {
    const unsigned up = (unsigned)p, wo = (unsigned)g.Wo, ho = (unsigned)g.Ho;
    const int ox = (int)(up % wo), oy = (int)((up / wo) % ho), bb = (int)(up / (wo * ho));
    const int iy = oy * g.stride + dy, ix = ox * g.stride + dx;
    if (iy < 0 || iy >= g.H || ix < 0 || ix >= g.W) continue;
    float xv[CI], dv[CO];
    const T* xr = x + ((int64_t)(bb * g.H + iy) * g.W + ix) * CI;
#pragma unroll
    for (int b = 0; b < CI; ++b) xv[b] = ldf(xr + b);
#pragma unroll
    for (int a = 0; a < CO; a += 8) pm_ld8(dz + (int64_t)p * CO + a, dv + a);
#pragma unroll
    for (int a = 0; a < CO; ++a)
#pragma unroll
      for (int b = 0; b < CI; ++b) acc[a][b] += dv[a] * xv[b];
  }
  __shared__ float red[4][CO * CI];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
  for (int a = 0; a < CO; ++a)
#pragma unroll
    for (int b = 0; b < CI; ++b) {
      const float s = pm_wave_sum(acc[a][b]);
      if (lane == 0) red[wave][a * CI + b] = s;
    }
  __syncthreads();
  if (threadIdx.x < CO * CI) {
    const int a = threadIdx.x / CI, b = threadIdx.x % CI;
    part[(int64_t)blockIdx.x * (CO * 9 * CI) + ((int64_t)a * 9 + tap) * CI + b] =
        red[0][threadIdx.x] + red[1][threadIdx.x] + red[2][threadIdx.x] + red[3][threadIdx.x];
  }
}
constexpr int PM_CONV_THIN_GROUPS = 64;

// da = dy * [y > 0];  dz = da * scale_bkwd;  dscale += sum da * z;  dshift += sum da.  The caller zeroes
// dscale / dshift at the start of a minibatch.  With `part` the block writes its sums to
// part[block][0 = scale | 1 = shift][C] and the reduce launch that ends the backward pass adds them up
// (hundreds of blocks adding into the same few dozen addresses with fp32 atomics serialise: that tail
// cost more than the streaming part of the kernel); without it, fp32 atomics.  Thread t of a block always
// sees channel (t * 8 .. t * 8 + 7) mod C because a block's span is a multiple of C elements.
template <typename T>
__global__ __launch_bounds__(256) void pm_conv_affine_bwd_kernel(const T* __restrict__ dy, const T* __restrict__ y,
                                                                 const T* __restrict__ z, PmWLoc<T> scale_bkwd,
                                                                 T* __restrict__ da, T* __restrict__ dz,
                                                                 float* __restrict__ dscale, float* __restrict__ dshift,
                                                                 float* __restrict__ part, int64_t total, int C) {
  __shared__ float red[4][2][256];
  const T* sbk = scale_bkwd.get();
  const int c0 = (threadIdx.x * 8) % C;            // C is a power of two, 8 <= C <= 256
  float s8[8], as[8], at[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    s8[e] = ldf(sbk + c0 + e);
    as[e] = 0.f;
    at[e] = 0.f;
  }
  for (int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8; i < total; i += (int64_t)gridDim.x * 2048) {
    float a[8], b[8], c[8], o1[8], o2[8];
    pm_ld8(dy + i, a);
    pm_ld8(y + i, b);
    pm_ld8(z + i, c);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float d = b[e] > 0.f ? a[e] : 0.f;
      o1[e] = d;
      o2[e] = d * s8[e];
      as[e] += d * c[e];
      at[e] += d;
    }
    pm_st8(da + i, o1);
    pm_st8(dz + i, o2);
  }
  // lanes l and l + C / 8 (mod 64) own the same channels: butterfly over the lane bits above C / 8, then
  // the four waves meet in LDS (plain stores: LDS float atomics are slow), one fp32 atomic per channel and block
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, per = C >> 3;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    for (int o = 32; o >= per && o > 0; o >>= 1) {
      as[e] += __shfl_xor(as[e], o, 64);
      at[e] += __shfl_xor(at[e], o, 64);
    }
  }
  if (lane < per || per > 64) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      red[wave][0][c0 + e] = as[e];
      red[wave][1][c0 + e] = at[e];
    }
  }
  __syncthreads();
  for (int j = threadIdx.x; j < C; j += 256) {
    const float vs = red[0][0][j] + red[1][0][j] + red[2][0][j] + red[3][0][j];
    const float vt = red[0][1][j] + red[1][1][j] + red[2][1][j] + red[3][1][j];
    if (part) {
      part[((int64_t)blockIdx.x * 2 + 0) * C + j] = vs;
      part[((int64_t)blockIdx.x * 2 + 1) * C + j] = vt;
    } else {
      atomicAdd(dscale + j, vs);
      atomicAdd(dshift + j, vt);
    }
  }
}

// global average pool: out[b][c] = mean over the HW pixels
template <typename T>
__global__ __launch_bounds__(256) void pm_pool_fwd_kernel(const T* __restrict__ y, T* __restrict__ out, int B, int HW, int C) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= B * C) return;
  const int b = i / C, c = i % C;
  float acc = 0.f;
  for (int p = 0; p < HW; ++p) acc += ldf(y + ((int64_t)b * HW + p) * C + c);
  stf(out + i, acc / (float)HW);
}
// The same with one block per image when the channel count divides 256: the block's 256 / C groups of
// threads each sum a share of the pixels (independent loads, consecutive lanes on consecutive channels),
// then the shares are added through LDS - instead of one thread walking all pixels of a channel with
// dependent 2-byte loads (20 us for 64 pixels).
template <typename T>
__global__ __launch_bounds__(256) void pm_pool_fwd_block_kernel(const T* __restrict__ y, T* __restrict__ out, int HW, int C) {
  __shared__ float part[256];
  const int b = blockIdx.x, c = threadIdx.x % C, grp = threadIdx.x / C, ngrp = 256 / C;
  float acc = 0.f;
  for (int p = grp; p < HW; p += ngrp) acc += ldf(y + ((int64_t)b * HW + p) * C + c);
  part[threadIdx.x] = acc;
  __syncthreads();
  if (grp == 0) {
    for (int q = 1; q < ngrp; ++q) acc += part[q * C + c];
    stf(out + (int64_t)b * C + c, acc / (float)HW);
  }
}
template <typename T>
inline void pm_pool_fwd_launch(hipStream_t st, const T* y, T* out, int B, int HW, int C) {
  if (C <= 256 && 256 % C == 0)
    hipLaunchKernelGGL((pm_pool_fwd_block_kernel<T>), dim3(B), dim3(256), 0, st, y, out, HW, C);
  else
    hipLaunchKernelGGL((pm_pool_fwd_kernel<T>), dim3((B * C + 255) / 256), dim3(256), 0, st, y, out, B, HW, C);
}
template <typename T>
__global__ __launch_bounds__(256) void pm_pool_bwd_kernel(const T* __restrict__ dpool, T* __restrict__ dy, int B, int HW, int C) {
  const int64_t total = (int64_t)B * HW * C;
  const float inv = 1.f / (float)HW;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const int c = (int)(i % C), b = (int)(i / ((int64_t)HW * C));
    stf(dy + i, ldf(dpool + (int64_t)b * C + c) * inv);
  }
}

// out[e] (+)= sum over nparts partial vectors of n elements each (part[p][e]); one launch takes a list of jobs.
struct PmReduceJob {
  const float* part;
  int nparts, n;
  float* out;
  int accumulate;
  int cin, cpad;     // rows of cin elements lie cpad apart in the partials (0: they lie as in the output)
};
constexpr int PM_CONV_JOBS = 24;       // jobs of one launch (they travel as kernel arguments)
constexpr int PM_REDUCE_JOBS = 64;     // (3.4 KB of arguments)
struct PmReduceList {
  PmReduceJob job[PM_REDUCE_JOBS];
  int end[PM_REDUCE_JOBS];             // first block behind each job
  int count;
};
// A job of few elements and many partials (the channel sums of the affine backward: 32 .. 128 elements, up to 1024 partials) has
// one block, whose chain of loads the whole launch waits for: there a thread takes four neighbouring elements of every 256 / (n / 4)-th
// partial.
inline __host__ __device__ bool pm_conv_reduce_narrow(const PmReduceJob& jb) { return jb.n <= 128 && jb.n % 4 == 0 && !jb.cpad && jb.nparts >= 64; }
// Block = 16 slices of the partial range x 64 elements, four per thread: many short chains of independent
// loads instead of a few long ones (the arrays are small; what matters is the latency of the longest chain).
__global__ __launch_bounds__(256) void pm_conv_reduce_kernel(PmReduceList list) {
  int k = 0;
  while (k + 1 < list.count && (int)blockIdx.x >= list.end[k]) ++k;
  const PmReduceJob jb = list.job[k];
  __shared__ __attribute__((aligned(16))) float s[16][64];
  if (pm_conv_reduce_narrow(jb)) {                           // uniform over the block
    const int n4 = jb.n >> 2, slices = 256 / n4, slice = (int)threadIdx.x / n4, c = ((int)threadIdx.x - slice * n4) * 4;
    float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
    auto add = [&](const float4& v) __attribute__((always_inline)) { sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w; };
    if (slice < slices) {
      const float* p = jb.part + c;
      int r = slice;
      for (; r + 7 * slices < jb.nparts; r += 8 * slices) {
        float4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const float4*>(p + (int64_t)(r + u * slices) * jb.n);
#pragma unroll
        for (int u = 0; u < 8; ++u) add(v[u]);
      }
      for (; r < jb.nparts; r += slices) add(*reinterpret_cast<const float4*>(p + (int64_t)r * jb.n));
    }
    float4* all = reinterpret_cast<float4*>(&s[0][0]);
    all[threadIdx.x] = sum;
    __syncthreads();
    if ((int)threadIdx.x < n4) {
#pragma unroll 8
      for (int q = 1; q < slices; ++q) add(all[q * n4 + threadIdx.x]);
      float* o = jb.out + c;
      const float out[4] = {sum.x, sum.y, sum.z, sum.w};
#pragma unroll
      for (int q = 0; q < 4; ++q) o[q] = jb.accumulate ? o[q] + out[q] : out[q];
    }
    return;
  }
  const int el = threadIdx.x & 15, sl = threadIdx.x >> 4;
  const int e0 = ((int)blockIdx.x - (k ? list.end[k - 1] : 0)) * 64;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  int off[4];
  const int ns = jb.cpad ? jb.n / jb.cin * jb.cpad : jb.n;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    off[q] = min(e0 + 16 * q + el, jb.n - 1);
    if (jb.cpad) off[q] = off[q] / jb.cin * jb.cpad + off[q] % jb.cin;
  }
  int p = sl;
  auto rows = [&](auto count) __attribute__((always_inline)) {
    constexpr int R = decltype(count)::value;
    float v[R][4];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int q = 0; q < 4; ++q) v[r][q] = jb.part[(int64_t)(p + 16 * r) * ns + off[q]];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[q] += v[r][q];
  };
#pragma unroll 1
  for (; p + 112 < jb.nparts; p += 128) rows(std::integral_constant<int, 8>());
#pragma unroll 1
  for (; p + 16 < jb.nparts; p += 32) rows(std::integral_constant<int, 2>());
  if (p < jb.nparts) rows(std::integral_constant<int, 1>());
#pragma unroll
  for (int q = 0; q < 4; ++q) s[sl][16 * q + el] = acc[q];
  __syncthreads();
  if (threadIdx.x < 64 && e0 + (int)threadIdx.x < jb.n) {
    float v = 0.f;
#pragma unroll
    for (int q = 0; q < 16; ++q) v += s[q][threadIdx.x];
    float* o = jb.out + e0 + threadIdx.x;
    *o = jb.accumulate ? *o + v : v;
  }
}
// the jobs of `v`, in launches of up to PM_REDUCE_JOBS
inline void pm_conv_reduce_launch(hipStream_t st, const PmReduceJob* v, int count) {
  for (int at = 0; at < count; at += PM_REDUCE_JOBS) {
    PmReduceList l{};
    l.count = std::min(PM_REDUCE_JOBS, count - at);
    int blocks = 0;
    for (int k = 0; k < l.count; ++k) {
      l.job[k] = v[at + k];
      l.end[k] = blocks += pm_conv_reduce_narrow(v[at + k]) ? 1 : (v[at + k].n + 63) / 64;
    }
    hipLaunchKernelGGL(pm_conv_reduce_kernel, dim3((unsigned)blocks), dim3(256), 0, st, l);
  }
}

// ---------------------------------------------------------------------------------------------
// implicit-GEMM kernels (bf16, Cin and Cout multiples of 16, at most 64)
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ pm_bf16x8 pm_cv_ld8(const bf16_t* p) { return *reinterpret_cast<const pm_bf16x8*>(p); }

// Pixel index -> (image, row, column) of a W x H map (32-bit divisions but for maps beyond 2^31 pixels).
__device__ __forceinline__ void pm_cv_split(int64_t p, int W, int H, int& b, int& y, int& x) {
  if (p < ((int64_t)1 << 31)) {
    const unsigned u = (unsigned)p, r = u / (unsigned)W;
    x = (int)(u - r * (unsigned)W);
    b = (int)(r / (unsigned)H);
    y = (int)(r - (unsigned)b * (unsigned)H);
  } else {
    const int64_t r = p / W;
    x = (int)(p - r * W);
    b = (int)(r / H);
    y = (int)(r - (int64_t)b * H);
  }
}

// Product of one wave: 32 pixels (lane % 32) x NCT tiles of 32 channels, rows wrow[.] of the weights, contraction over 9
// taps of 16 KC channels.  BWD: the source is dz and the weights are [ci][tap][co].  All loads are unconditional (a tap
// outside the map reads pixel 0 and is masked when it arrives) and are requested ahead of the products, AHEAD tap rows
// of them (registers).  Under a predicate each load came out with a wait of its own, 9 KC round trips to memory one
// behind the other, and the kernels spent nearly all their time there.
template <int KC, bool BWD, int NCT, int AHEAD>
__device__ __forceinline__ void pm_cv_core(const PmConvGeom& g, const bf16_t* __restrict__ src, const bf16_t* const (&wrow)[NCT],
                                           bool pv, int b, int y, int x, int kg, pm_f32x16 (&acc)[NCT]) {
  constexpr int C = 16 * KC;
  const int SH = BWD ? g.Ho : g.H, SW = BWD ? g.Wo : g.W;
  union Frag { pm_bf16x8 v; uint4 q; };
  Frag fx[AHEAD][3][KC], fw[AHEAD][3][KC][NCT];
  unsigned m[AHEAD][3];
  auto load = [&](int r, int at) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      int iy, ix;
      bool ok = pv;
      if (BWD) {
        const int sh = g.stride - 1;                      // stride 1 or 2
        iy = y + 1 - r;
        ix = x + 1 - c;
        ok = ok && iy >= 0 && ix >= 0 && !((iy | ix) & sh);
        iy >>= sh;
        ix >>= sh;
        ok = ok && iy < SH && ix < SW;
      } else {
        iy = y * g.stride + r - 1;
        ix = x * g.stride + c - 1;
        ok = ok && iy >= 0 && iy < SH && ix >= 0 && ix < SW;
      }
      m[at][c] = ok ? 0xffffffffu : 0u;
      const bf16_t* sp = src + (ok ? (((int64_t)b * SH + iy) * SW + ix) * C : (int64_t)0) + 8 * kg;
#pragma unroll
      for (int k = 0; k < KC; ++k) {
        fx[at][c][k].q = *reinterpret_cast<const uint4*>(sp + 16 * k);
#pragma unroll
        for (int t = 0; t < NCT; ++t) fw[at][c][k][t].q = *reinterpret_cast<const uint4*>(wrow[t] + (r * 3 + c) * C + 8 * kg + 16 * k);
      }
    }
  };
  auto mma = [&](int at) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int k = 0; k < KC; ++k) {
        Frag f = fx[at][c][k];
        const unsigned w = m[at][c];
        f.q = make_uint4(f.q.x & w, f.q.y & w, f.q.z & w, f.q.w & w);
#pragma unroll
        for (int t = 0; t < NCT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[at][c][k][t].v, f.v, acc[t], 0, 0, 0);
      }
  };
  if constexpr (AHEAD == 1) {
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      load(r, 0);
      mma(0);
    }
  } else {
    // (scheduling barriers: left to itself the compiler moves each load down to its use)
    load(0, 0);
    load(1, 1);
    if (AHEAD == 3) load(2, 2 % AHEAD);
    __builtin_amdgcn_sched_barrier(0);
    mma(0);
    if (AHEAD == 2) {
      load(2, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    mma(1);
    mma(2 % AHEAD);
  }
}
__device__ __forceinline__ float4 pm_cv_unpack(uint2 a) {
  return make_float4(__uint_as_float(a.x << 16), __uint_as_float(a.x & 0xffff0000u), __uint_as_float(a.y << 16),
                     __uint_as_float(a.y & 0xffff0000u));
}
__device__ __forceinline__ uint2 pm_cv_mask(uint2 a, bool on) {
  const unsigned m = on ? 0xffffffffu : 0u;
  return make_uint2(a.x & m, a.y & m);
}

// forward.  One wave = 32 output pixels x NCT x 32 output channels (blockIdx.y: which); blockDim.x / 64 waves per
// block, no LDS.  What the epilogue reads is requested before the contraction where loads go ahead.
// 128 x 32 x 32 x 16 channels 10.4 -> 7.0 us, 128 x 8 x 8 x 64 channels 19.0 -> 7.0 us; large maps 512 x 64 x 64 x 16 83 -> 76,
// 256 x 16 x 16 x 64 34 -> 32 us, against loads under predicates with one load in flight per wave.
template <int KC, int NCT, int AHEAD>    // Cin = 16 KC
__global__ __launch_bounds__(256) void pm_conv_fwd_mfma_kernel(PmConvGeom g, const bf16_t* __restrict__ x,
                                                               PmWLoc<bf16_t> wloc, PmShortcut<bf16_t> sc,
                                                               bf16_t* __restrict__ z, bf16_t* __restrict__ y) {
  const bf16_t* Wt = wloc.get();
  const bf16_t* scale = Wt + (int64_t)g.Cout * 9 * g.Cin;
  const bf16_t* shift = scale + g.Cout;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, pl = lane & 31, kg = lane >> 5, c0 = blockIdx.y * 32 * NCT;
  const int64_t npix = (int64_t)g.B * g.Ho * g.Wo;
  const int64_t p = ((int64_t)blockIdx.x * (blockDim.x >> 6) + wave) * 32 + pl;
  const bool pv = p < npix;
  int b, oy, ox;
  pm_cv_split(pv ? p : 0, g.Wo, g.Ho, b, oy, ox);
  // a lane's channels: c0 + 32 t + 8 a + 4 kg + 0 .. 3; groups past Cout are left out (uniform: Cout is a multiple of 16)
  uint2 rs[NCT][4], rt[NCT][4], rc[NCT][4];
  const bf16_t* sp = sc.src ? sc.src + (((int64_t)b * sc.Hs + oy * sc.stride) * sc.Ws + ox * sc.stride) * sc.Cs : nullptr;
  auto affine = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < NCT; ++t)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        if (c0 + 32 * t + 8 * a >= g.Cout) continue;
        const int co = c0 + 32 * t + 8 * a + 4 * kg;
        rs[t][a] = *reinterpret_cast<const uint2*>(scale + co);
        rt[t][a] = *reinterpret_cast<const uint2*>(shift + co);
        rc[t][a] = make_uint2(0u, 0u);
        // whole groups of 8 lie inside or outside the shortcut's channels (Cs is a multiple of 8)
        if (sp && c0 + 32 * t + 8 * a < sc.Cs) rc[t][a] = *reinterpret_cast<const uint2*>(sp + co);
      }
  };
  if (AHEAD > 1) affine();
  pm_f32x16 acc[NCT];
  const bf16_t* wrow[NCT];
#pragma unroll
  for (int t = 0; t < NCT; ++t) {
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
    wrow[t] = Wt + (int64_t)min(c0 + 32 * t + pl, g.Cout - 1) * 9 * g.Cin;      // channels past Cout repeat the last one: not stored
  }
  pm_cv_core<KC, false, NCT, AHEAD>(g, x, wrow, pv, b, oy, ox, kg, acc);
  if (AHEAD == 1) affine();
  if (!pv) return;
#pragma unroll
  for (int t = 0; t < NCT; ++t)
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      if (c0 + 32 * t + 8 * a >= g.Cout) continue;
      const int co = c0 + 32 * t + 8 * a + 4 * kg;
      const float4 s4 = pm_cv_unpack(rs[t][a]), t4 = pm_cv_unpack(rt[t][a]), c4 = pm_cv_unpack(rc[t][a]);
      const float ss[4] = {s4.x, s4.y, s4.z, s4.w}, tt[4] = {t4.x, t4.y, t4.z, t4.w}, cc[4] = {c4.x, c4.y, c4.z, c4.w};
      float yy[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float av = ss[j] * acc[t][4 * a + j] + tt[j] + cc[j];
        yy[j] = av > 0.f ? av : 0.f;
      }
      pm_st4(z + p * g.Cout + co, make_float4(acc[t][4 * a], acc[t][4 * a + 1], acc[t][4 * a + 2], acc[t][4 * a + 3]));
      pm_st4(y + p * g.Cout + co, make_float4(yy[0], yy[1], yy[2], yy[3]));
    }
}

// The kernel tensors of the backward weights, transposed for the data gradient: [co][tap][ci] -> [ci][tap][co],
// all units in one launch.
struct PmCvTransposeJob {
  PmWLoc<bf16_t> w;
  bf16_t* wt;
  int Cin, Cout;
};
struct PmCvTransposeList {
  PmCvTransposeJob job[PM_CONV_JOBS];
};
__global__ __launch_bounds__(256) void pm_conv_transpose_kernel(PmCvTransposeList list) {
  const PmCvTransposeJob jb = list.job[blockIdx.y];
  const bf16_t* w = jb.w.get();
  const int n = jb.Cin * 9 * jb.Cout;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
    const int co = i % jb.Cout, r = i / jb.Cout, tap = r % 9, ci = r / 9;
    jb.wt[i] = w[(co * 9 + tap) * jb.Cin + ci];
  }
}

template <int O>
__device__ __forceinline__ void pm_cv_exchange(float (&v)[32], int pl) {
  const bool up = (pl & O) != 0;
#pragma unroll
  for (int i = 0; i < O; ++i) {
    const float send = up ? v[i] : v[i + O], keep = up ? v[i + O] : v[i];
    v[i] = keep + __shfl_xor(send, O, 64);
  }
}

// data gradient of a unit with the affine backward of the unit below in its epilogue: the product is dy of that
// unit; with its y and z at the same places
//   da = dy [y > 0] (stored where a shortcut will read it),  dz = da * scale_bkwd,
//   sums over the block's pixels of da z and of da -> part[block][0 = scale | 1 = shift][Cin].
// Same scheme as the forward kernel, on the transposed kernel tensor.  One launch and no dy in memory in place of
// the data gradient (11.6 us on 128 x 32 x 32 x 16 channels, 18.7 on 128 x 8 x 8 x 64: it parked the whole kernel
// tensor in LDS first) and a pass over dy, y and z (7 us): 10.0 and 9.4 us.
template <int KC>    // Cout = 16 KC
__global__ __launch_bounds__(256, KC == 1 ? 4 : 1) void pm_conv_dgrad_affine_kernel(PmConvGeom g, const bf16_t* __restrict__ dz,
                                                                   const bf16_t* __restrict__ wt, PmShortcutBwd<bf16_t> sb,
                                                                   const bf16_t* __restrict__ y, const bf16_t* __restrict__ z,
                                                                   PmWLoc<bf16_t> scale_bkwd, bf16_t* __restrict__ da_out,
                                                                   bf16_t* __restrict__ dz_out, float* __restrict__ part) {
  const bf16_t* scale = scale_bkwd.get();
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, pl = lane & 31, kg = lane >> 5, c0 = blockIdx.y * 32;
  const int64_t npix = (int64_t)g.B * g.H * g.W;
  const int64_t p = ((int64_t)blockIdx.x * (blockDim.x >> 6) + wave) * 32 + pl;
  const bool pv = p < npix;
  int b, iy, ix;
  pm_cv_split(pv ? p : 0, g.W, g.H, b, iy, ix);
  const int64_t row = (pv ? p : 0) * g.Cin;
  uint2 rs[4], ry[4], rz[4], rc[4];
  const bool sv = sb.da && (sb.stride == 1 || !((iy | ix) & 1));
  const bf16_t* sp = sb.da ? sb.da + (sv ? (((int64_t)b * sb.Ho + iy / sb.stride) * sb.Wo + ix / sb.stride) * sb.Co : (int64_t)0) : scale;
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const int ci = c0 + 8 * a + 4 * kg, cc = ci < g.Cin ? ci : 0;
    rs[a] = *reinterpret_cast<const uint2*>(scale + cc);
    ry[a] = *reinterpret_cast<const uint2*>(y + row + cc);
    rz[a] = *reinterpret_cast<const uint2*>(z + row + cc);
    rc[a] = *reinterpret_cast<const uint2*>(sp + cc);      // (no shortcut: the scale's address, masked)
  }
  pm_f32x16 acc1[1];
  pm_f32x16& acc = acc1[0];
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
  const bf16_t* wrow[1] = {wt + (int64_t)min(c0 + pl, g.Cin - 1) * 9 * g.Cout};
  pm_cv_core<KC, true, 1, KC <= 2 ? 3 : 2>(g, dz, wrow, pv, b, iy, ix, kg, acc1);
  float v[32];                                           // [which sum][a][j]
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const int ci = c0 + 8 * a + 4 * kg;
    const bool st = pv && ci < g.Cin;
    const float4 s4 = pm_cv_unpack(rs[a]), y4 = pm_cv_unpack(ry[a]), z4 = pm_cv_unpack(rz[a]), c4 = pm_cv_unpack(pm_cv_mask(rc[a], sv));
    const float ss[4] = {s4.x, s4.y, s4.z, s4.w}, yy[4] = {y4.x, y4.y, y4.z, y4.w}, zz[4] = {z4.x, z4.y, z4.z, z4.w};
    // dy is rounded to bf16 as an activation gradient in memory is
    const float4 d4 = pm_cv_unpack(make_uint2(pm_pack_bf16(acc[4 * a] + c4.x, acc[4 * a + 1] + c4.y),
                                              pm_pack_bf16(acc[4 * a + 2] + c4.z, acc[4 * a + 3] + c4.w)));
    const float dd[4] = {d4.x, d4.y, d4.z, d4.w};
    float d[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      d[j] = yy[j] > 0.f ? dd[j] : 0.f;
      v[4 * a + j] = st ? d[j] * zz[j] : 0.f;
      v[16 + 4 * a + j] = st ? d[j] : 0.f;
    }
    if (st) {
      if (da_out) pm_st4(da_out + row + ci, make_float4(d[0], d[1], d[2], d[3]));
      pm_st4(dz_out + row + ci, make_float4(d[0] * ss[0], d[1] * ss[1], d[2] * ss[2], d[3] * ss[3]));
    }
  }
  // 32 sums over 32 lanes: each exchange adds the half that the partner keeps, 31 exchanges in all, and lane pl
  // ends with sum number pl
  pm_cv_exchange<16>(v, pl);
  pm_cv_exchange<8>(v, pl);
  pm_cv_exchange<4>(v, pl);
  pm_cv_exchange<2>(v, pl);
  pm_cv_exchange<1>(v, pl);
  __shared__ float red[4][64];
  red[wave][(pl >> 4) * 32 + 8 * ((pl >> 2) & 3) + 4 * kg + (pl & 3)] = v[0];
  __syncthreads();
  if (threadIdx.x < 64) {
    const int which = threadIdx.x >> 5, ci = c0 + (threadIdx.x & 31);
    float t = red[0][threadIdx.x];
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w) t += red[w][threadIdx.x];
    if (ci < g.Cin) part[((int64_t)blockIdx.x * 2 + which) * g.Cin + ci] = t;
  }
}

// data gradient on the kernel tensor as it lies, for the entry point that has no room for a transposed one
// and no unit below.  One wave = 32 input pixels x all input channels.  The whole kernel tensor of the
// backward weights sits in LDS as it lies in memory ([co][tap * Cin + ci], padded rows); its
// transposed fragments (row = ci, contraction = co) come from LDS transpose loads.
template <int NCO, int NCT>   // channel tiles of 32: Cout <= 32 NCO, Cin <= 32 NCT
__global__ __launch_bounds__(256) void pm_conv_dgrad_mfma_kernel(PmConvGeom g, const bf16_t* __restrict__ dz,
                                                                 PmWLoc<bf16_t> wloc, PmShortcutBwd<bf16_t> sb,
                                                                 bf16_t* __restrict__ dx) {
  __shared__ __attribute__((aligned(16))) bf16_t sW[(32 * NCO + 16) * (9 * 32 * NCT + 8)];
  const int K9 = 9 * g.Cin, WS = K9 + 8;                 // LDS row stride: 16-byte aligned rows
  {
    const bf16_t* Wt = wloc.get();
    const int chunks = g.Cout * (K9 / 8);
    for (int c = threadIdx.x; c < chunks; c += blockDim.x) {
      const int r = c / (K9 / 8), col = (c % (K9 / 8)) * 8;
      *reinterpret_cast<uint4*>(sW + r * WS + col) = *reinterpret_cast<const uint4*>(Wt + (int64_t)r * K9 + col);
    }
    // fragment reads of a channel tile wider than Cin run past a row's end into the next row (those
    // MFMA rows are discarded); the 16 tail rows keep such reads of the last row inside the array
    for (int c = threadIdx.x; c < 16 * WS / 8; c += blockDim.x) *reinterpret_cast<uint4*>(sW + g.Cout * WS + c * 8) = make_uint4(0, 0, 0, 0);
  }
  __syncthreads();
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, pl = lane & 31, kg = lane >> 5;
  const int64_t npix = (int64_t)g.B * g.H * g.W;
  const int64_t p = ((int64_t)blockIdx.x * (blockDim.x >> 6) + wave) * 32 + pl;
  const bool pv = p < npix;
  const int ix = (int)(p % g.W), iy = (int)((p / g.W) % g.H), b = (int)(p / ((int64_t)g.W * g.H));
  pm_f32x16 acc[NCT];
#pragma unroll
  for (int t = 0; t < NCT; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
  const int ql = lane >> 4, q = lane & 15;               // transpose-load lane mapping (see pm_at_frag_tr)
  for (int tap = 0; tap < 9; ++tap) {
    const int ny = iy + 1 - tap / 3, nx = ix + 1 - tap % 3;
    bool ok = pv && ny >= 0 && nx >= 0 && (ny % g.stride) == 0 && (nx % g.stride) == 0;
    const int oy = ny / g.stride, ox = nx / g.stride;
    ok = ok && oy < g.Ho && ox < g.Wo;
    const bf16_t* dr = dz + (((int64_t)b * g.Ho + oy) * g.Wo + ox) * g.Cout + 8 * kg;
    for (int kc = 0; kc < g.Cout; kc += 16) {
      const pm_bf16x8 fb = ok ? pm_cv_ld8(dr + kc) : pm_at_zero8();
#pragma unroll
      for (int t = 0; t < NCT; ++t) {
        // A = W^T: MFMA row = ci = t * 32 + lane % 32 (LDS column tap * Cin + ci), contraction = co rows kc ..
        const bf16_t* pp = sW + (kc + 8 * (ql >> 1) + (q >> 2)) * WS + tap * g.Cin + t * 32 + 16 * (ql & 1) + 4 * (q & 3);
        typedef pm_v4s __attribute__((address_space(3))) * lds_v4s;
        union { pm_bf16x8 v; pm_v4s h[2]; } u;
        u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(pp));
        u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(pp + 4 * WS));
        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(u.v, fb, acc[t], 0, 0, 0);
      }
    }
  }
  if (!pv) return;
#pragma unroll
  for (int t = 0; t < NCT; ++t)
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const int ci = t * 32 + 8 * a + 4 * kg;
      if (ci >= g.Cin) continue;
      float v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = acc[t][4 * a + j] + sb.at(b, iy, ix, ci + j);
      pm_st4(dx + p * g.Cin + ci, make_float4(v[0], v[1], v[2], v[3]));
    }
}

// weight gradient.  Nothing of the backward chain waits for it, so the units of a step share one launch (one per
// pair of channel tiles).  A block takes the three taps of one row (blockIdx.y) and a run of 32-pixel chunks
// for each of its waves.  Per chunk a wave parks the dz rows and the three shifted sets of input rows in its own
// LDS region and reads all of them transposed (contraction = pixels); the loads of the next chunk are in flight
// meanwhile.  The taps' sums stay in registers until the end, when the four waves meet in LDS and the block
// writes its partial of the three taps; pm_conv_reduce_kernel adds the blocks' partials.
// Taking one tap of a chunk at a time left every load - park - multiply round trip exposed (36 of them in a row),
// in a launch per unit that filled the chip once: 16 - 20 us per unit, 313 us for the 18 units of ResNet-20 on
// 128 images; now 93 us with the image layer.
struct PmCvWgradJob {
  PmConvGeom g;
  const bf16_t* dz;
  const bf16_t* x;
  float* part;       // [block][Cout][9][Cin]
  int nch;           // chunks of 32 pixels per wave
};
struct PmCvWgradList {
  PmCvWgradJob job[PM_CONV_JOBS];
  int end[PM_CONV_JOBS];               // first blockIdx.x behind each job
  int count;
};
// PA, PB: 16-byte pieces per lane of 32 pixels of Cout and Cin channels: 1 (both 16), 2 (up to 32), 4 (up to 64).
// With 16 channels a transposed read of 32 columns runs into the next row; those rows of the product are not
// stored.  That takes 24 KB of LDS a block instead of 40, and half the loads.
template <int PA, int PB>
struct PmCvWgradLds {
  static constexpr int NTO = (PA + 1) / 2, NTI = (PB + 1) / 2;   // channel tiles of 32
  static constexpr int SA = PA * 16 + 8, SB = PB * 16 + 8;       // LDS row strides (elements)
  static constexpr int RW = NTI * 32;                            // row width of the block's reduction tile
  static constexpr int WAVE = 32 * SA + 3 * 32 * SB + (PB == 1 ? 16 : 0);   // elements of a wave's region, with what a read of the last row runs into
  static constexpr size_t BYTES = sizeof(bf16_t) * 4 * WAVE > sizeof(float) * 4 * NTO * 32 * RW ? sizeof(bf16_t) * 4 * WAVE
                                                                                                : sizeof(float) * 4 * NTO * 32 * RW;
};
template <int PA, int PB>
__device__ __forceinline__ void pm_conv_wgrad_block(const PmCvWgradJob& jb, int bid, unsigned char* lds) {
  using S = PmCvWgradLds<PA, PB>;
  constexpr int NTO = S::NTO, NTI = S::NTI, SA = S::SA, SB = S::SB, RW = S::RW, WAVE = S::WAVE;
  const PmConvGeom g = jb.g;
  const bf16_t* __restrict__ dz = jb.dz;
  const bf16_t* __restrict__ x = jb.x;
  const int dy = (int)blockIdx.y - 1, nch = jb.nch;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  bf16_t* wa = reinterpret_cast<bf16_t*>(lds) + wave * WAVE;
  bf16_t* wb = wa + 32 * SA;
  for (int c = lane; c < WAVE / 8; c += 64) *reinterpret_cast<uint4*>(wa + c * 8) = make_uint4(0, 0, 0, 0);
  const int npix = g.B * g.Ho * g.Wo;                      // fits 32 bits (checked by the dispatcher)
  const int pa = g.Cout / 8, pb = g.Cin / 8;               // 16-byte pieces per row
  const int first = (bid * 4 + wave) * nch * 32;           // (below npix + 4 * 32 * nch: fits as well)
  // where this lane's pieces lie: pixel of the chunk and column
  int ap[PA], ac[PA], bp[PB], bc[PB];
#pragma unroll
  for (int j = 0; j < PA; ++j) {
    const int c = lane + 64 * j;
    ap[j] = c / pa;
    ac[j] = (c - ap[j] * pa) * 8;
  }
#pragma unroll
  for (int j = 0; j < PB; ++j) {
    const int c = lane + 64 * j;
    bp[j] = c / pb;
    bc[j] = (c - bp[j] * pb) * 8;
  }
  uint4 ra[PA], rb[3][PB];
  unsigned ma[PA], mb[3][PB];
  // loads are unconditional (element 0 where there is nothing to read) and masked when they are parked
  auto load = [&](int p0) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < PA; ++j) {
      const bool ok = ap[j] < 32 && p0 + ap[j] < npix;
      ma[j] = ok ? 0xffffffffu : 0u;
      ra[j] = *reinterpret_cast<const uint4*>(dz + (ok ? (p0 + ap[j]) * g.Cout + ac[j] : 0));
    }
#pragma unroll
    for (int j = 0; j < PB; ++j) {
      const int p = p0 + bp[j];
      const bool in = bp[j] < 32 && p < npix;
      const unsigned up = in ? (unsigned)p : 0u, r = up / (unsigned)g.Wo, bb = r / (unsigned)g.Ho;
      const int iy = (int)(r - bb * (unsigned)g.Ho) * g.stride + dy, ix = (int)(up - r * (unsigned)g.Wo) * g.stride;
      const bool iny = in && iy >= 0 && iy < g.H;
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        const bool ok = iny && ix + t - 1 >= 0 && ix + t - 1 < g.W;
        mb[t][j] = ok ? 0xffffffffu : 0u;
        rb[t][j] = *reinterpret_cast<const uint4*>(x + (ok ? (((int)bb * g.H + iy) * g.W + ix + t - 1) * g.Cin + bc[j] : 0));
      }
    }
  };
  auto park = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < PA; ++j)
      if (ap[j] < 32) {
        const unsigned m = ma[j];
        *reinterpret_cast<uint4*>(wa + ap[j] * SA + ac[j]) = make_uint4(ra[j].x & m, ra[j].y & m, ra[j].z & m, ra[j].w & m);
      }
#pragma unroll
    for (int j = 0; j < PB; ++j)
      if (bp[j] < 32) {
#pragma unroll
        for (int t = 0; t < 3; ++t) {
          const unsigned m = mb[t][j];
          *reinterpret_cast<uint4*>(wb + (t * 32 + bp[j]) * SB + bc[j]) =
              make_uint4(rb[t][j].x & m, rb[t][j].y & m, rb[t][j].z & m, rb[t][j].w & m);
        }
      }
  };
  typedef pm_v4s __attribute__((address_space(3))) * lds_v4s;
  const int ql = lane >> 4, q = lane & 15;                 // transpose-load lane mapping (see pm_at_frag_tr)
  auto frag = [&](const bf16_t* base, int stride, int ks, int tile) __attribute__((always_inline)) {
    const bf16_t* pp = base + (ks * 16 + 8 * (ql >> 1) + (q >> 2)) * stride + tile * 32 + 16 * (ql & 1) + 4 * (q & 3);
    union { pm_bf16x8 v; pm_v4s h[2]; } u;
    u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(pp));
    u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(pp + 4 * stride));
    return u.v;
  };
  pm_f32x16 acc[3][NTO][NTI];
#pragma unroll
  for (int t = 0; t < 3; ++t)
#pragma unroll
    for (int a = 0; a < NTO; ++a)
#pragma unroll
      for (int bb = 0; bb < NTI; ++bb)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[t][a][bb][e] = 0.f;
  load(first);
#pragma unroll 1
  for (int ch = 0; ch < nch; ++ch) {
    park();
    if (ch + 1 < nch) load(first + (ch + 1) * 32);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      pm_bf16x8 fa[NTO];
#pragma unroll
      for (int a = 0; a < NTO; ++a) fa[a] = frag(wa, SA, ks, a);
#pragma unroll
      for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int bb = 0; bb < NTI; ++bb) {
          const pm_bf16x8 fb = frag(wb + t * 32 * SB, SB, ks, bb);
#pragma unroll
          for (int a = 0; a < NTO; ++a)
            acc[t][a][bb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[a], fb, acc[t][a][bb], 0, 0, 0);
        }
    }
    __builtin_amdgcn_wave_barrier();
  }
  // per tap the four waves' sums meet in LDS: value v of lane l is row co = 32 a + 8 (v / 4) + 4 (l / 32) + v % 4,
  // column ci = 32 bb + l % 32
  float* red = reinterpret_cast<float*>(lds);
  constexpr int IMG = NTO * 32 * RW;
  float* my_part = jb.part + (int64_t)bid * g.Cout * 9 * g.Cin;
  const int kg = lane >> 5, cl = lane & 31;
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    __syncthreads();
#pragma unroll
    for (int a = 0; a < NTO; ++a)
#pragma unroll
      for (int bb = 0; bb < NTI; ++bb)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          red[wave * IMG + (a * 32 + 8 * (v >> 2) + 4 * kg + (v & 3)) * RW + bb * 32 + cl] = acc[t][a][bb][v];
    __syncthreads();
    const int c4 = g.Cin / 4;
    for (int e = threadIdx.x; e < g.Cout * c4; e += 256) {
      const int co = e / c4, ci = (e - co * c4) * 4, o = co * RW + ci;
      float4 sum = *reinterpret_cast<const float4*>(red + o);
#pragma unroll
      for (int w = 1; w < 4; ++w) {
        const float4 v = *reinterpret_cast<const float4*>(red + w * IMG + o);
        sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
      }
      *reinterpret_cast<float4*>(my_part + (co * 9 + blockIdx.y * 3 + t) * g.Cin + ci) = sum;
    }
  }
}

template <int PA, int PB>
__global__ __launch_bounds__(256) void pm_conv_wgrad_mfma_kernel(PmCvWgradList list) {
  __shared__ __attribute__((aligned(16))) unsigned char lds[PmCvWgradLds<PA, PB>::BYTES];
  int k = 0;
  while (k + 1 < list.count && (int)blockIdx.x >= list.end[k]) ++k;
  pm_conv_wgrad_block<PA, PB>(list.job[k], (int)blockIdx.x - (k ? list.end[k - 1] : 0), lds);
}
// Units of more than 16 channels, all pairs of channel tiles in one launch (at the LDS and registers of the widest: two
// blocks per compute unit).  The launches per pair are short and each leaves much of the chip idle: 32 us for the 8 units of
// ResNet-14 on 37 images in three launches, 25 in one.  The 16-channel units keep a launch of their own, whose blocks are smaller
// and share a compute unit in sixes.
__global__ __launch_bounds__(256) void pm_conv_wgrad_wide_kernel(PmCvWgradList list) {
  __shared__ __attribute__((aligned(16))) unsigned char lds[PmCvWgradLds<4, 4>::BYTES];
  int k = 0;
  while (k + 1 < list.count && (int)blockIdx.x >= list.end[k]) ++k;
  const PmCvWgradJob& jb = list.job[k];
  const int bid = (int)blockIdx.x - (k ? list.end[k - 1] : 0);
  if (jb.g.Cout > 32) {
    if (jb.g.Cin > 32) pm_conv_wgrad_block<4, 4>(jb, bid, lds);
    else pm_conv_wgrad_block<4, 2>(jb, bid, lds);
  } else {
    if (jb.g.Cin > 32) pm_conv_wgrad_block<2, 4>(jb, bid, lds);
    else pm_conv_wgrad_block<2, 2>(jb, bid, lds);
  }
}

// ---------------------------------------------------------------------------------------------
// host-side dispatch
// ---------------------------------------------------------------------------------------------
inline bool pm_conv_mfma_fits(int Cin, int Cout) { return (Cin % 16) == 0 && (Cout % 16) == 0 && Cin <= 64 && Cout <= 64; }

// Waves (of 32 pixels) per block of the forward and data-gradient kernels: one where the pixel groups times the
// channel tiles are fewer than eight waves per compute unit, so that they spread over all of them.
inline int pm_conv_waves(int64_t npix, int channels) {
  return (npix + 31) / 32 * ((channels + 31) / 32) >= 2048 ? 4 : 1;
}

template <typename T>
inline void pm_conv_fwd_launch(hipStream_t st, const PmConvGeom& g, const T* x, PmWLoc<T> w, PmShortcut<T> sc, T* z, T* y) {
  const int64_t npix = (int64_t)g.B * g.Ho * g.Wo;
  if constexpr (sizeof(T) == 2) {
    if (pm_conv_mfma_fits(g.Cin, g.Cout)) {
      const int wpb = pm_conv_waves(npix, g.Cout);
      auto go = [&](auto kc, auto nct, auto ahead) {
        const dim3 grid((unsigned)((npix + 32 * wpb - 1) / (32 * wpb)), (g.Cout + 32 * nct - 1) / (32 * nct)), blk(64 * wpb);
        hipLaunchKernelGGL((pm_conv_fwd_mfma_kernel<kc, nct, ahead>), grid, blk, 0, st, g, x, w, sc, z, y);
      };
      using std::integral_constant;
      auto with = [&](auto kc) {
        constexpr int KC = decltype(kc)::value;
        // many wide pixels: both channel tiles in one wave, so that the gathered operand is read once, and few registers
        // (128 x 16 x 16 x 64 channels 21.1 -> 17.5 us, 2048 x 8 x 8 73 -> 58; 128 x 8 x 8 7.0 against 8.2 the other way)
        if (KC > 2 && g.Cout > 32 && wpb == 4) go(kc, integral_constant<int, 2>(), integral_constant<int, 1>());
        else go(kc, integral_constant<int, 1>(), integral_constant<int, (KC <= 2 ? 3 : 2)>());
      };
      if (g.Cin == 16) with(integral_constant<int, 1>());
      else if (g.Cin == 32) with(integral_constant<int, 2>());
      else if (g.Cin == 48) with(integral_constant<int, 3>());
      else with(integral_constant<int, 4>());
      return;
    }
  }
  if (g.Cin == 3 && g.Cout == 16) {                     // the image layer
    hipLaunchKernelGGL((pm_conv_fwd_thin_kernel<T>), dim3((unsigned)std::min<int64_t>(65535, (npix + 255) / 256)), dim3(256),
                       0, st, g, x, w, sc, z, y);
    return;
  }
  const int64_t total = npix * g.Cout;
  hipLaunchKernelGGL((pm_conv_fwd_plain_kernel<T>), dim3((unsigned)std::min<int64_t>(65535, (total + 255) / 256)), dim3(256), 0,
                     st, g, x, w, sc, z, y);
}

template <typename T>
inline void pm_conv_dgrad_launch(hipStream_t st, const PmConvGeom& g, const T* dz, PmWLoc<T> w, PmShortcutBwd<T> sb, T* dx) {
  const int64_t npix = (int64_t)g.B * g.H * g.W;
  if constexpr (sizeof(T) == 2) {
    if (pm_conv_mfma_fits(g.Cin, g.Cout)) {
      // (fewer waves per block on small maps were measured slower here: every block first loads the kernel tensor)
      const dim3 grid((unsigned)((npix + 127) / 128)), blk(256);
#define PM_CD(A, B) hipLaunchKernelGGL((pm_conv_dgrad_mfma_kernel<A, B>), grid, blk, 0, st, g, dz, w, sb, dx)
      if (g.Cout <= 32 && g.Cin <= 32) PM_CD(1, 1);
      else if (g.Cout <= 32) PM_CD(1, 2);
      else if (g.Cin <= 32) PM_CD(2, 1);
      else PM_CD(2, 2);
#undef PM_CD
      return;
    }
  }
  const int64_t total = npix * g.Cin;
  hipLaunchKernelGGL((pm_conv_dgrad_plain_kernel<T>), dim3((unsigned)std::min<int64_t>(65535, (total + 255) / 256)), dim3(256),
                     0, st, g, dz, w, sb, dx);
}

// blocks of the fused data gradient over the pixels: the partial sums it writes
inline int pm_conv_dgrad_affine_blocks(const PmConvGeom& g) {
  const int64_t npix = (int64_t)g.B * g.H * g.W;
  const int wpb = pm_conv_waves(npix, g.Cin);
  return (int)((npix + 32 * wpb - 1) / (32 * wpb));
}
inline void pm_conv_dgrad_affine_launch(hipStream_t st, const PmConvGeom& g, const bf16_t* dz, const bf16_t* wt,
                                        PmShortcutBwd<bf16_t> sb, const bf16_t* y, const bf16_t* z, PmWLoc<bf16_t> scale_bkwd,
                                        bf16_t* da_out, bf16_t* dz_out, float* part) {
  const int wpb = pm_conv_waves((int64_t)g.B * g.H * g.W, g.Cin);
  const dim3 grid((unsigned)pm_conv_dgrad_affine_blocks(g), (g.Cin + 31) / 32), blk(64 * wpb);
#define PM_CA(K) hipLaunchKernelGGL((pm_conv_dgrad_affine_kernel<K>), grid, blk, 0, st, g, dz, wt, sb, y, z, scale_bkwd, da_out, dz_out, part)
  if (g.Cout == 16) PM_CA(1);
  else if (g.Cout == 32) PM_CA(2);
  else if (g.Cout == 48) PM_CA(3);
  else PM_CA(4);
#undef PM_CA
}
inline void pm_conv_transpose_launch(hipStream_t st, const PmCvTransposeJob* v, int count) {
  for (int at = 0; at < count; at += PM_CONV_JOBS) {
    PmCvTransposeList l{};
    const int n = std::min(PM_CONV_JOBS, count - at);
    for (int k = 0; k < n; ++k) l.job[k] = v[at + k];
    hipLaunchKernelGGL(pm_conv_transpose_kernel, dim3(16, (unsigned)n), dim3(256), 0, st, l);
  }
}

// Chunks of 32 pixels per wave and blocks of the MFMA weight-gradient kernel.  Each block (times three tap rows) writes a
// partial that is read once more.  In a step, whose units share launches: at most 64, 32 of the wide tensors, whose
// partials are 147 KB each, and eight chunks a wave where the map has them (a block's start and the sums of its waves cost as
// much as two or three chunks: ResNet-20 on 128 images 476 us a step with as few as one, 469 from 4, 461 from 8; ResNet-14 on 37
// of 28 x 28: 215, 210 and, where that leaves too few blocks, 216).  A unit by itself (ALONE) has to fill the chip: up to 256 and 64 where that leaves a wave four
// chunks.  Us with 64 (32) blocks, now, and with twice as many: 512 x 64 x 64 x 16 channels 184, 77, 81; 512 x 32 x 32 x 32 68,
// 34, 42; 256 x 32 x 32 x 64 137, 76, 107; 128 x 16 x 16 x 32, below four chunks, 12, 12, 15.  Never more partials than
// pm_conv_wgrad_scratch_elems has room for: one per 16 chunks from 2048 chunks on, one per 4 below.
inline void pm_conv_wgrad_plan(const PmConvGeom& g, bool alone, int* blocks, int* nch) {
  const int64_t chunks = ((int64_t)g.B * g.Ho * g.Wo + 31) / 32;
  const bool wide = g.Cin * g.Cout > 1024;
  int64_t most = wide ? 32 : 64;
  if (alone) most = std::max<int64_t>(most, std::min<int64_t>(wide ? 64 : 256, chunks / 16));
  int64_t c = (chunks + 4 * most - 1) / (4 * most);
  if (!alone) c = std::max(c, std::min<int64_t>(8, (chunks + 27) / 28));
  *nch = (int)c;
  *blocks = (int)((chunks + c * 4 - 1) / (c * 4));
}
inline bool pm_conv_thin_fits(const PmConvGeom& g) {
  return g.Cin == 3 && g.Cout == 16 && (int64_t)g.B * g.H * g.W * 16 < ((int64_t)1 << 31);
}
template <typename T>
inline bool pm_conv_wgrad_mfma_fits(const PmConvGeom& g) {       // 32-bit indexing inside
  return sizeof(T) == 2 && pm_conv_mfma_fits(g.Cin, g.Cout) &&
         (int64_t)g.B * g.H * g.W * std::max(g.Cin, g.Cout) < (int64_t)1 << 31;
}
// partial vectors of Cout * 9 * Cin floats that the weight gradient writes (0: the plain path is used)
template <typename T>
inline int pm_conv_wgrad_parts(const PmConvGeom& g, bool alone = false) {
  if (pm_conv_thin_fits(g)) return PM_CONV_THIN_GROUPS;
  if (!pm_conv_wgrad_mfma_fits<T>(g)) return 0;
  int blocks, nch;
  pm_conv_wgrad_plan(g, alone, &blocks, &nch);
  return blocks;
}
// fp32 scratch elements that the entry points ask for: a partial per 128 pixels, per 512 on large maps.  The
// kernel writes fewer; callers hold workspaces of this size, and the entry without one refuses by it.
template <typename T>
inline size_t pm_conv_wgrad_scratch_elems(const PmConvGeom& g) {
  if (pm_conv_thin_fits(g)) return (size_t)PM_CONV_THIN_GROUPS * g.Cout * 9 * g.Cin;
  if (!pm_conv_wgrad_mfma_fits<T>(g)) return 0;
  const int64_t chunks = ((int64_t)g.B * g.Ho * g.Wo + 31) / 32, c = chunks >= 2048 ? 16 : 4;
  return (size_t)((chunks + c - 1) / c) * g.Cout * 9 * g.Cin;
}

// The MFMA weight gradients of a list of units: one launch for those of 16 channels and one for all others, per PM_CONV_JOBS units
inline void pm_conv_wgrad_group_launch(hipStream_t st, const PmCvWgradJob* v, int count, bool alone = false) {
  auto class_of = [](const PmConvGeom& g) { return g.Cin == 16 && g.Cout == 16 ? 4 : (g.Cout > 32 ? 2 : 0) + (g.Cin > 32 ? 1 : 0); };
  for (int thin = 0; thin < 2; ++thin) {
    PmCvWgradList l{};
    int blocks = 0, classes = 0;                          // (bit per class)
    auto flush = [&]() {
      if (!l.count) return;
      const dim3 grid((unsigned)blocks, 3), blk(256);
      switch (classes) {
        case 1 << 0: hipLaunchKernelGGL((pm_conv_wgrad_mfma_kernel<2, 2>), grid, blk, 0, st, l); break;
        case 1 << 1: hipLaunchKernelGGL((pm_conv_wgrad_mfma_kernel<2, 4>), grid, blk, 0, st, l); break;
        case 1 << 2: hipLaunchKernelGGL((pm_conv_wgrad_mfma_kernel<4, 2>), grid, blk, 0, st, l); break;
        case 1 << 3: hipLaunchKernelGGL((pm_conv_wgrad_mfma_kernel<4, 4>), grid, blk, 0, st, l); break;
        case 1 << 4: hipLaunchKernelGGL((pm_conv_wgrad_mfma_kernel<1, 1>), grid, blk, 0, st, l); break;
        default: hipLaunchKernelGGL(pm_conv_wgrad_wide_kernel, grid, blk, 0, st, l);
      }
      l.count = blocks = classes = 0;
    };
    for (int cls = thin ? 4 : 3; cls >= (thin ? 4 : 0); --cls)      // the widest, and so the longest, blocks first
      for (int i = 0; i < count; ++i) {
        if (class_of(v[i].g) != cls) continue;
        int nb, nch;
        pm_conv_wgrad_plan(v[i].g, alone, &nb, &nch);
        l.job[l.count] = v[i];
        l.job[l.count].nch = nch;
        l.end[l.count++] = blocks += nb;
        classes |= 1 << class_of(v[i].g);
        if (l.count == PM_CONV_JOBS) flush();
      }
    flush();
  }
}
template <typename T>
inline void pm_conv_wgrad_thin_launch(hipStream_t st, const PmConvGeom& g, const T* dz, const T* x, float* part) {
  hipLaunchKernelGGL((pm_conv_wgrad_thin_kernel<T, 16, 3>), dim3(PM_CONV_THIN_GROUPS, 9), dim3(256), 0, st, g, dz, x, part);
}
template <typename T>
inline void pm_conv_wgrad_plain_launch(hipStream_t st, const PmConvGeom& g, const T* dz, const T* x, float* dW, int accumulate) {
  hipLaunchKernelGGL((pm_conv_wgrad_plain_kernel<T>), dim3((unsigned)(g.Cout * 9 * g.Cin)), dim3(256), 0, st, g, dz, x, dW,
                     accumulate);
}
// one unit by itself: dW (fp32 [Cout][9][Cin]) = correlation of dz with x.  `scratch` holds
// pm_conv_wgrad_scratch_elems floats (unused by the plain path).
template <typename T>
inline void pm_conv_wgrad_launch(hipStream_t st, const PmConvGeom& g, const T* dz, const T* x, float* dW, float* scratch) {
  const int parts = pm_conv_wgrad_parts<T>(g, true);
  if (!parts) {
    pm_conv_wgrad_plain_launch<T>(st, g, dz, x, dW, 0);
    return;
  }
  if (pm_conv_thin_fits(g)) {
    pm_conv_wgrad_thin_launch<T>(st, g, dz, x, scratch);
  } else if constexpr (sizeof(T) == 2) {
    const PmCvWgradJob jb{g, dz, x, scratch, 0};
    pm_conv_wgrad_group_launch(st, &jb, 1, true);
  }
  const PmReduceJob r{scratch, parts, g.Cout * 9 * g.Cin, dW, 0};
  pm_conv_reduce_launch(st, &r, 1);
}

constexpr int PM_CONV_AFFINE_MAX_BLOCKS = 1024;
// part: NULL (fp32 atomics into dscale / dshift), or room for PM_CONV_AFFINE_MAX_BLOCKS * 2 * C floats; then
// *job receives the reduction the caller must hand to the next reduce launch (out = dscale, n = 2 C:
// dshift follows dscale in memory).
template <typename T>
inline bool pm_conv_affine_bwd_launch(hipStream_t st, const T* dy, const T* y, const T* z, PmWLoc<T> scale_bkwd, T* da, T* dz,
                                      float* dscale, float* dshift, int64_t total, int C, float* part = nullptr,
                                      PmReduceJob* job = nullptr) {
  if (C < 8 || C > 256 || (C & (C - 1))) return false;        // a power of two in 8 .. 256
  if (part && dshift != dscale + C) return false;
  const unsigned blocks = (unsigned)std::max<int64_t>(1, std::min<int64_t>(part ? PM_CONV_AFFINE_MAX_BLOCKS : 512, (total + 2047) / 2048));
  hipLaunchKernelGGL((pm_conv_affine_bwd_kernel<T>), dim3(blocks), dim3(256), 0, st, dy, y, z, scale_bkwd, da, dz, dscale,
                     dshift, part, total, C);
  if (part && job) *job = PmReduceJob{part, (int)blocks, 2 * C, dscale, 1};
  return true;
}
