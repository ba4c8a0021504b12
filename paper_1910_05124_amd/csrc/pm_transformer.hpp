// Weight-free and vector-weight kernels of the fine-grained Transformer stages: embedding,
// LayerNorm, causal attention core.  The matrix stages reuse the Linear GEMMs.
//
// Row t = b * S + s of every [tokens, width] matrix is token s of sequence b.  The residual stream
// and its gradient are fp32; GEMM operands are in the compute dtype T (bf16 or fp32).
//
// Two-weight backward (Sec. 2.1): a backward kernel reads a weight only where a gradient flows
// through it: LayerNorm's dx uses the backward gain (corrected buffer or ring slot, like the
// Linear units' dz . W); the gain / bias gradients use forward quantities only.
#pragma once
#include "pm_common.hpp"
#include "pm_update.hpp"
#include "pm_attn_api.hpp"

constexpr float PM_LN_EPS = 1e-5f;

// ---------------------------------------------------------------------------------------------
// GEMM epilogues of the residual blocks (used with the same GEMM kernels as the Linear epilogues)
// ---------------------------------------------------------------------------------------------
// out[i, j] = res[i, j] + acc + b[j], fp32: the residual stream after an attention / feed-forward block
template <typename T>
struct PmEpiFwdRes {
  static constexpr bool kColSumA = false, kAKC = true, kBKC = true;
  __device__ __forceinline__ bool wants_colsum() const { return false; }
  __device__ __forceinline__ void colsum(int, float) const {}
  PmWLoc<T> bias;
  const float* res; float* out; int ld;
  const T* b_;
  __device__ __forceinline__ void begin() { b_ = bias.get(); }
  __device__ __forceinline__ void operator()(int i, int j, float acc) const {
    const int64_t o = (int64_t)i * ld + j;
    out[o] = res[o] + acc + ldf(b_ + j);
  }
  struct Pre { PmRaw8<T> b; PmRaw8<float> r; };
  __device__ __forceinline__ Pre pre8(int i, int j) const {
    Pre p;
    p.b.load(b_ + j);
    p.r.load(res + (int64_t)i * ld + j);
    return p;
  }
  __device__ __forceinline__ void op8(int i, int j, const float* acc, const Pre& p) const {
    const int64_t o = (int64_t)i * ld + j;
    float v[8], bb[8], rr[8];
    p.b.widen(bb);
    p.r.widen(rr);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = rr[e] + acc[e] + bb[e];
    pm_st8(out + o, v);
  }
};
// out[i, j] (+)= acc, fp32: data gradients that enter a LayerNorm backward (summed over the
// consumers of the LayerNorm output)
struct PmEpiF32 {
  static constexpr bool kColSumA = false, kAKC = true, kBKC = false;
  __device__ __forceinline__ bool wants_colsum() const { return false; }
  __device__ __forceinline__ void colsum(int, float) const {}
  float* out; int ld; int accumulate;
  __device__ __forceinline__ void begin() {}
  __device__ __forceinline__ void operator()(int i, int j, float acc) const {
    const int64_t o = (int64_t)i * ld + j;
    out[o] = accumulate ? out[o] + acc : acc;
  }
  struct Pre { float o[8]; };
  __device__ __forceinline__ Pre pre8(int i, int j) const {
    Pre p;
    if (accumulate) pm_ld8(out + (int64_t)i * ld + j, p.o);
    return p;
  }
  __device__ __forceinline__ void op8(int i, int j, const float* acc, const Pre& p) const {
    const int64_t o = (int64_t)i * ld + j;
    float v[8];
    if (accumulate) {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = p.o[e] + acc[e];
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = acc[e];
    }
    pm_st8(out + o, v);
  }
};

// zero a list of regions of a flat fp32 array: region r = [reg[2r], reg[2r] + reg[2r+1]); grid (x, regions)
static __global__ __launch_bounds__(256) void pm_zero_regions_kernel(float* base, const int64_t* __restrict__ reg) {
  const int64_t off = reg[2 * blockIdx.y], n = reg[2 * blockIdx.y + 1];
  float4* p = reinterpret_cast<float4*>(base + off);          // regions are chunk-aligned and chunk-sized
  const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < (n >> 2); i += (int64_t)gridDim.x * blockDim.x) p[i] = z;
}

// First kernel of a Transformer microbatch: refreshes the step table at the start of a minibatch
// (L > 0) and clears the loss accumulator.  A launch of its own because the next kernel (the
// embedding lookup) already reads its ring slot from the table.
static __global__ void pm_begin_tokens_kernel(PmStepHdr* hdr, const PmLayerStatic* ls, PmLayerStep* ld, int L, PmSchedDev sc,
                                       int par) {
  if (L > 0) pm_prologue_block(hdr, ls, ld, L, sc, par);
  pm_loss_clear(hdr);
}

// ---------------------------------------------------------------------------------------------
// embedding: x[t, :] = E[token[t], :] + pos[t mod S, :]
// ---------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void pm_embed_fwd_kernel(const int32_t* __restrict__ tokens, PmWLoc<T> E,
                                                           const float* __restrict__ pos, float* __restrict__ x,
                                                           int tokens_n, int S, int d, int vocab) {
  const T* e = E.get();
  const int64_t total = (int64_t)tokens_n * d;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const int t = (int)(i / d), j = (int)(i % d);
    int tok = tokens[t];
    tok = tok < 0 ? 0 : (tok >= vocab ? vocab - 1 : tok);          // out-of-range ids are clamped
    x[i] = ldf(e + (int64_t)tok * d + j) + pos[(int64_t)(t % S) * d + j];
  }
}

// Weights of the products that follow a LayerNorm, read while it runs, by the first `blocks` blocks of its launch: a weight matrix was last
// touched many steps ago (a ring slot) or by the update of the step before, so a product that finds it in memory waits 1.5 to 3 us longer
// than one that finds it in the last-level cache.  Step time without, with 64 blocks a launch, and with a line for each thread: 6 x 512
// layers, 4096 rows 1683, 1657, 1626 us; 3 x 768, four times 2048 rows 4411, 4311, 4227; 4 x 320, 2400 rows 787, 773, 761.
struct PmReadAhead {
  struct Span { const unsigned char* base; const int32_t* slot; int64_t stride_bytes; int64_t bytes; };
  Span m[4];
  int count, blocks;
  // a line for each thread, in blocks of nt, but no more than two blocks of 256 threads per compute unit
  void spread(int nt) {
    int64_t lines = 0;
    for (int k = 0; k < count; ++k) lines += (m[k].bytes + 127) / 128;
    const int64_t most = 512 * 256 / 2 / nt, want = (lines + nt - 1) / nt;
    blocks = (int)(want < most ? want : most);
  }
};
__device__ __forceinline__ void pm_read_ahead(const PmReadAhead& ra) {
  uint32_t acc = 0;
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;         // line of 128 bytes, counted through all matrices
  for (int k = 0; k < ra.count; ++k) {
    const PmReadAhead::Span& s = ra.m[k];
    const unsigned char* base = s.base + (s.slot ? (int64_t)(*s.slot) * s.stride_bytes : 0);
    for (; i * 128 < s.bytes; i += (int64_t)ra.blocks * blockDim.x) acc |= *reinterpret_cast<const uint32_t*>(base + i * 128);
    i -= (s.bytes + 127) / 128;
  }
  asm volatile("" ::"v"(acc));                            // the reads have no other use: keep them
}

// ---------------------------------------------------------------------------------------------
// LayerNorm forward: one wavefront per row, the row held in registers (lane l owns columns
// 256 c + 4 l .. + 3, d <= 256 NC, d a multiple of 4).  Stores mean and 1/sqrt(var + eps) for the
// backward.  gb: gain at offset 0, bias at offset boff of the unit's ring slot.
// ---------------------------------------------------------------------------------------------
template <typename T, int NC>
__global__ __launch_bounds__(256) void pm_ln_fwd_kernel(const float* __restrict__ x, PmWLoc<T> gb, int boff,
                                                        T* __restrict__ out, float* __restrict__ mean,
                                                        float* __restrict__ rstd, int rows, int d, PmReadAhead ra) {
  if ((int)blockIdx.x < ra.blocks) {
    pm_read_ahead(ra);
    return;
  }
  const int row = ((int)blockIdx.x - ra.blocks) * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= rows) return;
  const int64_t ro = (int64_t)row * d;
  float4 xv[NC];
  float s = 0.f;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int j = 256 * c + 4 * lane;
    xv[c] = j < d ? pm_ld4(x + ro + j) : make_float4(0.f, 0.f, 0.f, 0.f);
    s += xv[c].x + xv[c].y + xv[c].z + xv[c].w;
  }
  const float mu = pm_wave_sum(s) / (float)d;
  float v = 0.f;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int j = 256 * c + 4 * lane;
    if (j < d) {
      xv[c] = make_float4(xv[c].x - mu, xv[c].y - mu, xv[c].z - mu, xv[c].w - mu);
      v += xv[c].x * xv[c].x + xv[c].y * xv[c].y + xv[c].z * xv[c].z + xv[c].w * xv[c].w;
    }
  }
  const float rs = rsqrtf(pm_wave_sum(v) / (float)d + PM_LN_EPS);
  const T* g = gb.get();
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int j = 256 * c + 4 * lane;
    if (j < d) {
      const float4 gg = pm_ld4(g + j), bb = pm_ld4(g + boff + j);
      pm_st4(out + ro + j, make_float4(xv[c].x * rs * gg.x + bb.x, xv[c].y * rs * gg.y + bb.y, xv[c].z * rs * gg.z + bb.z,
                                       xv[c].w * rs * gg.w + bb.w));
    }
  }
  if (lane == 0) {
    mean[row] = mu;
    rstd[row] = rs;
  }
}

// ---------------------------------------------------------------------------------------------
// LayerNorm backward.  dy fp32 [rows, d] is the gradient w.r.t. the LayerNorm output.
//   dx_out = dx_res + rstd * (dxh - mean(dxh) - xhat * mean(dxh * xhat)),  dxh = dy * gain_bkwd
//   dgain += sum_rows dy * xhat,  dbias += sum_rows dy
// dx_res is the gradient already on the residual stream (same shape); dx_out may alias it.
// dx_out_t (optional) receives a copy in the compute dtype for the GEMMs that consume it.
// Block = 8 waves x RPW rows; lane l owns columns 256 c + 4 l .. + 3 (16-byte accesses), d <= 256 NC,
// d a multiple of 4.
//
// The column sums of a block go to dgain / dbias by fp32 atomics, or (PART) to its own row of a table that
// pm_ln_params_block adds up for all LayerNorms of the step at once.  With atomics fewer, larger blocks win (each
// block's 2 d atomics meet those of all others on the same addresses), which left 64 blocks of 2048 rows on 256 compute units;
// with the table, blocks of 8 rows: 2048 x 768 10.9 -> 7.6 us, 4096 x 512 12.1 -> 9.3 (16 rows), 2400 x 320 8.6 -> 5.7, 512 x 256
// 4.9 -> 2.7.  8192 x 1024 is bound by its 151 MB (35 us either way, 5 TB/s inside a step) and the table would be 2 MB more to
// write and read, so beyond 4096 rows the atomics stay.
// ---------------------------------------------------------------------------------------------
constexpr int PM_LN_PART_ROWS = 4096;
inline int pm_ln_part_rpw(int64_t rows) { return rows <= 2048 ? 1 : 2; }              // at most 256 blocks
inline int64_t pm_ln_part_blocks(int64_t rows) {                                     // rows of the table; 0: atomics
  const int64_t per = 8 * pm_ln_part_rpw(rows);
  return rows <= PM_LN_PART_ROWS ? (rows + per - 1) / per : 0;
}
template <typename T, int NC, int RPW, bool PART>
__global__ __launch_bounds__(512) void pm_ln_bwd_kernel(const float* __restrict__ dy, const float* __restrict__ x,
                                                        const float* __restrict__ mean, const float* __restrict__ rstd,
                                                        PmWLoc<T> gain_bkwd, const float* dx_res, float* dx_out,
                                                        T* dx_out_t, float* __restrict__ dgain, float* __restrict__ dbias,
                                                        int rows, int d, int parts, int64_t part_stride, PmReadAhead ra) {
  if ((int)blockIdx.x < ra.blocks) {
    pm_read_ahead(ra);
    return;
  }
  const int block = (int)blockIdx.x - ra.blocks;
  __shared__ float4 red[8][2][64 * NC];                       // per wave: gain and bias partial sums
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const T* g = gain_bkwd.get();
  const float4 zero4 = make_float4(0.f, 0.f, 0.f, 0.f);
  float4 gj[NC], ag[NC], ab[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int j = 256 * c + 4 * lane;
    gj[c] = j < d ? pm_ld4(g + j) : zero4;
    ag[c] = zero4;
    ab[c] = zero4;
  }
  // all loads of the wave's rows go out first (rows past the end re-read the last row and are
  // masked out below), so the wave pays the memory latency once instead of once per row
  float4 dyr[RPW][NC], xr[RPW][NC], rrr[RPW][NC];
  float mur[RPW], rsr[RPW];
#pragma unroll
  for (int r = 0; r < RPW; ++r) {
    const int row = block * (8 * RPW) + wave * RPW + r;
    const int rowc = row < rows ? row : rows - 1;
    const int64_t ro = (int64_t)rowc * d;
    mur[r] = mean[rowc];
    rsr[r] = rstd[rowc];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int j = 256 * c + 4 * lane;
      dyr[r][c] = j < d ? pm_ld4(dy + ro + j) : zero4;
      xr[r][c] = j < d ? pm_ld4(x + ro + j) : zero4;
      // (requested here, not row by row below: a load issued behind the stores of the row before would wait for them)
      rrr[r][c] = (dx_res && j < d) ? pm_ld4(dx_res + ro + j) : zero4;
    }
  }
#pragma unroll
  for (int r = 0; r < RPW; ++r)
    for (int p = 1; p < parts; ++p) {                         // the gradient arrives as several addends
      const int row = block * (8 * RPW) + wave * RPW + r;
      const float* dyp = dy + p * part_stride + (int64_t)(row < rows ? row : rows - 1) * d;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int j = 256 * c + 4 * lane;
        const float4 e = j < d ? pm_ld4(dyp + j) : zero4;
        dyr[r][c].x += e.x; dyr[r][c].y += e.y; dyr[r][c].z += e.z; dyr[r][c].w += e.w;
      }
    }
#pragma unroll
  for (int r = 0; r < RPW; ++r) {
    const int row = block * (8 * RPW) + wave * RPW + r;
    if (row >= rows) break;                                   // wave-uniform
    const float mu = mur[r], rs = rsr[r];
    const int64_t ro = (int64_t)row * d;
    float4 xh[NC], dxh[NC], rr[NC];
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int j = 256 * c + 4 * lane;
      float4 dyv = dyr[r][c], xv = zero4;
      rr[c] = rrr[r][c];
      if (j < d) {
        xv = xr[r][c];
        xv = make_float4((xv.x - mu) * rs, (xv.y - mu) * rs, (xv.z - mu) * rs, (xv.w - mu) * rs);
      }
      xh[c] = xv;
      dxh[c] = make_float4(dyv.x * gj[c].x, dyv.y * gj[c].y, dyv.z * gj[c].z, dyv.w * gj[c].w);
      ag[c].x += dyv.x * xv.x; ag[c].y += dyv.y * xv.y; ag[c].z += dyv.z * xv.z; ag[c].w += dyv.w * xv.w;
      ab[c].x += dyv.x; ab[c].y += dyv.y; ab[c].z += dyv.z; ab[c].w += dyv.w;
      s1 += dxh[c].x + dxh[c].y + dxh[c].z + dxh[c].w;
      s2 += dxh[c].x * xv.x + dxh[c].y * xv.y + dxh[c].z * xv.z + dxh[c].w * xv.w;
    }
    s1 = pm_wave_sum(s1) / (float)d;
    s2 = pm_wave_sum(s2) / (float)d;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int j = 256 * c + 4 * lane;
      if (j < d) {
        float4 v;
        v.x = rr[c].x + rs * (dxh[c].x - s1 - xh[c].x * s2);
        v.y = rr[c].y + rs * (dxh[c].y - s1 - xh[c].y * s2);
        v.z = rr[c].z + rs * (dxh[c].z - s1 - xh[c].z * s2);
        v.w = rr[c].w + rs * (dxh[c].w - s1 - xh[c].w * s2);
        pm_st4(dx_out + ro + j, v);
        if (dx_out_t) pm_st4(dx_out_t + ro + j, v);
      }
    }
  }
  // block sum of the per-wave partials (plain LDS stores and loads: LDS float atomics were measured
  // several times slower)
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    red[wave][0][64 * c + lane] = ag[c];
    red[wave][1][64 * c + lane] = ab[c];
  }
  __syncthreads();
  for (int j = threadIdx.x; j < d; j += 512) {
    float sg = 0.f, sb = 0.f;
    const int c = j >> 8, l4 = (j & 255) >> 2, e = j & 3;      // column j = 256 c + 4 lane + e
#pragma unroll
    for (int w = 0; w < 8; ++w) {
      const float* pg = reinterpret_cast<const float*>(&red[w][0][64 * c + l4]);
      const float* pb = reinterpret_cast<const float*>(&red[w][1][64 * c + l4]);
      sg += pg[e];
      sb += pb[e];
    }
    if (PART) {                                               // dgain: the table [blocks][2][d]
      dgain[(int64_t)block * 2 * d + j] = sg;
      dgain[(int64_t)block * 2 * d + d + j] = sb;
    } else {
      atomicAdd(dgain + j, sg);
      atomicAdd(dbias + j, sb);
    }
  }
}

// Adds up the tables of all LayerNorms of a step: block b takes 64 of the 2 d columns of LayerNorm b / blocks per LayerNorm,
// four groups of threads a quarter of the rows each.  where[2 n], where[2 n + 1]: offsets of LayerNorm n's gain and bias gradients in g.
__device__ __forceinline__ void pm_ln_params_block(int b, const float* __restrict__ part, const int64_t* __restrict__ where, float* __restrict__ g,
                                                   int rows, int d) {
  __shared__ float sum[4][64];
  const int cb = (2 * d + 63) / 64, n = b / cb, col = (b - n * cb) * 64 + (threadIdx.x & 63), rg = threadIdx.x >> 6;
  float acc = 0.f;
  if (col < 2 * d) {
    const float* p = part + (int64_t)n * rows * 2 * d + col;
#pragma unroll 8
    for (int r = rg; r < rows; r += 4) acc += p[(int64_t)r * 2 * d];
  }
  sum[rg][threadIdx.x & 63] = acc;
  __syncthreads();
  if (rg == 0 && col < 2 * d) {
    float* o = g + (col < d ? where[2 * n] + col : where[2 * n + 1] + col - d);
    *o += (sum[0][threadIdx.x] + sum[1][threadIdx.x]) + (sum[2][threadIdx.x] + sum[3][threadIdx.x]);
  }
}

// Last launch of a backward pass: dE[token[t], :] += dx[t, :] (fp32 atomics; the caller zeroes dE first unless accumulating) in
// the first n_embed blocks, and in the others the sums of the LayerNorms' tables.
//
// A block takes PM_EMB_TOK tokens and 256 columns and adds up the rows of equal tokens before it touches dE: with the frequencies of
// text one token in eight is the same, and its row's atomics, one per token, kept the launch waiting (26 us before, 14 now on 4096 x 512;
// 2048 x 768 19 and 11).
constexpr int PM_EMB_TOK = 32;
inline int pm_embed_bwd_blocks(int tokens, int d) { return (tokens + PM_EMB_TOK - 1) / PM_EMB_TOK * ((d + 255) / 256); }
static __global__ __launch_bounds__(256) void pm_embed_bwd_kernel(const int32_t* __restrict__ tokens, const float* __restrict__ dx,
                                                           float* __restrict__ dE, int tokens_n, int d, int vocab, int n_embed,
                                                           const float* __restrict__ part, const int64_t* __restrict__ where,
                                                           float* __restrict__ g, int part_rows) {
  if ((int)blockIdx.x >= n_embed) {
    pm_ln_params_block(blockIdx.x - n_embed, part, where, g, part_rows, d);
    return;
  }
  __shared__ int32_t ids[PM_EMB_TOK], sorted[PM_EMB_TOK], from[PM_EMB_TOK];
  const int cols = (d + 255) / 256, t0 = blockIdx.x / cols * PM_EMB_TOK, j = (blockIdx.x % cols) * 256 + threadIdx.x;
  const int n = tokens_n - t0 < PM_EMB_TOK ? tokens_n - t0 : PM_EMB_TOK, t = threadIdx.x;
  if (t < n) {
    const int tok = tokens[t0 + t];
    ids[t] = tok < 0 ? 0 : (tok >= vocab ? vocab - 1 : tok);
  }
  __syncthreads();
  if (t < n) {                                     // equal tokens side by side, each in its old order
    int r = 0;
    for (int u = 0; u < n; ++u) r += ids[u] < ids[t] || (ids[u] == ids[t] && u < t);
    sorted[r] = ids[t];
    from[r] = t;
  }
  __syncthreads();
  if (j >= d) return;
  float v[PM_EMB_TOK];
#pragma unroll
  for (int r = 0; r < PM_EMB_TOK; ++r) v[r] = r < n ? dx[(int64_t)(t0 + from[r]) * d + j] : 0.f;
  float acc = 0.f;
#pragma unroll
  for (int r = 0; r < PM_EMB_TOK; ++r) {
    if (r >= n) break;
    acc += v[r];
    if (r + 1 == n || sorted[r + 1] != sorted[r]) {                    // uniform over the block
      atomicAdd(dE + (int64_t)sorted[r] * d + j, acc);
      acc = 0.f;
    }
  }
}

// copy fp32 -> compute dtype (the residual gradient entering a GEMM)
template <typename T>
__global__ __launch_bounds__(256) void pm_cast_kernel(const float* __restrict__ in, T* __restrict__ out, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    stf(out + i, in[i]);
}

// ---------------------------------------------------------------------------------------------
// host-side dispatch
// ---------------------------------------------------------------------------------------------
template <typename T>
inline bool pm_ln_fwd_launch(hipStream_t st, const float* x, PmWLoc<T> gb, int boff, T* out, float* mean, float* rstd,
                             int rows, int d, const PmReadAhead& ra = PmReadAhead{}) {
  if ((d & 3) || (boff & 3)) return false;
  const dim3 grid(ra.blocks + (rows + 3) / 4), blk(256);
#define PM_LNF(NC) hipLaunchKernelGGL((pm_ln_fwd_kernel<T, NC>), grid, blk, 0, st, x, gb, boff, out, mean, rstd, rows, d, ra)
  if (d <= 256) PM_LNF(1);
  else if (d <= 512) PM_LNF(2);
  else if (d <= 768) PM_LNF(3);
  else if (d <= 1024) PM_LNF(4);
  else return false;
#undef PM_LNF
  return true;
}

// table: null (the sums meet in dgain / dbias by atomics), or pm_ln_part_blocks(rows) rows of 2 d values to be added up later
template <typename T>
inline bool pm_ln_bwd_launch(hipStream_t st, const float* dy, const float* x, const float* mean, const float* rstd,
                             PmWLoc<T> gain_bkwd, const float* dx_res, float* dx_out, T* dx_out_t, float* dgain,
                             float* dbias, int rows, int d, int parts = 1, int64_t part_stride = 0, float* table = nullptr,
                             const PmReadAhead& ra = PmReadAhead{}) {
  if (d & 3) return false;
  const int rpw = table ? pm_ln_part_rpw(rows) : 4;
  const dim3 grid(ra.blocks + (rows + 8 * rpw - 1) / (8 * rpw)), blk(512);
#define PM_LNB(NC, RPW, PART) hipLaunchKernelGGL((pm_ln_bwd_kernel<T, NC, RPW, PART>), grid, blk, 0, st, dy, x, mean, rstd, gain_bkwd, dx_res, dx_out, dx_out_t, PART ? table : dgain, dbias, rows, d, parts, part_stride, ra)
#define PM_LNB_ROWS(NC) do { if (!table) PM_LNB(NC, 4, false); else if (rpw == 1) PM_LNB(NC, 1, true); else PM_LNB(NC, 2, true); } while (0)
  if (d <= 256) PM_LNB_ROWS(1);
  else if (d <= 512) PM_LNB_ROWS(2);
  else if (d <= 768) PM_LNB_ROWS(3);
  else if (d <= 1024) PM_LNB_ROWS(4);
  else return false;
#undef PM_LNB_ROWS
#undef PM_LNB
  return true;
}
