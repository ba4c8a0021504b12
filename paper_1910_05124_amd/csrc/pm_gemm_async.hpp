// bf16 products of the Linear units, from a few rows to many thousands:
//
//   C[i, j] = sum_k A(i, k) * B(j, k),   each operand read along the contraction (KC) or across it (RC):
//   forward KC, KC; data gradient KC, RC; weight gradient RC, RC
//
// What bounds such a product is how fast a compute unit gets its operand tiles: measured, 83 bytes per ns reach the LDS of
// one unit whatever the tile (64 x 64, 128 x 64, 32 x 32 outputs per block, alone on the chip or with all units busy), and
// through registers (load, wait, LDS store; pm_gemm_mfma.hpp) less, because the stores and the fragment reads share the
// LDS: 4096 x 512 x 2048 took 20 us at a fifth of the matrix rate.  So the load unit writes the LDS itself
// (buffer_load_dwordx4 ... lds), ST slabs ahead; a slab's fragments go to registers while the slab before multiplies; one
// barrier per slab.  From 256 x 256 outputs per block on the matrix rate bounds: 53 us per 8192 x 4096 x 1024 (1.28
// PFLOP/s, of 1.47 that the matrix units reach on such data) and 13 us per round of blocks for start and output.
//
// Measured (us per launch alone, the weights from memory each time; before, through registers on 64 x 64 and 128 x 128 blocks
// or 32 x 32 with the whole contraction at once -> now; forward unless said): 500 x 768 x 768 8.0 -> 6.0, 500 x 768 x 3072
// 17.4 -> 13.1, 700 x 768 x 3072 33 -> 16.5, 2400 x 320 x 1280 19.0 -> 9.3, its data gradient 20.4 -> 9.1, 1000 x 2048 x 2048
// 19.1 -> 16.3, 4096 x 512 x 2048 18.8 -> 16.9, 2048 x 768 x 3072 26.3 -> 22.5, 8192 x 1024 x 4096 75.9 -> 66.9,
// 8192 x 4096 x 1024 84.9 -> 73.2.  Weights that come from
// memory add 1.5 - 3 us to a launch; more slabs ahead (6 and 8) did not take that back.
//
// The sum over the contraction is cut by WK (see PmAsyncCfg) and otherwise in index order, fp32 accumulation throughout.
#pragma once
#include "pm_gemm_async_api.hpp"

// BI x BJ outputs per block; WI x WJ waves tile them, WK groups of such waves share every slab of BK contraction indices
// (each takes BK / WK of them; the groups' sums meet in LDS at the end); ST slabs in LDS.
template <int BI_, int BJ_, int WI_, int WJ_, int WK_, int BK_, int ST_>
struct PmAsyncCfg {
  static constexpr int BI = BI_, BJ = BJ_, WI = WI_, WJ = WJ_, WK = WK_, BK = BK_, ST = ST_, NT = WI_ * WJ_ * WK_ * 64;
  static constexpr int TI = BI / WI / 32, TJ = BJ / WJ / 32, KS = BK / 16 / WK;
  static_assert(BI % (WI * 32) == 0 && BJ % (WJ * 32) == 0 && BK % (16 * WK) == 0, "tile shape");
};

// A slab of an operand in LDS: KC as ROWS rows of BK indices, RC as BK rows of ROWS.  A wave's load writes 1 KB of
// consecutive LDS, so there is no padding; instead piece c (16 bytes) of LDS row r lies in place c ^ swz(r).  KC: the 16
// lanes of a fragment read's phase then cover all banks once.  RC: a transpose read touches 4 consecutive rows, 32 bytes
// each per group of 16 lanes and the next 32 in the group beside it; swz is even, so that the 32 bytes stay together.
template <int ROWS, bool KC, int BK>
struct PmAsyncTile {
  static constexpr int rows = KC ? ROWS : BK, cpr = (KC ? BK : ROWS) / 8, chunks = rows * cpr, bytes = chunks * 16;
  static constexpr __host__ __device__ int swz(int r) {
    if (KC) return cpr >= 16 ? r & 15 : (r / (16 / cpr)) & (cpr - 1);
    return cpr == 4 ? 2 * ((r >> 3) & 1) : cpr == 8 ? 4 * ((r >> 1) & 1) ^ 2 * ((r >> 3) & 1) : 4 * (r & 3) ^ 2 * ((r >> 3) & 1);
  }
};

typedef int pm_i32x4 __attribute__((ext_vector_type(4)));
// Loads of one operand's slabs, in order.  Every load carries the bounds of what it may touch: the buffer descriptor states
// the bytes from the slab's first element to the end of the operand's last row (KC) or index (RC) inside the tile, and the load unit
// writes zeros for a piece that starts beyond.
template <int ROWS, bool KC, int BK, int NT>
struct PmAsyncLoader {
  using S = PmAsyncTile<ROWS, KC, BK>;
  static_assert(S::chunks % NT == 0, "tile must split evenly over the block");
  static constexpr int PER = S::chunks / NT;
  uint32_t off[PER];       // byte offsets of this thread's pieces from the slab's first element
  uint64_t base, step;     // the next slab's first element, bytes from slab to slab
  int64_t ld;
  int rows;                // valid rows (KC: of the tile, RC: to the end of the operand, in whole groups of 8)
  // tid of NT threads
  __device__ __forceinline__ void init(const bf16_t* X, int64_t ld_, int r0, int R, int tid) {
    ld = ld_;
    rows = KC ? (R - r0 < ROWS ? R - r0 : ROWS) : ((R + 7) & ~7) - r0;
    start(X, r0);
    step = (uint64_t)(KC ? BK : BK * ld) * 2;
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int c = p * NT + tid, r = c / S::cpr, q = (c % S::cpr) ^ S::swz(r);
      off[p] = (uint32_t)(r * (int)ld * 2 + q * 16);
    }
  }
  __device__ __forceinline__ void start(const bf16_t* X, int r0) {
    base = (uint64_t)(uintptr_t)(KC ? X + (int64_t)r0 * ld : X + r0);
  }
  // the next slab into LDS at s (wave-uniform); left: contraction indices from its first one to the end.  TAIL: left < BK
  template <bool TAIL>
  __device__ __forceinline__ void load(uint32_t s, int left, int wave, int tid) {
    const int k8 = TAIL ? (left + 7) & ~7 : BK;
    const int64_t last = KC ? (rows - 1) * ld + k8 : ((TAIL ? left : BK) - 1) * ld + rows;
    const pm_i32x4 rsrc = {(int)__builtin_amdgcn_readfirstlane((uint32_t)base), (int)__builtin_amdgcn_readfirstlane((uint32_t)(base >> 32) & 0xffffu),
                           (int)__builtin_amdgcn_readfirstlane((uint32_t)(last * 2)), 0x00020000};
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      uint32_t o = off[p];
      if (TAIL && KC) {                                  // indices past the end inside a row: past the end of the buffer
        const int c = p * NT + tid, r = c / S::cpr, q = (c % S::cpr) ^ S::swz(r);
        if (q * 8 >= left) o = 0x7ffffff0u;
      }
      // (by hand: behind the compiler's own form it puts a wait for all loads in front of every transpose read; nothing is
      // returned to registers, and the waits for the LDS contents are counted in pm_wait_vm_lds0)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                   :: "s"(s + (p * (NT / 64) + wave) * 1024), "v"(o), "s"(rsrc) : "memory", "m0");
    }
    base += step;
  }
};
// the descriptor and the offsets are 32 bits wide
template <class Cfg>
inline bool pm_async_fits(int64_t lda, int64_t ldb) {
  constexpr int64_t most = Cfg::BI > Cfg::BJ ? (Cfg::BI > Cfg::BK ? Cfg::BI : Cfg::BK) : (Cfg::BJ > Cfg::BK ? Cfg::BJ : Cfg::BK);
  return (lda > ldb ? lda : ldb) * 2 * most < ((int64_t)1 << 31) - 65536;
}

// the lane's part of the fragments' LDS addresses
template <int ROWS, bool KC, int BK>
struct PmAsyncFrag {
  using S = PmAsyncTile<ROWS, KC, BK>;
  int a0, x0;
  __device__ __forceinline__ void init(int lane) {
    if (KC) {
      a0 = (lane & 31) * S::cpr * 16;
      x0 = (lane >> 5) ^ S::swz(lane & 31);
    } else {                                             // (see pm_read_frag for the lanes of a transpose read)
      const int g = lane >> 4, q = lane & 15, k = 8 * (g >> 1) + (q >> 2);
      a0 = k * S::cpr * 16 + 8 * (q & 1);
      x0 = (2 * (g & 1) + ((q & 3) >> 1)) ^ S::swz(k);
    }
  }
  // operand rows r32 .. r32 + 31, contraction indices kb .. kb + 15 of the slab (multiples of 32 and 16)
  __device__ __forceinline__ pm_bf16x8 read(const unsigned char* s, int r32, int kb) const {
    if (KC) {
      return *reinterpret_cast<const pm_bf16x8*>(s + r32 * S::cpr * 16 + a0 + (((kb >> 3) ^ x0) << 4));
    } else {
      typedef pm_v4s __attribute__((address_space(3))) * lds_v4s;
      const unsigned char* p = s + kb * S::cpr * 16 + a0 + (((r32 >> 3) ^ x0) << 4);
      union { pm_bf16x8 v; pm_v4s h[2]; } u;
      u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(p));
      u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(p + 4 * S::cpr * 16));
      return u.v;
    }
  }
};

template <int VM>
__device__ __forceinline__ void pm_wait_vm_lds0() {          // at most VM loads outstanding, no LDS access outstanding
  static_assert(VM < 64, "the counter has 6 bits");
  __builtin_amdgcn_s_waitcnt((VM & 15) | (7 << 4) | ((VM >> 4) << 14));
}
// at most min(n, N) slabs of PER loads each outstanding (n uniform)
template <int N, int PER>
__device__ __forceinline__ void pm_wait_slabs(int n) {
  if constexpr (N == 0) pm_wait_vm_lds0<0>();
  else if (n >= N) pm_wait_vm_lds0<N * PER>();
  else pm_wait_slabs<N - 1, PER>(n);
}
__device__ __forceinline__ void pm_block_sync() {            // a barrier without the waits of __syncthreads
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

template <class Cfg, class Epi>
struct PmAsyncLds {
  static constexpr bool AKC = Epi::kAKC, BKC = Epi::kBKC;
  static constexpr int stage = PmAsyncTile<Cfg::BI, AKC, Cfg::BK>::bytes + PmAsyncTile<Cfg::BJ, BKC, Cfg::BK>::bytes;
  // what the epilogue passes through LDS.  WK > 1: the groups' whole tiles; else a 32-row stripe per wave
  static constexpr int red = Cfg::WK > 1 ? Cfg::WK * Cfg::BI * (Cfg::BJ + 4) * 4 : Cfg::WI * Cfg::WJ * 32 * (Cfg::TJ * 32 + 4) * 4;
  static constexpr int bytes = Cfg::ST * stage > red ? Cfg::ST * stage : red;
};

// Block ids go round the 8 XCDs: XCD x takes the x-th eighth of the tiles, walked in panels of 8 row tiles, so that the
// blocks that share operand panels share an L2.
__device__ __forceinline__ int pm_async_xcd_order(int id, int nblk) {
  const int x = id & 7, part = nblk >> 3, more = nblk & 7;
  return x * part + (x < more ? x : more) + (id >> 3);
}
__device__ __forceinline__ void pm_async_tile_of(int id, int tiles_i, int tiles_j, int& by, int& bx) {
  constexpr int GROUP = 8;
  const int panel = id / (GROUP * tiles_j), first = panel * GROUP, at = id % (GROUP * tiles_j);
  const int rows = tiles_i - first < GROUP ? tiles_i - first : GROUP;
  by = first + at % rows;
  bx = at / rows;
}

struct PmNoSeg {
  static constexpr bool on = false;
};

// Tile (by, bx).  CHECK false: whole tiles and whole slabs only.  Seg: PmNoSeg, or PmKSeg3 = three operand pairs
// of Kseg indices each, one behind the other.
template <class Cfg, bool CHECK, class Epi, class Seg = PmNoSeg>
__device__ __forceinline__ void pm_gemm_async_body(const PmGemmProb<Epi>& pr, int by, int bx, unsigned char* smem,
                                                   const Seg& sg = Seg()) {
  constexpr bool AKC = Epi::kAKC, BKC = Epi::kBKC;
  constexpr int BI = Cfg::BI, BJ = Cfg::BJ, WI = Cfg::WI, WJ = Cfg::WJ, WK = Cfg::WK, BK = Cfg::BK, ST = Cfg::ST, NT = Cfg::NT;
  constexpr int TI = Cfg::TI, TJ = Cfg::TJ, KS = Cfg::KS;
  using SA = PmAsyncTile<BI, AKC, BK>;
  constexpr int STAGE = PmAsyncLds<Cfg, Epi>::stage;
  const int I = pr.I, J = pr.J;
  const int i0 = by * BI, j0 = bx * BJ;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wj = wave % WJ, wi = (wave / WJ) % WI, wk = wave / (WJ * WI);
  const int lr = lane & 31, kg = lane >> 5;

  PmAsyncLoader<BI, AKC, BK, NT> la;
  PmAsyncLoader<BJ, BKC, BK, NT> lb;
  la.init(pr.A, pr.lda, i0, I, threadIdx.x);
  lb.init(pr.B.get(), pr.ldb, j0, J, threadIdx.x);
  constexpr int PER = decltype(la)::PER + decltype(lb)::PER;
  int Ks = pr.K, nk = (Ks + BK - 1) / BK, seg = 0;       // indices of a segment, slabs in all
  if constexpr (Seg::on) {
    Ks = sg.Kseg;
    nk = 3 * ((Ks + BK - 1) / BK);
  }
  int left = Ks;                                         // indices of the segment from the next slab on
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
  auto issue = [&](int place) __attribute__((always_inline)) {      // the next slab; place: its byte offset in LDS
    const uint32_t s = lds0 + place;
    if (CHECK && left < BK) {
      la.template load<true>(s, left, wave, threadIdx.x);
      lb.template load<true>(s + SA::bytes, left, wave, threadIdx.x);
    } else {
      la.template load<false>(s, left, wave, threadIdx.x);
      lb.template load<false>(s + SA::bytes, left, wave, threadIdx.x);
    }
    left -= BK;
    if constexpr (Seg::on) {
      if (left <= 0 && seg < 2) {
        const bf16_t *a1 = sg.A1, *a2 = sg.A2, *b1 = sg.B1.get(), *b2 = sg.B2.get();
        la.start(seg == 0 ? a1 : a2, i0);
        lb.start(seg == 0 ? b1 : b2, j0);
        ++seg;
        left = Ks;
      }
    }
  };
#pragma unroll
  for (int s = 0; s < ST; ++s)
    if (s < nk) issue(s * STAGE);
  PmAsyncFrag<BI, AKC, BK> ra;
  PmAsyncFrag<BJ, BKC, BK> rb;
  ra.init(lane);
  rb.init(lane);

  pm_f32x16 acc[TI][TJ];
#pragma unroll
  for (int a = 0; a < TI; ++a)
#pragma unroll
    for (int b = 0; b < TJ; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;
  struct Frags { pm_bf16x8 a[KS][TI], b[KS][TJ]; };
  auto read = [&](int place, Frags& f) __attribute__((always_inline)) {
    const unsigned char* s = smem + place;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int kb = (wk * KS + ks) * 16;
#pragma unroll
      for (int a = 0; a < TI; ++a) f.a[ks][a] = ra.read(s, (wi * TI + a) * 32, kb);
#pragma unroll
      for (int b = 0; b < TJ; ++b) f.b[ks][b] = rb.read(s + SA::bytes, (wj * TJ + b) * 32, kb);
    }
  };
  // bias gradient: column sums of A, from the fragments of the first column of tiles; of the WJ waves that hold the same rows
  // each sums a share of the 32-row tiles (one register of sums: with all four tiles per wave the 256 x 256 block spilled)
  constexpr bool COLSUM = Epi::kColSumA && !AKC;
  float cs[(TI + WJ - 1) / WJ] = {};
  const bool do_colsum = COLSUM && bx == 0 && pr.epi.wants_colsum();
  auto mul = [&](const Frags& f) __attribute__((always_inline)) {
    if constexpr (COLSUM) {
      if (do_colsum) {
#pragma unroll
        for (int a = 0; a < TI; ++a)
          if (a % WJ == wj) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) cs[a / WJ] += pm_frag_sum(f.a[ks][a]);
          }
      }
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int a = 0; a < TI; ++a)
#pragma unroll
        for (int b = 0; b < TJ; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[ks][a], f.b[ks][b], acc[a][b], 0, 0, 0);
  };
  // waits until a slab has landed for every wave; `behind` slabs requested after it may still be on their way
  auto arrive = [&](int behind) __attribute__((always_inline)) {
    pm_wait_slabs<ST - 1, PER>(behind);
    pm_block_sync();
  };
  Frags f0, f1;
  arrive(nk - 1 < ST - 1 ? nk - 1 : ST - 1);
  read(0, f0);
  // Slab kt is in registers (cur).  Once every wave has read it (its own reads are waited for in front of the barrier) its place in LDS takes slab
  // kt + ST; slab kt + 1 goes to registers (nxt) under the products of slab kt.
  int here = 0;                                          // place of slab kt
  auto slab = [&](auto steady, int kt, const Frags& cur, Frags& nxt) __attribute__((always_inline)) {
    constexpr bool STEADY = decltype(steady)::value;     // slabs kt + 1 .. kt + ST exist
    if (STEADY || kt + 1 < nk) {
      const int behind = nk - 2 - kt;                    // slabs after kt + 1; requested are those up to kt + ST - 1
      if (STEADY) { pm_wait_vm_lds0<(ST - 2) * PER>(); pm_block_sync(); }
      else arrive(behind < ST - 2 ? behind : ST - 2);
      const int freed = here;
      here = here == (ST - 1) * STAGE ? 0 : here + STAGE;
      read(here, nxt);
      __builtin_amdgcn_sched_barrier(0);
      if (STEADY || kt + ST < nk) issue(freed);
      __builtin_amdgcn_sched_barrier(0);
    }
    mul(cur);
  };
  int kt = 0;
  for (; kt + 1 + ST < nk; kt += 2) {
    slab(std::true_type{}, kt, f0, f1);
    slab(std::true_type{}, kt + 1, f1, f0);
  }
  for (; kt + 1 < nk; kt += 2) {
    slab(std::false_type{}, kt, f0, f1);
    slab(std::false_type{}, kt + 1, f1, f0);
  }
  if (kt < nk) slab(std::false_type{}, kt, f0, f1);

  Epi epi = pr.epi;
  epi.begin();
  if constexpr (COLSUM) {
    if (do_colsum) {                                     // uniform over the block
      float* part = reinterpret_cast<float*>(smem);      // [WK][BI]
      __syncthreads();
#pragma unroll
      for (int a = 0; a < TI; ++a)
        if (a % WJ == wj) {
          const float half = cs[a / WJ] + __shfl_xor(cs[a / WJ], 32, 64);
          if (lane < 32) part[wk * BI + (wi * TI + a) * 32 + lane] = half;
        }
      __syncthreads();
      if ((int)threadIdx.x < BI && i0 + (int)threadIdx.x < I) {
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < WK; ++w) sum += part[w * BI + threadIdx.x];
        epi.colsum(i0 + threadIdx.x, sum);
      }
    }
  }
  auto store = [&](auto check_) __attribute__((always_inline)) {
  constexpr bool CHECKED = decltype(check_)::value;
  float* red = reinterpret_cast<float*>(smem);
  __syncthreads();                                       // every wave has read its last slab
  // A lane takes 8 consecutive columns of a row, in groups of pieces whose memory reads are requested together.
  // value v of a 32 x 32 tile's accumulator: row 8 (v / 4) + 4 (lane / 32) + v % 4, column lane % 32
  if constexpr (WK == 1) {
    // a wave's 32-row stripes pass through a part of LDS of its own: no barrier
    constexpr int WT_J = TJ * 32, ES = WT_J + 4, ITERS = 32 * (WT_J / 8) / 64;
    float* es = red + (size_t)wave * 32 * ES;
    const int wi0 = i0 + wi * TI * 32, wj0 = j0 + wj * WT_J;
#pragma unroll
    for (int a = 0; a < TI; ++a) {
#pragma unroll
      for (int b = 0; b < TJ; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) es[(8 * (v >> 2) + 4 * kg + (v & 3)) * ES + b * 32 + lr] = acc[a][b][v];
      typename Epi::Pre pre[ITERS];
      bool full[ITERS];
#pragma unroll
      for (int u = 0; u < ITERS; ++u) {
        const int c = lane + 64 * u, i = wi0 + a * 32 + c / (WT_J / 8), j = wj0 + c % (WT_J / 8) * 8;
        full[u] = !CHECKED || (i < I && j + 8 <= J);
        if (full[u]) pre[u] = epi.pre8(i, j);
      }
#pragma unroll
      for (int u = 0; u < ITERS; ++u) {
        const int c = lane + 64 * u, r = c / (WT_J / 8), c8 = c % (WT_J / 8) * 8, i = wi0 + a * 32 + r, j = wj0 + c8;
        if (CHECKED && (i >= I || j >= J)) continue;
        float vals[8];
        const float4 v0 = *reinterpret_cast<const float4*>(es + r * ES + c8);
        const float4 v1 = *reinterpret_cast<const float4*>(es + r * ES + c8 + 4);
        vals[0] = v0.x; vals[1] = v0.y; vals[2] = v0.z; vals[3] = v0.w;
        vals[4] = v1.x; vals[5] = v1.y; vals[6] = v1.z; vals[7] = v1.w;
        if (full[u]) {
          epi.op8(i, j, vals, pre[u]);
        } else {
          for (int e = 0; e < 8 && j + e < J; ++e) epi(i, j + e, vals[e]);
        }
      }
    }
  } else {
    constexpr int ES = BJ + 4, TOTAL = BI * BJ / 8, PIECES = (TOTAL + NT - 1) / NT, GRP = PIECES < 4 ? PIECES : 4;
    static_assert(PIECES % GRP == 0 && (TOTAL % NT == 0 || PIECES == 1), "output pieces must split evenly");
#pragma unroll
    for (int a = 0; a < TI; ++a)
#pragma unroll
      for (int b = 0; b < TJ; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          red[(wk * BI + (wi * TI + a) * 32 + 8 * (v >> 2) + 4 * kg + (v & 3)) * ES + (wj * TJ + b) * 32 + lr] = acc[a][b][v];
    __syncthreads();
#pragma unroll
    for (int g0 = 0; g0 < PIECES; g0 += GRP) {
      typename Epi::Pre pre[GRP];
      bool full[GRP];
#pragma unroll
      for (int u = 0; u < GRP; ++u) {
        const int c = (g0 + u) * NT + threadIdx.x, i = i0 + c / (BJ / 8), j = j0 + c % (BJ / 8) * 8;
        full[u] = (TOTAL % NT == 0 || c < TOTAL) && (!CHECKED || (i < I && j + 8 <= J));
        if (full[u]) pre[u] = epi.pre8(i, j);
      }
#pragma unroll
      for (int u = 0; u < GRP; ++u) {
        const int c = (g0 + u) * NT + threadIdx.x, r = c / (BJ / 8), c8 = c % (BJ / 8) * 8, i = i0 + r, j = j0 + c8;
        if ((TOTAL % NT && c >= TOTAL) || (CHECKED && (i >= I || j >= J))) continue;
        float vals[8] = {};
#pragma unroll
        for (int w = 0; w < WK; ++w) {
          const float4 v0 = *reinterpret_cast<const float4*>(red + (w * BI + r) * ES + c8);
          const float4 v1 = *reinterpret_cast<const float4*>(red + (w * BI + r) * ES + c8 + 4);
          vals[0] += v0.x; vals[1] += v0.y; vals[2] += v0.z; vals[3] += v0.w;
          vals[4] += v1.x; vals[5] += v1.y; vals[6] += v1.z; vals[7] += v1.w;
        }
        if (full[u]) {
          epi.op8(i, j, vals, pre[u]);
        } else {
          for (int e = 0; e < 8 && j + e < J; ++e) epi(i, j + e, vals[e]);
        }
      }
    }
  }
  };
  if (CHECK && (i0 + BI > I || j0 + BJ > J)) store(std::true_type());
  else store(std::false_type());
  if constexpr (pm_has_tile_update<Epi>::value) {
    static_assert(!CHECK, "whole tiles only");
    __syncthreads();      // the block's stores of the tile are visible to all its waves
    epi.template update_tile<BI, BJ, NT>(i0, j0);
  }
}
// tile `id` of tiles_i x tiles_j, spread over the XCDs
template <class Cfg, bool CHECK, class Epi, class Seg = PmNoSeg>
__device__ __forceinline__ void pm_gemm_async_tile(const PmGemmProb<Epi>& pr, int id, int tiles_i, int tiles_j, unsigned char* smem,
                                                   const Seg& sg = Seg()) {
  int by, bx;
  pm_async_tile_of(pm_async_xcd_order(id, tiles_i * tiles_j), tiles_i, tiles_j, by, bx);
  pm_gemm_async_body<Cfg, CHECK>(pr, by, bx, smem, sg);
}

#define PM_ASYNC_KERNEL __global__ __launch_bounds__(Cfg::NT) __attribute__((amdgpu_waves_per_eu(2))) void

// one product; blocks from tiles_i * tiles_j on read ahead the next product's weights (see PmPrefetch)
template <class Cfg, bool CHECK, class Epi>
PM_ASYNC_KERNEL pm_gemm_async_kernel(PmGemmProb<Epi> pr, PmPrefetch pf, int tiles_i, int tiles_j) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[PmAsyncLds<Cfg, Epi>::bytes];
  const int nt = tiles_i * tiles_j;
  if ((int)blockIdx.x >= nt) {
    pm_prefetch_block(pf, blockIdx.x - nt, 0, gridDim.x - nt, 1);
    return;
  }
  pm_gemm_async_tile<Cfg, CHECK>(pr, blockIdx.x, tiles_i, tiles_j, smem);
}

// A product of few outputs and at most 1024 indices (the layers of a chain at 16 .. 256 rows): 32 x 32 outputs per block, wave w
// takes indices 64 w .. 64 w + 63 through 8 KB of LDS of its own.  Everything is requested at once and a wave waits for nobody
// until the partial tiles are added, which bounds it: launch, one memory latency, 64 KB of partials through LDS, the store.
template <class Epi>
__device__ __forceinline__ void pm_gemm_once_body(const PmGemmProb<Epi>& pr, int id, int tiles_i, int tiles_j, unsigned char* smem) {
  constexpr bool BKC = Epi::kBKC;
  using SA = PmAsyncTile<32, true, 64>;
  constexpr int PART = SA::bytes + PmAsyncTile<32, BKC, 64>::bytes;
  static_assert(PART == 8192, "a wave's part of LDS");
  int by, bx;
  pm_async_tile_of(pm_async_xcd_order(id, tiles_i * tiles_j), tiles_i, tiles_j, by, bx);
  const int I = pr.I, J = pr.J, K = pr.K, i0 = by * 32, j0 = bx * 32;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int k0 = wave * 64, nw = (K + 63) >> 6;          // waves with a share
  const bf16_t* B = pr.B.get();
  Epi epi = pr.epi;
  if (wave < nw) {
    PmAsyncLoader<32, true, 64, 64> la;
    PmAsyncLoader<32, BKC, 64, 64> lb;
    la.init(pr.A + k0, pr.lda, i0, I, lane);
    lb.init(B + (BKC ? k0 : k0 * pr.ldb), pr.ldb, j0, J, lane);
    const uint32_t s = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem + wave * PART;
    if (K - k0 < 64) {
      la.template load<true>(s, K - k0, 0, lane);
      lb.template load<true>(s + SA::bytes, K - k0, 0, lane);
    } else {
      la.template load<false>(s, K - k0, 0, lane);
      lb.template load<false>(s + SA::bytes, K - k0, 0, lane);
    }
    PmAsyncFrag<32, true, 64> ra;
    PmAsyncFrag<32, BKC, 64> rb;
    ra.init(lane);
    rb.init(lane);
    pm_f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    pm_wait_vm_lds0<0>();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    pm_bf16x8 fa[4], fb[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      fa[ks] = ra.read(smem + wave * PART, 0, ks * 16);
      fb[ks] = rb.read(smem + wave * PART + SA::bytes, 0, ks * 16);
    }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ks], fb[ks], acc, 0, 0, 0);
    // the partial tile over the wave's own operands (its LDS accesses complete in order)
    float* red = reinterpret_cast<float*>(smem + wave * PART);
#pragma unroll
    for (int v = 0; v < 16; ++v) red[(8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * 32 + (lane & 31)] = acc[v];
  }
  epi.begin();
  __syncthreads();
  const int e = threadIdx.x, i = i0 + e / 32, j = j0 + e % 32;
  const float* red = reinterpret_cast<const float*>(smem) + e;
  float sum = 0.f;
#pragma unroll
  for (int w = 0; w < 16; ++w)
    if (w < nw) sum += red[w * (PART / 4)];
  if (i < I && j < J) epi(i, j, sum);
}
template <class Epi>
__global__ __launch_bounds__(1024) void pm_gemm_once_kernel(PmGemmProb<Epi> pr, PmPrefetch pf, int tiles_i, int tiles_j) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[16 * 8192];
  const int nt = tiles_i * tiles_j;
  if ((int)blockIdx.x >= nt) {
    pm_prefetch_block(pf, blockIdx.x - nt, 0, gridDim.x - nt, 1);
    return;
  }
  pm_gemm_once_body(pr, blockIdx.x, tiles_i, tiles_j, smem);
}

// three products of equal shape in one launch (the query / key / value projections share their input)
template <class Cfg, bool CHECK, class Epi>
PM_ASYNC_KERNEL pm_gemm_async_multi3_kernel(PmGemmProb<Epi> p0, PmGemmProb<Epi> p1, PmGemmProb<Epi> p2, int tiles_i, int tiles_j) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[PmAsyncLds<Cfg, Epi>::bytes];
  const int nt = tiles_i * tiles_j, p = blockIdx.x / nt;          // uniform over the block
  pm_gemm_async_tile<Cfg, CHECK>(p == 0 ? p0 : p == 1 ? p1 : p2, blockIdx.x - p * nt, tiles_i, tiles_j, smem);
}

// one product over three operand pairs, out = A0 B0 + A1 B1 + A2 B2 (their data gradients meet in one tensor)
template <class Cfg, bool CHECK, class Epi>
PM_ASYNC_KERNEL pm_gemm_async_kseg3_kernel(PmGemmProb<Epi> pr, PmKSeg3 sg, int tiles_i, int tiles_j) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[PmAsyncLds<Cfg, Epi>::bytes];
  pm_gemm_async_tile<Cfg, CHECK>(pr, blockIdx.x, tiles_i, tiles_j, smem, sg);
}

// One product with a long contraction and too few output tiles to fill the chip, its contraction cut into parts that
// run side by side: block b works on part b / (tiles_i * tiles_j), indices part * kpart on, and writes that part's fp32
// output at part * part_stride; the consumer adds the parts in order.  kpart is a multiple of 64.
template <class Cfg, bool CHECK, class Epi>
PM_ASYNC_KERNEL pm_gemm_async_ksplit_kernel(PmGemmProb<Epi> pr, int kpart, int64_t part_stride, int tiles_i, int tiles_j) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[PmAsyncLds<Cfg, Epi>::bytes];
  const int nt = tiles_i * tiles_j, p = blockIdx.x / nt, k0 = p * kpart;       // uniform over the block
  pr.A += k0;
  pr.B.base += (int64_t)k0 * (Epi::kBKC ? 1 : pr.ldb);
  pr.K = pr.K - k0 < kpart ? pr.K - k0 : kpart;
  pr.epi.out += p * part_stride;
  pm_gemm_async_tile<Cfg, CHECK>(pr, blockIdx.x - p * nt, tiles_i, tiles_j, smem);
}

// Weight gradients of whole tiles, many problems in one launch, by per-XCD work lists as in pm_gemm_big_grouped_kernel.  12 x 1024
// layers, 8192 rows, with the update of the parameters inside: 3801 us with the operands through registers, 3640 here; 6 x 512
// layers, 4096 rows: 264 -> 239.  (Ragged problems and accumulating ones stay on 128 x 128 blocks there, two of which share a compute
// unit: what bounds those is the gradient's read and write, and 16000 x 768 and twelve smaller ones took 192 us there, 206 here.)
template <class Cfg, class Epi>
PM_ASYNC_KERNEL pm_gemm_async_grouped_kernel(const PmGemmProb<Epi>* __restrict__ probs, const PmXcdSeg* __restrict__ segs, const int32_t* __restrict__ xcd_tiles, int max_segs) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[PmAsyncLds<Cfg, Epi>::bytes];
  const int x = blockIdx.x & 7, pos = blockIdx.x >> 3;
  if (pos >= xcd_tiles[x]) return;
  const PmXcdSeg* list = segs + (size_t)x * max_segs;
  int lo = 0, hi = max_segs - 1;                 // last segment with start <= pos
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (list[mid].start <= pos) lo = mid; else hi = mid - 1;
  }
  const PmXcdSeg sg = list[lo];
  const PmGemmProb<Epi> pr = probs[sg.prob];
  const int ti = (pr.I + Cfg::BI - 1) / Cfg::BI, tj = (pr.J + Cfg::BJ - 1) / Cfg::BJ;
  int by, bx;
  pm_async_tile_of(sg.tile0 + (pos - sg.start), ti, tj, by, bx);
  pm_gemm_async_body<Cfg, false>(pr, by, bx, smem);
}

// Block shapes, and what a launch on each costs: us = start + rounds * (per1k * K / 1000 + round), rounds = blocks over 256
// compute units, rounded up.  Fitted to 73 measured products (16 .. 8192 rows, 256 .. 20000 columns, K = 320 .. 32000, both
// directions, weights from memory; rms 8 - 18 %): the shape this rule picks took 0.9 % longer than the fastest of each, and 14 % less than
// the kernels before.  per1k is the operand traffic (32 x 32: 128 KB per 1000 indices) or, from 256 x 128 on, the matrix units.
struct PmAsyncCost { float start, per1k, round; };
template <class Cfg> struct PmAsyncShape;
using PmAsync32 = PmAsyncCfg<32, 32, 1, 1, 8, 128, 4>;
using PmAsync64x32 = PmAsyncCfg<64, 32, 2, 1, 4, 128, 3>;
using PmAsync64Short = PmAsyncCfg<64, 64, 2, 2, 1, 64, 3>;
using PmAsync64 = PmAsyncCfg<64, 64, 2, 2, 2, 64, 4>;
using PmAsync128x64 = PmAsyncCfg<128, 64, 2, 2, 2, 64, 4>;
using PmAsync128Pair = PmAsyncCfg<128, 128, 2, 2, 1, 64, 2>;
using PmAsync128 = PmAsyncCfg<128, 128, 2, 2, 2, 64, 3>;
using PmAsync256x128 = PmAsyncCfg<256, 128, 4, 2, 1, 64, 3>;
using PmAsync256 = PmAsyncCfg<256, 256, 2, 4, 1, 32, 4>;
template <> struct PmAsyncShape<PmAsync32> { static constexpr PmAsyncCost cost{3.29f, 2.07f, 0.f}; };
template <> struct PmAsyncShape<PmAsync64x32> { static constexpr PmAsyncCost cost{3.23f, 2.95f, 0.f}; };
template <> struct PmAsyncShape<PmAsync64Short> { static constexpr PmAsyncCost cost{3.62f, 3.94f, 0.f}; };
template <> struct PmAsyncShape<PmAsync64> { static constexpr PmAsyncCost cost{3.15f, 3.58f, 0.44f}; };
template <> struct PmAsyncShape<PmAsync128x64> { static constexpr PmAsyncCost cost{0.93f, 5.66f, 2.74f}; };
template <> struct PmAsyncShape<PmAsync128Pair> { static constexpr PmAsyncCost cost{6.29f, 11.23f, 0.f}; };
template <> struct PmAsyncShape<PmAsync128> { static constexpr PmAsyncCost cost{0.76f, 8.13f, 4.81f}; };
template <> struct PmAsyncShape<PmAsync256x128> { static constexpr PmAsyncCost cost{0.f, 12.1f, 7.48f}; };
template <> struct PmAsyncShape<PmAsync256> { static constexpr PmAsyncCost cost{0.f, 21.58f, 11.37f}; };

inline int64_t pm_async_tiles(int I, int J, int BI, int BJ) { return (int64_t)((I + BI - 1) / BI) * ((J + BJ - 1) / BJ); }

template <class Cfg>
inline float pm_async_rounds_us(int64_t blocks, float slabs) {
  constexpr PmAsyncCost c = PmAsyncShape<Cfg>::cost;
  return c.start + (float)((blocks + 255) / 256) * (c.per1k * 1e-3f * slabs + c.round);
}
// the rule for one block shape; n products of I x J outputs over `segs` operand pairs of K indices each
template <class Cfg>
inline float pm_async_us(int n, int I, int J, int K, int segs) {
  return pm_async_rounds_us<Cfg>(n * pm_async_tiles(I, J, Cfg::BI, Cfg::BJ), (float)segs * ((K + Cfg::BK - 1) / Cfg::BK) * Cfg::BK);
}
template <class F>
inline void pm_async_each(F&& f) {
  f(PmAsync32()); f(PmAsync64x32()); f(PmAsync64Short()); f(PmAsync64()); f(PmAsync128x64()); f(PmAsync128Pair()); f(PmAsync128());
  f(PmAsync256x128()); f(PmAsync256());
}

// Calls go(Cfg, whole tiles and slabs?) with the cheapest block shape for `n` products of I x J outputs over `segs` operand pairs of K indices
// each; false (nothing called) where an operand's rows are too long for the loads' 32-bit offsets.
template <class F>
inline bool pm_async_pick(int n, int I, int J, int K, int segs, int64_t lda, int64_t ldb, F&& go) {
  float best = 3e38f;
  int which = -1, at = 0;
  pm_async_each([&](auto cfg) {
    using Cfg = decltype(cfg);
    const float us = pm_async_us<Cfg>(n, I, J, K, segs);
    if (us < best && n * pm_async_tiles(I, J, Cfg::BI, Cfg::BJ) < ((int64_t)1 << 31) && pm_async_fits<Cfg>(lda, ldb)) best = us, which = at;
    ++at;
  });
  if (which < 0) return false;
  at = 0;
  pm_async_each([&](auto cfg) {
    using Cfg = decltype(cfg);
    if (at++ != which) return;
    if (I % Cfg::BI == 0 && J % Cfg::BJ == 0 && K % Cfg::BK == 0) go(cfg, std::true_type());
    else go(cfg, std::false_type());
  });
  return true;
}

template <class Epi>
bool pm_async_try(hipStream_t st, const PmGemmProb<Epi>& pr, const PmPrefetch* pf) {
  const int64_t t32 = pm_async_tiles(pr.I, pr.J, 32, 32);
  if (t32 <= 256 && pr.K <= 1024 && pm_async_fits<PmAsync64>(pr.lda, pr.ldb)) {
    const int ti = (pr.I + 31) / 32, tj = (pr.J + 31) / 32, nt = (int)t32;
    // reading ahead: as many blocks as compute units are idle, in whole rounds over the XCDs
    const int extra = pf && pf->base && (nt & 7) == 0 ? 256 - nt : 0;
    hipLaunchKernelGGL((pm_gemm_once_kernel<Epi>), dim3(nt + extra), dim3(1024), 0, st, pr,
                       extra ? *pf : PmPrefetch{nullptr, nullptr, 0, 0, 0, 0, 0, 0}, ti, tj);
    return true;
  }
  return pm_async_pick(1, pr.I, pr.J, pr.K, 1, pr.lda, pr.ldb, [&](auto cfg, auto whole) {
    using Cfg = decltype(cfg);
    const int ti = (pr.I + Cfg::BI - 1) / Cfg::BI, tj = (pr.J + Cfg::BJ - 1) / Cfg::BJ, nt = ti * tj;
    const int extra = pf && pf->base && nt < 256 && (nt & 7) == 0 ? 256 - nt : 0;
    hipLaunchKernelGGL((pm_gemm_async_kernel<Cfg, !decltype(whole)::value, Epi>), dim3(nt + extra), dim3(Cfg::NT), 0, st, pr,
                       extra ? *pf : PmPrefetch{nullptr, nullptr, 0, 0, 0, 0, 0, 0}, ti, tj);
  });
}

// Three products of equal shape and layout in one launch.  False (nothing launched) if the operands do not suit.
template <class Epi>
bool pm_gemm_multi3_try(hipStream_t st, const PmGemmProb<Epi> (&pr)[3]) {
  const int I = pr[0].I, J = pr[0].J, K = pr[0].K;
  for (int p = 0; p < 3; ++p) {
    if (pr[p].I != I || pr[p].J != J || pr[p].K != K || pr[p].lda != pr[0].lda || pr[p].ldb != pr[0].ldb) return false;
    if (!pm_mfma_takes(I, J, K, pr[p].A, pr[p].lda, 1, pr[p].B.base, pr[p].B.stride, pr[p].ldb, 1)) return false;
  }
  return pm_async_pick(3, I, J, K, 1, pr[0].lda, pr[0].ldb, [&](auto cfg, auto whole) {
    using Cfg = decltype(cfg);
    const int ti = (I + Cfg::BI - 1) / Cfg::BI, tj = (J + Cfg::BJ - 1) / Cfg::BJ;
    hipLaunchKernelGGL((pm_gemm_async_multi3_kernel<Cfg, !decltype(whole)::value, Epi>), dim3(3 * ti * tj), dim3(Cfg::NT), 0, st,
                       pr[0], pr[1], pr[2], ti, tj);
  });
}

// out = sum over p of A_p B_p with A_p (I x Kseg, row-major) and B_p (Kseg x J, row-major) as one product.
template <class Epi>
bool pm_gemm_kseg3_try(hipStream_t st, int I, int J, int Kseg, const bf16_t* const (&A)[3], int64_t lda,
                              const PmWLoc<bf16_t> (&B)[3], int64_t ldb, const Epi& epi) {
  for (int p = 0; p < 3; ++p)
    if (!pm_mfma_takes(I, J, Kseg, A[p], lda, 1, B[p].base, B[p].stride, 1, ldb)) return false;
  const PmGemmProb<Epi> pr{I, J, 3 * Kseg, A[0], lda, B[0], ldb, epi};
  const PmKSeg3 sg{A[1], A[2], B[1], B[2], Kseg};
  return pm_async_pick(1, I, J, Kseg, 3, lda, ldb, [&](auto cfg, auto whole) {
    using Cfg = decltype(cfg);
    const int ti = (I + Cfg::BI - 1) / Cfg::BI, tj = (J + Cfg::BJ - 1) / Cfg::BJ;
    hipLaunchKernelGGL((pm_gemm_async_kseg3_kernel<Cfg, !decltype(whole)::value, Epi>), dim3(ti * tj), dim3(Cfg::NT), 0, st, pr, sg, ti, tj);
  });
}

template <class Epi>
bool pm_gemm_ksplit_try(hipStream_t st, const PmGemmProb<Epi>& pr, const PmKSplit& s, int64_t part_stride) {
  if (s.parts < 2 || !pm_mfma_takes(pr.I, pr.J, pr.K, pr.A, pr.lda, 1, pr.B.base, pr.B.stride, 1, pr.ldb)) return false;
  return pm_async_pick(s.parts, pr.I, pr.J, s.kpart, 1, pr.lda, pr.ldb, [&](auto cfg, auto whole) {
    using Cfg = decltype(cfg);
    const int ti = (pr.I + Cfg::BI - 1) / Cfg::BI, tj = (pr.J + Cfg::BJ - 1) / Cfg::BJ;
    auto go = [&](auto check) {
      hipLaunchKernelGGL((pm_gemm_async_ksplit_kernel<Cfg, decltype(check)::value, Epi>), dim3(s.parts * ti * tj), dim3(Cfg::NT), 0, st,
                         pr, s.kpart, part_stride, ti, tj);
    };
    if (decltype(whole)::value && pr.K % Cfg::BK == 0) go(std::false_type());      // (the last part may be shorter)
    else go(std::true_type());
  });
}
