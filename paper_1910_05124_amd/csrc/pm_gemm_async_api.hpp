// Launchers of the bf16 products (pm_gemm_async.hpp).  Their kernels - nine block shapes, six epilogues, with
// and without ragged edges - take a minute and more to compile, so they are instantiated in translation units of their own,
// pm_gemm_fwd.hip, pm_gemm_bwd.hip and pm_gemm_wgrad.hip, for the epilogues named at the end of those files.
#pragma once
#include "pm_gemm_mfma.hpp"

struct PmKSeg3 {                     // pair 0 is the problem's own A and B
  static constexpr bool on = true;
  const bf16_t* A1;
  const bf16_t* A2;
  PmWLoc<bf16_t> B1, B2;
  int Kseg;
};

// One product; pf (may be null): weights that idle blocks read ahead.  All of these return false, with nothing launched, where the
// operands do not suit.
template <class Epi>
bool pm_async_try(hipStream_t st, const PmGemmProb<Epi>& pr, const PmPrefetch* pf);
// Three products of equal shape and layout in one launch.
template <class Epi>
bool pm_gemm_multi3_try(hipStream_t st, const PmGemmProb<Epi> (&pr)[3]);
// out = sum over p of A_p B_p with A_p (I x Kseg, row-major) and B_p (Kseg x J, row-major) as one product.
template <class Epi>
bool pm_gemm_kseg3_try(hipStream_t st, int I, int J, int Kseg, const bf16_t* const (&A)[3], int64_t lda,
                       const PmWLoc<bf16_t> (&B)[3], int64_t ldb, const Epi& epi);
// A product with K >> I, J in parts that run side by side, part p's fp32 output at p * part_stride; the consumer adds them.
struct PmKSplit { int parts, kpart; };      // parts = 1: not cut
PmKSplit pm_ksplit_plan(int I, int J, int K, int max_parts);
template <class Epi>
bool pm_gemm_ksplit_try(hipStream_t st, const PmGemmProb<Epi>& pr, const PmKSplit& s, int64_t part_stride);

// Weight gradients of many units in one launch on 256 x 256 blocks, scheduled per XCD (see pm_gemm_async_grouped_kernel); every problem is
// a whole number of such tiles and of 64 rows.  blocks = 8 x the longest list.
void pm_wgrad_grouped256_launch(hipStream_t st, const PmGemmProb<PmEpiBwdWeight>* probs, const PmXcdSeg* segs,
                                const int32_t* xcd_tiles, int max_segs, int blocks);
void pm_wgrad_grouped256_launch(hipStream_t st, const PmGemmProb<PmEpiBwdWeightUpd>* probs, const PmXcdSeg* segs,
                                const int32_t* xcd_tiles, int max_segs, int blocks);
