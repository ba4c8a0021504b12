// The order in which a pipelined product (pm_gemm_big_body) walks its contraction, and the indices its loads ask for.
// Plain constexpr functions, apart from the kernels, so that a host program can check them.
#pragma once

constexpr int PM_SLAB = 64;      // contraction indices per slab

// STEADY: slabs kt + 1 and kt + 2 exist and lie wholly inside the contraction, so their loads and stores are
// unconditional and unclamped.  SET: which of the two register sets is free.
template <bool STEADY_, int SET_>
struct PmSlabTag {
  static constexpr bool STEADY = STEADY_;
  static constexpr int SET = SET_;
};

// Calls slab(tag, kt) for every slab of a contraction of K indices.  Slab kt requests slab kt + 2, so the second slab of
// a steady pair requests kt + 3, which has to be a whole one as well: with K no multiple of PM_SLAB the last
// slab is requested by a slab that clamps.
template <class F>
constexpr __attribute__((always_inline)) void pm_slab_walk(int K, F&& slab) {
  const int nk = (K + PM_SLAB - 1) / PM_SLAB, whole = K / PM_SLAB;
  int kt = 0;
  for (; kt + 3 < whole; kt += 2) {
    slab(PmSlabTag<true, 0>{}, kt);
    slab(PmSlabTag<true, 1>{}, kt + 1);
  }
  for (; kt < nk; kt += 2) {              // the last one to four slabs
    slab(PmSlabTag<false, 0>{}, kt);
    if (kt + 1 < nk) slab(PmSlabTag<false, 1>{}, kt + 1);
  }
}

// Row or contraction index n of an operand that holds N of them, for a load that may reach past the end: such loads repeat
// the last one.  GROUPS: the index runs along memory and n is the first of a group of 8 (operands are readable up to the
// next multiple of 8).
template <bool GROUPS>
constexpr __attribute__((always_inline)) int pm_clamp_index(int n, int N) {
  const int last = GROUPS ? ((N + 7) & ~7) - 8 : N - 1;
  return n > last ? last : n;
}
