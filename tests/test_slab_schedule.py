"""The pipelined bf16 products ask for nothing outside their operands: the slab schedule of the kernels, walked on the host."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1910_05124_amd", "csrc")

# Every slab of a contraction of K indices is loaded once, before it is used, into the register set that the slab two
# before has left free; a load that is not clamped stays inside the contraction, a clamped one inside the
# operand (its rows padded to 8 along memory).
PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "pm_slabs.hpp"
int main() {
  int bad = 0;
  auto check = [&](bool ok, int K, const char* what) { if (!ok) { ++bad; std::printf("K = %d: %s\n", K, what); } };
  for (int K = 1; K <= 14 * PM_SLAB; ++K) {
    const int nk = (K + PM_SLAB - 1) / PM_SLAB;
    std::vector<int> loaded(nk, 0), used(nk, 0);
    auto load = [&](int slab, bool clamp) {
      check(slab < nk, K, "a slab behind the last one");
      if (slab < nk) ++loaded[slab];
      for (int c = 0; c < PM_SLAB; ++c) {
        const int k = slab * PM_SLAB + c;
        check((clamp ? pm_clamp_index<false>(k, K) : k) < K, K, "an index past the end (row-contiguous operand)");
        if (c % 8 == 0) check((clamp ? pm_clamp_index<true>(k, K) : k) + 8 <= (K + 7) / 8 * 8, K, "a group past the end");
      }
    };
    load(0, true);
    if (nk > 1) load(1, true);
    pm_slab_walk(K, [&](auto tag, int kt) {
      const bool steady = decltype(tag)::STEADY;
      check(decltype(tag)::SET == kt % 2, K, "the wrong register set");
      check(kt < nk && loaded[kt] == 1, K, "a slab used before it is loaded");
      if (steady || kt + 2 < nk) load(kt + 2, !steady);
      check(!steady || (kt + 1) * PM_SLAB + PM_SLAB <= K, K, "a partial slab stored without its zeros");
      ++used[kt];
    });
    for (int s = 0; s < nk; ++s) check(loaded[s] == 1 && used[s] == 1, K, "a slab loaded or used twice or not at all");
  }
  return bad != 0;
}
"""


def test_no_load_leaves_the_operands(tmp_path):
    src, exe = tmp_path / "slabs.cpp", tmp_path / "slabs"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0, r.stdout[:2000]
