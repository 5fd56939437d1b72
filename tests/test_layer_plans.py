"""Rules of the draft layer's dispatch, on the CPU.  csrc/gemm_plan.hpp: how its products are cut into column tiles and K ranges
(the GEMM and every kernel that adds its partial sums up work the plan out for themselves, so it has to be the same in each of
them).  csrc/attn_plan.hpp: which calls take the attention on the matrix cores."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PLAN = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include "gemm_plan.hpp"
using namespace ddd;
// Every price of random products (sizes of the draft layer and of single linears), and what is wrong with the cheapest plan.
int main() {
  unsigned s = 12345;
  auto rnd = [&](int lo, int hi) { s = s * 1664525u + 1013904223u; return lo + (int)((s >> 8) % (unsigned)(hi - lo + 1)); };
  unsigned long long hash = 1469598103934665603ull;
  int bad = 0, split = 0;
  for (int i = 0; i < 20000; ++i) {
    const int ab = rnd(2, 3), bbmax = ab == 3 ? 5 : (rnd(0, 1) ? 5 : rnd(2, 3));
    const SplitShape g = {ab, bbmax, 2 * rnd(1, 90), 4 * rnd(1, i % 8 ? 4096 : 40000), 256, rnd(0, 3) ? 8 : 1, 1ll << rnd(14, 26)};
    const int n_act = rnd(0, 3) ? rnd(17, 64 * bbmax) : rnd(1, 4096), nblk = (n_act + 31) / 32;
    double best = 0;
    int NT = 0, S = 0;
    for (int l = 0; l < 64; ++l) {
      const auto price = plan_price(g, n_act, plan_least_tiles(g, n_act) + (l & 7), (l >> 3) + 1);
      unsigned char b[sizeof(price)];
      std::memcpy(b, &price, sizeof(price));
      for (unsigned char c : b) hash = (hash ^ c) * 1099511628211ull;
      if (price > 0 && (best == 0 || (double)price < best)) {
        best = (double)price;
        NT = plan_least_tiles(g, n_act) + (l & 7);
        S = (l >> 3) + 1;
      }
    }
    split += S > 1;
    const int bpt = NT ? (nblk + NT - 1) / NT : 0;
    if (NT < 1 || bpt > 2 * bbmax || bpt * NT < nblk || bpt * (NT - 1) >= nblk || S > g.smax || (S > 1 && (long long)S * n_act * g.N > g.cap))
      ++bad;
  }
  std::printf("%llx bad %d split %d\n", hash, bad, split);
  return 0;
}
"""


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_plan_does_not_depend_on_the_compiler(tmp_path):
    """The same prices, bit for bit, with multiplications and additions fused and not; and every product has a plan that covers
    its rows, with no more sums than there is room for."""
    src = tmp_path / "plan.cpp"
    src.write_text(PLAN)
    out = {}
    for mode in ("off", "fast"):
        exe = str(tmp_path / f"plan_{mode}")
        subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-O3", "-std=c++17", "-mfma", f"-ffp-contract={mode}",
                        "-I", os.path.join(ROOT, "paper_2409_00142_amd", "csrc"), str(src), "-o", exe], check=True)
        out[mode] = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split()
    assert out["off"] == out["fast"]
    assert out["off"][1:3] == ["bad", "0"] and int(out["off"][4]) > 1000


ATTENTION = r"""
#include <cstdio>
#include "attn_plan.hpp"
#include "ddd_body.h"
using namespace ddd;
int main() {
  int bad = 0, on = 0;
  for (int L = 0; L <= DDD_BODY_LMAX; ++L)
    for (int step = 0; step < DDD_DMAX; ++step) {
      const bool mf = attention_on_matrix_cores(40, 4, L, step);
      const MfLds m = mf_lds(L, step);
      on += mf;
      if (mf && (m.total > 160 * 1024 || L < 32)) ++bad;
      if (!mf && L >= 32 && (L <= 1024 || L <= 1046 - step)) ++bad;
      for (size_t at : {m.rsum, m.anc, m.ks, m.vs, m.aw, m.sct, m.ph, m.pl}) bad += at % 16 != 0;
      bad += m.spitch % 4 != 0 || m.spitch < L + 3 || m.ppitch % 8 != 0 || m.ppitch < (L + 31) / 32 * 32;
    }
  for (int L : {0, 31, 256}) bad += attention_on_matrix_cores(16, 4, L, 1) || attention_on_matrix_cores(40, 17, L, 1);
  std::printf("bad %d on %d\n", bad, on);
  return 0;
}
"""


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_prompts_on_the_matrix_cores(tmp_path):
    """Batched calls with 32 to 1024 prompt positions, and up to 1046 less the call's number, take the matrix cores, and what
    they lay out in LDS fits a CU."""
    src, exe = tmp_path / "attn.cpp", str(tmp_path / "attn")
    src.write_text(ATTENTION)
    subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2409_00142_amd", "csrc"), str(src), "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split()
    assert out[:2] == ["bad", "0"] and int(out[3]) > 30000
