"""How tree attention is split over workgroups (csrc/tree_attn_plan.hpp), on the CPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PLAN = r"""
#include <cstdio>
#include "tree_attn_plan.hpp"
using namespace ddd;
int main() {
  const int trees[] = {1, 2, 31, 32, 33, 61, 64, 65, 128, 129};
  long long shrinks = 0, over = 0, uncovered = 0, passes = 0, fewer = 0;
  for (int n_cu : {64, 256, 304})
    for (int B = 1; B <= 6; ++B)
      for (int nh = 1; nh <= 40; ++nh)
        for (int T : trees) {
          int before = 0;
          for (int L = 0; L <= 20000; L += (L < 300 ? 1 : L % 32 == 0 ? 1 : 31)) {   // multiples of 32 and the next length
            const int room = tree_attention_splits(B, nh, T, L, n_cu);
            shrinks += room < before;
            before = room;
            const AttnLaunch p = attn_launch(B, nh, T, L, n_cu);
            over += p.nsplit > room || p.nsplit < 1;
            if (p.per == 0) continue;
            ++passes;
            fewer += p.nsplit < room;
            const int all = (L + 31) / 32 + (T + 31) / 32;   // every chunk has a workgroup, every workgroup a chunk
            uncovered += p.per > kPassChunks || p.nsplit * p.per < all || (p.nsplit - 1) * p.per >= all;
          }
        }
  std::printf("%lld %lld %lld %lld %lld\n", shrinks, over, uncovered, passes, fewer);
  return 0;
}
"""


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_a_longer_prompt_needs_no_less_room(tmp_path):
    """The workspace of a longer prompt serves a shorter one (one of a program's longest prompt serves all), no launch takes more
    partials than it holds, and workgroups that take their chunks in one pass cover the keys, none without a chunk."""
    src, exe = tmp_path / "plan.cpp", str(tmp_path / "plan")
    src.write_text(PLAN)
    subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-I",
                    os.path.join(ROOT, "paper_2409_00142_amd", "csrc"), str(src), "-o", exe], check=True)
    out = [int(x) for x in subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split()]
    assert out[:3] == [0, 0, 0] and out[3] > 10000 and out[4] > 1000, out
