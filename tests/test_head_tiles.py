"""Tiles of the LM head's MFMA GEMM: the plan on the CPU (csrc/gemm_plan.hpp), its products on the GPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PLAN = r"""
#include <cstdio>
#include "gemm_plan.hpp"
using namespace ddd;
int main() {
  unsigned s = 4711;
  auto rnd = [&](int lo, int hi) { s = s * 1664525u + 1013904223u; return lo + (int)((s >> 8) % (unsigned)(hi - lo + 1)); };
  int bad = 0, wide = 0, narrow = 0;
  for (int i = 0; i < 100000; ++i) {
    const float row2 = rnd(0, 1) ? 0.0171f : rnd(0, 1) ? 0.0196f : 0.042f, once = rnd(0, 1) ? 1.f : 1.23f;
    const HeadShape h = {rnd(1, i % 4 ? 40000 : 131072), 2 * rnd(1, 40), 8 * rnd(1, 32), rnd(0, 1) ? 4 : 10, 0.0171f, row2, once, rnd(0, 1) ? 4 : 1 << 30};
    const int n = rnd(0, 7) ? rnd(1, 700) : rnd(1, 524288), nblk = (n + 31) / 32;
    const HeadPlan p = head_plan_host(h, n);
    // every block of rows has a tile, no tile is empty or wider than its code
    if ((p.bm != 128 && p.bm != 256) || p.NT < 1 || p.NT > nblk || p.bpt != (nblk + p.NT - 1) / p.NT || p.bpt > (p.bm == 256 ? h.most : 10))
      ++bad;
    (p.bm == 256 ? wide : narrow)++;
  }
  // a vocabulary whose 128-row tiles are more than the workgroups, against up to 128 rows: W is received once
  int twice = 0;
  for (int V = 32769; V <= 131072; V += 61)
    for (int kt : {32, 64, 80})
      for (int n = 17; n <= 128; ++n)
        for (int c = 0; c < 16; ++c) {
          const HeadShape h = {V, kt, 256, c & 1 ? 4 : 10, 0.0171f, c & 2 ? 0.0171f : c & 8 ? 0.0196f : 0.042f, c & 4 ? 1.f : 1.23f, 4};
          twice += head_plan_host(h, n).NT > 1;
        }
  std::printf("bad %d wide %d narrow %d twice %d\n", bad, wide, narrow, twice);
  return 0;
}
"""


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_every_call_has_a_plan(tmp_path):
    src, exe = tmp_path / "plan.cpp", str(tmp_path / "plan")
    src.write_text(PLAN)
    subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-I",
                    os.path.join(ROOT, "paper_2409_00142_amd", "csrc"), str(src), "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split()
    assert out[1] == out[7] == "0" and int(out[3]) > 1000 and int(out[5]) > 1000, out


@pytest.mark.gpu
@pytest.mark.parametrize("packed", [False, True], ids=["rows", "packed"])
@pytest.mark.parametrize("V,R", [(32003, R) for R in (17, 33, 97, 161, 257, 320, 330, 385, 447, 450, 513, 577, 640, 700)] +
                         [(4001, 40), (4001, 640), (17001, 449), (17001, 641), (66001, 449), (66001, 130)])
def test_products_of_every_tile(V, R, packed):
    """Logits against the product in 64 bits, for one or two blocks of rows beside every width of tile; the same rows through the
    list of active rows, bit for bit.

    Tolerance: products of bf16 numbers are exact in fp32, 128 sums of terms of size 0.1 round with 2^-24 relative to a partial sum
    of a few units each: below 1e-5."""
    import torch
    import paper_2409_00142_amd as D
    print(f"[case] head_tiles V={V} R={R} packed={packed}", flush=True)
    k, H = 5, 128
    g = torch.Generator(device="cuda")
    g.manual_seed(V + R)
    W = torch.empty(V, H, dtype=torch.bfloat16, device="cuda").normal_(0, 0.1, generator=g)
    hid = torch.empty(R, H, dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    ctx = D.ddd_create(D.make_config((R + k - 1) // k, H, V, k, 3, 10, 0.3))
    try:
        if packed:
            D.ddd_weights_pack(ctx, W)
        outs = []
        for active in (None, (torch.arange(R, device="cuda") % 3 != 1).to(torch.uint8)):
            o = (torch.zeros(R, k, dtype=torch.int32, device="cuda"), torch.zeros(R, k, device="cuda"), torch.zeros(R, device="cuda"))
            dbg = torch.zeros(R, V, device="cuda")
            D.ddd_lmhead_topk(ctx, W, hid, R, active, *o, dbg)
            torch.cuda.synchronize()
            outs.append(o + (dbg,))
        on = active.bool()
    finally:
        D.ddd_destroy(ctx)
    tok, lp, lse, logits = outs[0]
    want = hid.double() @ W.double().T.contiguous()
    assert float((logits.double() - want).abs().max()) < 1e-5
    assert float((lse.double() - torch.logsumexp(want, 1)).abs().max()) < 1e-4
    assert torch.equal(torch.gather(logits, 1, tok.long()) - lse[:, None], lp)
    assert torch.equal(torch.topk(logits, k, dim=1).values, torch.gather(logits, 1, tok.long()))
    for a, b in zip(outs[0], outs[1]):
        assert torch.equal(a[on], b[on])
        assert not bool(b[~on].any())


@pytest.mark.gpu
@pytest.mark.parametrize("packed", [False, True], ids=["rows", "packed"])
@pytest.mark.parametrize("H", [384, 1024])
@pytest.mark.parametrize("V,R", [(32003, R) for R in (17, 64, 97, 161, 225, 289, 330, 385, 447, 450, 513, 577, 640)] +
                         [(17001, R) for R in (200, 257, 330, 450, 577)])
def test_rings_of_every_tile(V, R, H, packed):
    """Six and sixteen k tiles: every slot of the rings (two to four tiles deep) is filled again and read again, for every width of
    the 128-row and 256-row tiles, with as many blocks for each pair of waves and with one less.  W's columns grow with k, so a tile
    of another k cannot pass for the right one.

    Tolerance: products of bf16 numbers are exact in fp32; H additions round a partial sum of a few units by 2^-24 of it at most, and
    128 of them stay below 1e-5 (above)."""
    import torch
    import paper_2409_00142_amd as D
    print(f"[case] head_rings V={V} R={R} H={H} packed={packed}", flush=True)
    k = 5
    g = torch.Generator(device="cuda")
    g.manual_seed(V + R + H)
    W = (torch.empty(V, H, device="cuda").normal_(0, 0.1, generator=g) * torch.linspace(0.5, 1.5, H, device="cuda")).to(torch.bfloat16)
    hid = torch.empty(R, H, dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    ctx = D.ddd_create(D.make_config((R + k - 1) // k, H, V, k, 3, 10, 0.3))
    try:
        if packed:
            D.ddd_weights_pack(ctx, W)
        o = (torch.zeros(R, k, dtype=torch.int32, device="cuda"), torch.zeros(R, k, device="cuda"), torch.zeros(R, device="cuda"))
        dbg = [torch.zeros(R, V, device="cuda") for _ in range(2)]
        for out in dbg:
            D.ddd_lmhead_topk(ctx, W, hid, R, None, *o, out)
        torch.cuda.synchronize()
    finally:
        D.ddd_destroy(ctx)
    want = hid.double() @ W.double().T.contiguous()
    assert torch.equal(dbg[0], dbg[1])
    assert float((dbg[0].double() - want).abs().max()) < 1e-5 * H / 128
    assert torch.equal(torch.topk(dbg[0], k, dim=1).values, torch.gather(dbg[0], 1, o[0].long()))


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["random", "equal", "few_groups", "rising"])
@pytest.mark.parametrize("V,k", [(17, 16), (64, 16), (960, 16), (1024, 16), (16384, 16), (16385, 1), (32768, 16), (32769, 10), (65536, 16),
                                 (65537, 5), (131072, 16)])
def test_row_reduction_of_any_vocabulary(V, k, kind):
    """The reduction's slots per thread and its bound from fewer, as many and more groups than threads and beams: the k best of the
    logits that the same call writes out (ties to the lower token), and the log-sum-exp in 64 bits to 1e-4.  "equal" and
    "few_groups": more candidates than the lists hold; "rising": all of the best in the last groups."""
    import numpy as np
    import torch
    import paper_2409_00142_amd as D
    print(f"[case] row_reduction V={V} k={k} {kind}", flush=True)
    H, B = 128, (16 + k) // k + 1
    R = B * k
    g = torch.Generator(device="cuda")
    g.manual_seed(V * 3 + k)
    W = torch.empty(V, H, dtype=torch.bfloat16, device="cuda").normal_(0, 0.1, generator=g)
    if kind == "equal":
        W[:] = W[0]
    if kind == "few_groups":
        W[: V // 2] = W[0]
    if kind == "rising":
        W[:, 1:] = 0
        W[:, 0] = torch.linspace(0, 8, V, device="cuda").to(torch.bfloat16)
    hid = torch.empty(R, H, dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    if kind == "rising":
        hid[:, 0] = 1.0
    ctx = D.ddd_create(D.make_config(B, H, V, k, 3, 10, 0.3))
    try:
        o = (torch.full((R, k), -7, dtype=torch.int32, device="cuda"), torch.zeros(R, k, device="cuda"), torch.zeros(R, device="cuda"))
        dbg = torch.zeros(R, V, device="cuda")
        D.ddd_lmhead_topk(ctx, W, hid, R, None, *o, dbg)
        torch.cuda.synchronize()
    finally:
        D.ddd_destroy(ctx)
    logits = dbg.cpu().numpy()
    assert np.array_equal(o[0].cpu().numpy(), np.argsort(-logits, axis=1, kind="stable")[:, :k])
    assert float((o[2].double() - torch.logsumexp(dbg.double(), 1)).abs().max()) < 1e-4
