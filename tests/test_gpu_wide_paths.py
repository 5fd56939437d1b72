"""GPU tests of the wide-beam kernels' branches: row reduction by counting, candidates formed by the row reduction or by the
bookkeeping launch, selection by a bound or (many equal scores) by the radix select."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device (an MI355X)")
    import paper_2409_00142_amd as D
    return torch, D


def _bits(torch, a):
    return torch.from_numpy(a.view(np.int16)).cuda().view(torch.bfloat16)


@pytest.mark.parametrize("k", [17, 64, 65, 100, 128])
@pytest.mark.parametrize("V", [128, 2049, 8191, 65536, 65601, 131072])
def test_wide_row_topk(gpu, k, V):
    """Fewer groups than beams, up to 1024 groups (several threads per group), more (two groups per thread), ragged last
    groups, duplicated rows: tokens from a stable sort of the very logits, exactly."""
    torch, D = gpu
    print(f"[case] wide_row_topk k={k} V={V}", flush=True)
    H, R = 128, 5
    rng = np.random.default_rng(V + k)
    Wb = synth.make_lm_head(V, H, 0.2, V, ((3, V - 1), (5, V // 2)))
    hid = torch.from_numpy(rng.standard_normal((R, H)).astype(np.float32) * 2).cuda().to(torch.bfloat16)
    ctx = D.ddd_create(D.make_config(1, H, V, k, 2, 10, 0.3))
    tok = torch.full((R, k), -7, dtype=torch.int32, device="cuda")
    lp, lse, dbg = torch.zeros(R, k, device="cuda"), torch.zeros(R, device="cuda"), torch.zeros(R, V, device="cuda")
    try:
        D.ddd_lmhead_topk(ctx, _bits(torch, Wb), hid, R, None, tok, lp, lse, dbg)
        torch.cuda.synchronize()
    finally:
        D.ddd_destroy(ctx)
    x = dbg.cpu().numpy()
    want = np.argsort(-x, axis=1, kind="stable")[:, :k]
    assert np.array_equal(tok.cpu().numpy(), want)
    ref = np.log(np.exp(x.astype(np.float64) - x.max(1, keepdims=True)).sum(1)) + x.max(1)
    assert np.max(np.abs(lse.cpu().numpy() - ref)) <= 1e-4
    assert np.array_equal(lp.cpu().numpy(), np.take_along_axis(x, want, 1) - lse.cpu().numpy()[:, None])


@pytest.mark.parametrize("kind", ["random", "equal", "few_values"])
@pytest.mark.parametrize("B,k", [(1, 17), (2, 33), (1, 100), (3, 128)])
def test_draft_step_equals_its_parts(gpu, B, k, kind):
    """ddd_draft_step (candidates formed by the row reduction) against ddd_lmhead_topk + ddd_beam_select +
    ddd_depth_continue (formed by the bookkeeping launch): the same state, bit for bit, call after call; the beam against a
    sort of all candidates.  Equal logits, and rows of a few repeated ones, leave more candidates at the bound than fit."""
    torch, D = gpu
    print(f"[case] wide_draft_step B={B} k={k} {kind}", flush=True)
    H, V, calls = 128, 3000, 4
    rng = np.random.default_rng(B * 1000 + k)
    Wb = synth.make_lm_head(V, H, 0.2, 1)
    if kind == "equal":
        Wb[:] = Wb[0]
    elif kind == "few_values":
        Wb[:] = Wb[np.arange(V) % 7]
    W = _bits(torch, Wb)
    cfg = D.make_config(B, H, V, k, calls, 20, 0.0, 0)
    ctx = D.ddd_create(cfg)
    try:
        one, a = D.alloc_state(cfg)
        two, b = D.alloc_state(cfg)
        for st in (one, two):
            D.ddd_round_reset(ctx, st)
        for s in range(calls):
            R = B if s == 0 else B * k
            hid = torch.from_numpy(rng.standard_normal((R, H)).astype(np.float32) * 2).cuda().to(torch.bfloat16)
            before = {n: t.cpu().numpy().copy() for n, t in a.items()}
            D.ddd_draft_step(ctx, s, W, hid, one)
            tok = torch.zeros(R, k, dtype=torch.int32, device="cuda")
            lp, lse = torch.zeros(R, k, device="cuda"), torch.zeros(R, device="cuda")
            D.ddd_lmhead_topk(ctx, W, hid, R, None, tok, lp, lse)
            D.ddd_beam_select(ctx, s, tok, lp, two)
            D.ddd_depth_continue(ctx, s + 1, two)
            torch.cuda.synchronize()
            for n in a:
                assert torch.equal(a[n], b[n]), (s, n)
            if s == 0:
                continue
            base = 1 + k + (s - 1) * k * k
            got = {n: t.cpu().numpy() for n, t in a.items()}
            t_, l_ = tok.cpu().numpy().reshape(B, k * k), lp.cpu().numpy().reshape(B, k, k)
            for q in range(B):
                sc = (before["logprobsum"][q][:, None] + l_[q]).astype(np.float32).reshape(-1)
                assert np.array_equal(got["pool_score"][q, base:base + k * k], sc)
                assert np.array_equal(got["pool_parent"][q, base:base + k * k], np.repeat(before["beam_node"][q], k))
                order = np.lexsort((np.arange(k * k), t_[q], -sc))[:k]
                assert np.array_equal(got["beam_node"][q], base + order)
                assert np.array_equal(got["beam_token"][q], t_[q][order])
                assert np.array_equal(got["beam_parent_slot"][q], order // k)
                assert np.array_equal(got["logprobsum"][q], sc[order])
    finally:
        D.ddd_destroy(ctx)
