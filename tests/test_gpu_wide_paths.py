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
@pytest.mark.parametrize("V", [128, 2049, 8191, 32768, 32833, 65536, 65601, 131072])
def test_wide_row_topk(gpu, k, V):
    """Fewer groups than beams, up to 512 groups (several threads per group), more (folded by two, from 1025 on by four), ragged
    last groups, duplicated rows: tokens from a stable sort of the very logits, exactly."""
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


def _ordered(scores):
    """fp32 scores as unsigned integers in the total order of the rerank and beam keys (both zeros alike, a positive NaN above
    +inf)."""
    u = (np.ascontiguousarray(scores, dtype=np.float32) + np.float32(0.0)).view(np.uint32)
    return np.where(u >> 31, ~u, u | np.uint32(0x80000000)).astype(np.int64)


def _check_tree(tree, pool, n, m, b):
    """The final tree of sequence b against a sort of its pool's nodes 1 .. n - 1 by (score desc, node id asc)."""
    key = _ordered(pool["pool_score"][b, 1:n])
    best = np.sort(np.lexsort((np.arange(n - 1), -key))[:m] + 1)
    assert tree["n_sel"][b] == len(best)
    assert np.array_equal(tree["sel_node"][b][: len(best)], best)
    for got, want in (("tree_token", "pool_token"), ("pos", "pool_depth")):
        assert np.array_equal(tree[got][b][1 : len(best) + 1], pool[want][b][best])
    parent = pool["pool_parent"][b][best]
    at = np.searchsorted(best, parent)
    known = (at < len(best)) & (best[np.minimum(at, len(best) - 1)] == parent)
    assert np.array_equal(tree["parent_idx"][b][1 : len(best) + 1], np.where(parent == 0, 0, np.where(known, at + 1, -1)))


@pytest.mark.parametrize("special", ["none", "nan_first", "nan_all_of_the_first", "nan_negative", "nan_later", "inf", "minus_inf", "zeros"])
@pytest.mark.parametrize("k,calls,m", [(100, 4, 60), (17, 31, 127), (128, 2, 128)])
def test_final_tree_of_any_scores(gpu, k, calls, m, special):
    """ddd_tree_finalize over pools of several thousand nodes whose scores are not all finite: a NaN (a row whose largest logit
    is infinite has no finite logprob) has its place in the order like any other score."""
    torch, D = gpu
    print(f"[case] wide_tree k={k} calls={calls} m={m} {special}", flush=True)
    B, rng = 2, np.random.default_rng(k + calls)
    n = 1 + k + (calls - 1) * k * k
    depth = np.concatenate([[0], np.ones(k), np.repeat(np.arange(2, calls + 1), k * k)]).astype(np.int32)
    parent = np.concatenate([[-1], np.zeros(k), 1 + np.repeat(np.arange(n - 1 - k) // k, 1) % k]).astype(np.int32)
    score = (-rng.gamma(2.0, 1.0, (B, n)) - depth).astype(np.float32)
    at = {"nan_first": slice(3, 90), "nan_all_of_the_first": slice(1, 257), "nan_negative": slice(1, 257),
          "nan_later": slice(n - 300, n), "inf": slice(40, 50), "minus_inf": slice(10, n), "zeros": slice(5, 250)}
    if special != "none":
        value = {"inf": np.inf, "minus_inf": -np.inf, "zeros": 0.0}.get(special, np.nan)
        bits = np.float32(value).view(np.uint32) | np.uint32(0x80000000 if special == "nan_negative" else 0)
        score.view(np.uint32)[:, at[special]] = bits
        if special == "zeros":
            score[:, 5:250:2] = -0.0
    cfg = D.make_config(B, 128, 4000, k, calls, m, 0.0, 0)
    ctx = D.ddd_create(cfg)
    try:
        st, t = D.alloc_state(cfg)
        tree, tt = D.alloc_tree(cfg)
        tok = rng.integers(0, 4000, (B, n)).astype(np.int32)
        for name, v in (("pool_score", score), ("pool_token", tok), ("pool_parent", np.tile(parent, (B, 1))),
                        ("pool_depth", np.tile(depth, (B, 1)))):
            t[name][:, :n].copy_(torch.from_numpy(v))
        t["n_nodes"].fill_(n)
        D.ddd_tree_finalize(ctx, st, tree)
        torch.cuda.synchronize()
        got, pool = {x: v.cpu().numpy() for x, v in tt.items()}, {x: v.cpu().numpy() for x, v in t.items()}
    finally:
        D.ddd_destroy(ctx)
    for b in range(B):
        _check_tree(got, pool, n, m, b)


@pytest.mark.parametrize("B,k", [(1, 17), (2, 100), (1, 128)])
def test_wide_round_with_an_infinite_logit(gpu, B, k):
    """One hidden row of the second call meets a row of W whose product exceeds fp32 (+inf logit): its logprobs are NaN, and the
    beam, the later calls and the final tree follow the order of the keys like with any other scores."""
    torch, D = gpu
    print(f"[case] wide_infinite_logit B={B} k={k}", flush=True)
    H, V, calls, m = 128, 3000, 4, 40
    rng = np.random.default_rng(k)
    W = _bits(torch, synth.make_lm_head(V, H, 0.2, 1))
    W[:, 0] = 0.0
    W[5, 0] = 3e38
    cfg = D.make_config(B, H, V, k, calls, m, 0.0, 0)
    ctx = D.ddd_create(cfg)
    try:
        st, t = D.alloc_state(cfg)
        tree, tt = D.alloc_tree(cfg)
        D.ddd_round_reset(ctx, st)
        for s in range(calls):
            R = B if s == 0 else B * k
            hid = torch.from_numpy(rng.standard_normal((R, H)).astype(np.float32) * 2).cuda().to(torch.bfloat16)
            hid[:, 0] = 0.0
            if s == 1:
                hid[3, 0] = 100.0
            lps = t["logprobsum"].cpu().numpy().copy()
            D.ddd_draft_step(ctx, s, W, hid, st, tree)
            torch.cuda.synchronize()
            if s == 0:
                continue
            got = {n: v.cpu().numpy() for n, v in t.items()}
            base, kk = 1 + k + (s - 1) * k * k, k * k
            for b in range(B):
                sc, tok = got["pool_score"][b, base:base + kk], got["pool_token"][b, base:base + kk]
                assert tok.min() >= 0 and tok.max() < V
                bad = np.isnan(sc.reshape(k, k)).all(axis=1)
                assert np.array_equal(bad, np.isnan(lps[b]) | ((s == 1) & (b == 0) & (np.arange(k) == 3)))
                order = np.lexsort((np.arange(kk), tok, -_ordered(sc)))[:k]
                assert np.array_equal(got["beam_node"][b], base + order)
                assert np.array_equal(got["beam_parent_slot"][b], order // k)
                assert np.array_equal(got["beam_token"][b], tok[order])
        tree_np = {n: v.cpu().numpy() for n, v in tt.items()}
        for b in range(B):
            _check_tree(tree_np, got, 1 + k + (calls - 1) * k * k, m, b)
    finally:
        D.ddd_destroy(ctx)


@pytest.mark.parametrize("k,V", [(17, 128), (100, 3000), (128, 70001)])
def test_row_without_candidates(gpu, k, V):
    """A hidden row that holds no number has no logit above any bound: all k of its results are "no token" (-1), not what an
    earlier call left, and a draft call with such a row stays inside its beam and pool."""
    torch, D = gpu
    print(f"[case] wide_no_candidates k={k} V={V}", flush=True)
    H, bad = 128, 2
    rng = np.random.default_rng(k)
    W = _bits(torch, synth.make_lm_head(V, H, 0.2, 1))
    cfg = D.make_config(1, H, V, k, 4, 20, 0.0, 0)
    ctx = D.ddd_create(cfg)
    try:
        st, t = D.alloc_state(cfg)
        D.ddd_round_reset(ctx, st)
        for s in range(3):                                       # numbers in the first two calls: the scratch holds their keys
            hid = torch.from_numpy(rng.standard_normal((1 if s == 0 else k, H)).astype(np.float32)).cuda().to(torch.bfloat16)
            if s == 2:
                hid[bad] = float("nan")
            D.ddd_draft_step(ctx, s, W, hid, st)
        tok = torch.full((k, k), -7, dtype=torch.int32, device="cuda")
        lp, lse = torch.zeros(k, k, device="cuda"), torch.zeros(k, device="cuda")
        D.ddd_lmhead_topk(ctx, W, hid, k, None, tok, lp, lse)
        torch.cuda.synchronize()
        got, tok = {n: v.cpu().numpy()[0] for n, v in t.items() if n != "row_active"}, tok.cpu().numpy()
    finally:
        D.ddd_destroy(ctx)
    assert np.all(tok[bad] == -1)
    rest = np.delete(tok, bad, axis=0)
    assert rest.min() >= 0 and rest.max() < V
    base, kk = 1 + k + k * k, k * k
    assert np.array_equal(got["pool_token"][base:base + kk].reshape(k, k), tok)
    assert np.all(got["pool_depth"][base:base + kk] == 3)
    assert len(set(got["beam_node"])) == k and got["beam_node"].min() >= base and got["beam_node"].max() < base + kk
    assert np.array_equal(got["beam_parent_slot"], (got["beam_node"] - base) // k)


@pytest.mark.parametrize("k,calls", [(10, 3), (10, 6), (100, 2)])
def test_final_tree_of_a_pool_out_of_order(gpu, k, calls):
    """A pool in which nodes are their own or each other's parents (a state that no round leaves): the tree is built without
    those edges, as if the nodes had no parent in it."""
    torch, D = gpu
    print(f"[case] tree_out_of_order k={k} calls={calls}", flush=True)
    n, m = 1 + k + (calls - 1) * k * k, 20
    score = -np.arange(n, dtype=np.float32)                      # the first m nodes are the tree
    parent = np.zeros(n, np.int32)
    parent[0] = -1
    parent[3], parent[5], parent[6], parent[7] = 3, 6, 5, 9
    cfg = D.make_config(1, 128, 4000, k, calls, m, 0.0, 0)
    ctx = D.ddd_create(cfg)
    try:
        st, t = D.alloc_state(cfg)
        tree, tt = D.alloc_tree(cfg)
        t["pool_score"][0, :n].copy_(torch.from_numpy(score))
        t["pool_parent"][0, :n].copy_(torch.from_numpy(parent))
        t["n_nodes"].fill_(n)
        D.ddd_tree_finalize(ctx, st, tree)
        torch.cuda.synchronize()
        got = {x: v.cpu().numpy()[0] for x, v in tt.items()}
    finally:
        D.ddd_destroy(ctx)
    assert np.array_equal(got["sel_node"][:m], np.arange(1, m + 1))
    want = np.zeros(m + 1, np.int32)
    want[[0, 3, 5, 7]] = -1
    want[6] = 5
    assert np.array_equal(got["parent_idx"], want)
