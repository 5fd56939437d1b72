"""ddd_verify_sample where the walk ends at a leaf.  Small calls, and small trees of larger ones, have the leaves' sums made ahead;
elsewhere the workgroups of the walk make that row's sums, one part of the row each.  Against the oracle on either side of those
limits: rows of one to eight parts and of one to five chunks a block, whole parts without weight, bonus draws that rounding leaves
without a token, all statistics bound, several calls of one context."""
import numpy as np
import pytest

import synth
from oracle import ddd_oracle as O
from oracle.verify_sample import verify_sample

pytestmark = pytest.mark.gpu
MIN_MARGIN = 1e-10     # relative distance of a decision from its threshold below which fp64 summation order could matter
MB = 1 << 20


def _leaves_ahead(B, V, m):
    """Rows up to which a tree's leaves are summed ahead."""
    total = B * (m + 1) * V * 4
    return m + 1 if total <= 24 * MB or (B >= 24 and total <= 38 * MB) or (m <= 32 and total <= 64 * MB) else 10 * MB // (B * V * 4)


@pytest.mark.parametrize("B,V,m,ahead", [
    (6, 3, 2, True), (6, 300, 20, True), (6, 4096, 60, True), (6, 98304, 12, True), (24, 5001, 70, True),   # every leaf ahead
    (13, 4096, 128, False), (13, 4097, 128, False), (16, 10000, 60, False),                  # one, two and three parts
    (8, 28672, 48, False), (8, 28673, 48, False), (8, 32000, 65, False),                     # seven and eight
    (8, 32769, 40, False), (8, 65537, 33, False), (8, 98305, 33, False), (8, 131071, 33, False)])   # two, three, four chunks a block, five parts
def test_walk_ends_at_a_leaf(B, V, m, ahead):
    import torch
    import paper_2409_00142_amd as D
    print(f"[case] verify_sample leaf B={B} V={V} m={m}", flush=True)
    limit = _leaves_ahead(B, V, m)
    assert (limit == m + 1) == ahead
    k, Dm = min(4, V), 6
    rng = np.random.default_rng(V + m)
    n_sels = [m, m, max(1, m // 2), 1, 0, m] + [min(max(limit - 1, 0), m), min(limit, m)] + [m] * B
    n_sels = n_sels[:B]
    toks, pars = zip(*(synth.make_random_tree(m, n, k, V, Dm, seed=7 * V + b) for b, n in enumerate(n_sels)))
    lg = (rng.standard_normal((B, m + 1, V)) * 2).astype(np.float32)
    leaf = [[i not in set(pars[b][1:n_sels[b] + 1].tolist()) for i in range(m + 1)] for b in range(B)]
    ua, ub = np.zeros((B, m + 1)), rng.random((B, m + 1))     # every first child is accepted ...
    ua[5] = rng.random(m + 1)                                 # ... but in one sequence
    ub[0] = 1.0 + 1e-9                                        # no prefix gets there: the last token that has weight
    cfg = D.make_config(B, 128, V, k, Dm, m, 0.3)
    ctx = D.ddd_create(cfg)
    try:
        tree, t = D.alloc_tree(cfg)
        t["tree_token"].copy_(torch.from_numpy(np.stack(toks)).view_as(t["tree_token"]))
        t["parent_idx"].copy_(torch.from_numpy(np.stack(pars)).view_as(t["parent_idx"]))
        t["n_sel"].copy_(torch.tensor(n_sels, dtype=torch.int32))
        hists = {n: torch.zeros(32, dtype=torch.int64, device="cuda") for n in ("depth_hist", "accept_hist", "batch_depth_hist")}
        n_rounds = torch.zeros(1, dtype=torch.int64, device="cuda")
        steps = rng.integers(1, 20, B).astype(np.int32)
        steps_dev = torch.from_numpy(steps).cuda()            # outlives the binding
        D.ddd_stats_bind(ctx, rounds=n_rounds, steps=steps_dev, **hists)
        a, u = torch.from_numpy(ua).cuda(), torch.from_numpy(ub).cuda()
        seen = np.zeros(32, np.int64)
        on_demand = 0
        for call in range(3):
            x = np.roll(lg, call, axis=2)
            for i in range(m + 1):                            # a leaf's row: without weight up to the middle, or with a mask there
                if leaf[1][i]:
                    x[1, i, : V // 2] = -np.inf
                if leaf[2][i]:
                    x[2, i, V // 2:] = np.finfo(np.float32).min
            xd = torch.from_numpy(x).cuda()
            out = [torch.full((B,), -7, dtype=torch.int32, device="cuda"),
                   torch.full((B, Dm + 1), -7, dtype=torch.int32, device="cuda"),
                   torch.full((B,), -7, dtype=torch.int32, device="cuda")]
            D.ddd_verify_sample(ctx, tree, xd, 0.8, a, u, *out)
            torch.cuda.synchronize()
            alen, path, bonus = (o.cpu().numpy() for o in out)
            seen += np.bincount(alen, minlength=32)
            for b in range(B):
                pos = np.zeros(m + 1, np.int32)
                for i in range(1, n_sels[b] + 1):
                    pos[i] = pos[pars[b][i]] + 1
                tr = O.Tree(m=m, n_sel=n_sels[b], sel_node=np.full(m, -1, np.int32), tree_token=toks[b], pos=pos,
                            parent_idx=pars[b], mask=np.zeros((m + 1, m + 1), np.uint8))
                mg = []
                o_len, o_path, o_bonus = verify_sample(tr, x[b], float(np.float32(0.8)), ua[b], ub[b], Dm, margins=mg)
                on_demand += n_sels[b] + 1 > limit and leaf[b][o_path[o_len]]
                if b == 0:
                    mg.remove(0.0)                            # the draw without a token, which is meant
                if mg and min(mg) <= MIN_MARGIN:
                    continue
                assert (int(alen[b]), int(bonus[b])) == (o_len, o_bonus), (call, b)
                assert np.array_equal(path[b], o_path), (call, b)
        assert (on_demand == 0) if ahead else (on_demand >= 2 * 3)
        assert int(n_rounds.item()) == 3 and np.array_equal(hists["accept_hist"].cpu().numpy(), seen)
        assert np.array_equal(hists["depth_hist"].cpu().numpy(), 3 * np.bincount(steps, minlength=32))
        assert np.array_equal(hists["batch_depth_hist"].cpu().numpy(), 3 * np.bincount([steps.max()], minlength=32))
    finally:
        D.ddd_destroy(ctx)
