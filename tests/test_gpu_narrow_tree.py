"""Final tree of narrow pools (k <= 16) at the sizes where the selection changes its form, and the accept walk over it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _ordered(scores):
    """fp32 scores as integers in the order of the rerank keys (both zeros alike, a positive NaN above +inf)."""
    u = (np.ascontiguousarray(scores, dtype=np.float32) + np.float32(0.0)).view(np.uint32)
    return np.where(u >> 31, ~u, u | np.uint32(0x80000000)).astype(np.int64)


@pytest.mark.parametrize("scores", ["falling", "ties", "equal", "special"])
@pytest.mark.parametrize("k,calls,m,n", [(4, 3, 60, 1), (4, 3, 60, 2), (4, 3, 1, 37), (8, 9, 128, 129), (8, 9, 128, 130), (8, 9, 60, 257),
                                         (8, 9, 60, 258), (8, 9, 127, 513), (8, 9, 63, 514), (10, 10, 64, 769), (10, 10, 65, 770),
                                         (10, 10, 60, 911), (16, 9, 60, 1025), (16, 9, 60, 1026), (16, 9, 128, 2049), (16, 9, 128, 2050)])
def test_final_tree_and_accept_walk(k, calls, m, n, scores):
    """Against a sort of the pool's nodes 1 .. n - 1 by (score desc, node id asc), the ancestor closure and a walk by hand; all
    whole numbers."""
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device (an MI355X)")
    import paper_2409_00142_amd as D
    print(f"[case] narrow_tree k={k} calls={calls} m={m} n={n} {scores}", flush=True)
    B, rng = 2, np.random.default_rng(n * 7 + m)
    cfg = D.make_config(B, 128, 4000, k, calls, m, 0.0, 0)
    nmax = D.ddd_pool_capacity(cfg)
    assert n <= nmax
    parent = np.maximum(np.minimum((np.arange(nmax) - 1) // k, np.arange(nmax) - 1), 0).astype(np.int32)
    parent[0] = -1
    depth = np.zeros(nmax, np.int32)
    for i in range(1, nmax):
        depth[i] = depth[parent[i]] + 1
    step = rng.gamma(2.0, 0.5, (B, nmax)).astype(np.float32)
    if scores == "ties":
        step = np.round(step)
    score = np.zeros((B, nmax), np.float32)
    for i in range(1, nmax):
        score[:, i] = score[:, parent[i]] - (0 if scores == "equal" else step[:, i])
    if scores == "special":
        score[:, 1:nmax:3] = np.nan
        score[:, 2:nmax:5] = -np.inf
        score[1, 4:nmax:7] = np.inf
    tok = rng.integers(0, 40, (B, nmax)).astype(np.int32)
    target = rng.integers(0, 40, (B, m + 1)).astype(np.int32)
    ctx = D.ddd_create(cfg)
    try:
        st, t = D.alloc_state(cfg)
        tree, tt = D.alloc_tree(cfg)
        for name, v in (("pool_score", score), ("pool_token", tok), ("pool_parent", np.tile(parent, (B, 1))),
                        ("pool_depth", np.tile(depth, (B, 1)))):
            t[name].copy_(torch.from_numpy(v))
        t["n_nodes"].fill_(n)
        D.ddd_tree_finalize(ctx, st, tree)
        torch.cuda.synchronize()
        got = {x: v.cpu().numpy() for x, v in tt.items()}
        for b in range(B):                                       # the target follows some child of half of the nodes
            for i in range(got["n_sel"][b] + 1):
                kids = np.flatnonzero(got["parent_idx"][b] == i)
                if len(kids) and rng.random() < 0.7:
                    target[b, i] = got["tree_token"][b][rng.choice(kids)]
        acc = [torch.full((B,), -7, dtype=torch.int32, device="cuda"), torch.full((B, calls + 1), -7, dtype=torch.int32, device="cuda"),
               torch.full((B,), -7, dtype=torch.int32, device="cuda")]
        D.ddd_verify_accept(ctx, tree, torch.from_numpy(target).cuda(), *acc)
        torch.cuda.synchronize()
        acc = [x.cpu().numpy() for x in acc]
    finally:
        D.ddd_destroy(ctx)
    for b in range(B):
        best = np.sort(np.lexsort((np.arange(n - 1), -_ordered(score[b, 1:n])))[:m] + 1)
        s = len(best)
        assert got["n_sel"][b] == s
        assert np.array_equal(got["sel_node"][b], np.concatenate([best, np.full(m - s, -1)]))
        index = {0: 0, **{int(v): i + 1 for i, v in enumerate(best)}}
        par = np.array([-1] + [index.get(int(parent[v]), -1) for v in best] + [-1] * (m - s))
        assert np.array_equal(got["parent_idx"][b], par)
        assert np.array_equal(got["tree_token"][b], np.concatenate([[tok[b, 0]], tok[b, best], np.full(m - s, -1)]))
        assert np.array_equal(got["pos"][b], np.concatenate([[depth[0]], depth[best], np.zeros(m - s)]))
        mask = np.zeros((m + 1, m + 1), np.uint8)
        for i in range(s + 1):
            c = i
            while c >= 0:
                mask[i, c] = 1
                c = par[c]
        assert np.array_equal(got["mask"][b], mask)
        path = [0]
        while len(path) <= calls:
            kids = [c for c in range(1, s + 1) if par[c] == path[-1] and got["tree_token"][b][c] == target[b, path[-1]]]
            if not kids:
                break
            path.append(kids[0])
        assert acc[0][b] == len(path) - 1 and acc[2][b] == target[b, path[-1]]
        assert np.array_equal(acc[1][b], np.array(path + [-1] * (calls + 1 - len(path))))
