"""ddd_verify_sample has two routes: the sums of all rows first (small batches, the context's first stream) and a walk
that makes its own (any other stream, captured calls, larger batches).  Both against each other and the oracle."""
import numpy as np
import pytest

import synth
from oracle import ddd_oracle as O
from oracle.verify_sample import verify_sample

pytestmark = pytest.mark.gpu
MIN_MARGIN = 1e-10     # relative distance of a decision from its threshold below which fp64 summation order could matter


@pytest.mark.parametrize("V", [5, 255, 257, 1024, 4096, 4097, 8193, 32768, 32769, 65537, 98305, 131071, 131076])
@pytest.mark.parametrize("T", [1.0, 1e-3, 30.0])
def test_both_routes_agree(V, T):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device (an MI355X)")
    import paper_2409_00142_amd as D
    # up to 4096 tokens a row is one part of eight, from 4097 two, from 32769 a part is twice as long (five of them)
    print(f"[case] verify_sample routes V={V} T={T}", flush=True)
    B, k, Dm, m = 3, 4, 5, 12
    rng = np.random.default_rng(V)
    T32 = float(np.float32(T))
    toks, pars = zip(*(synth.make_random_tree(m, n, k, V, Dm, seed=V + b) for b, n in enumerate((m, 7, 0))))
    lg = (rng.standard_normal((B, m + 1, V)) * 2).astype(np.float32)
    for b in range(B):
        for c in range(1, m + 1):
            if pars[b][c] >= 0 and rng.random() < 0.7:
                lg[b, pars[b][c], toks[b][c]] += 9.0
    lg[0, 1, V // 2:] = -np.inf                                # most of a row without weight
    lg[1, 0, : V // 2] = np.finfo(np.float32).min              # a mask of the type's lowest value
    ua, ub = rng.random((B, m + 1)), rng.random((B, m + 1))
    cfg = D.make_config(B, 128, V, k, Dm, m, 0.3)
    ctx = D.ddd_create(cfg)
    got = []
    try:
        tree, t = D.alloc_tree(cfg)
        t["tree_token"].copy_(torch.from_numpy(np.stack(toks)).view_as(t["tree_token"]))
        t["parent_idx"].copy_(torch.from_numpy(np.stack(pars)).view_as(t["parent_idx"]))
        t["n_sel"].copy_(torch.tensor([m, 7, 0], dtype=torch.int32))
        x, a, u = torch.from_numpy(lg).cuda(), torch.from_numpy(ua).cuda(), torch.from_numpy(ub).cuda()
        torch.cuda.synchronize()
        other = torch.cuda.Stream()
        for stream in (torch.cuda.current_stream(), other, torch.cuda.current_stream()):
            out = [torch.full((B,), -7, dtype=torch.int32, device="cuda"),
                   torch.full((B, Dm + 1), -7, dtype=torch.int32, device="cuda"),
                   torch.full((B,), -7, dtype=torch.int32, device="cuda")]
            torch.cuda.synchronize()
            D.ddd_verify_sample(ctx, tree, x, T, a, u, *out, stream=stream.cuda_stream)
            torch.cuda.synchronize()
            got.append([o.cpu().numpy() for o in out])
    finally:
        D.ddd_destroy(ctx)
    for other_route in got[1:]:
        for p, q in zip(got[0], other_route):
            assert np.array_equal(p, q)
    for b in range(B):
        n_sel = (m, 7, 0)[b]
        pos = np.zeros(m + 1, np.int32)
        for i in range(1, n_sel + 1):
            pos[i] = pos[pars[b][i]] + 1
        tr = O.Tree(m=m, n_sel=n_sel, sel_node=np.full(m, -1, np.int32), tree_token=toks[b], pos=pos, parent_idx=pars[b],
                    mask=np.zeros((m + 1, m + 1), np.uint8))
        mg = []
        alen, path, bonus = verify_sample(tr, lg[b], T32, ua[b], ub[b], Dm, margins=mg)
        if mg and min(mg) <= MIN_MARGIN:
            continue
        assert (int(got[0][0][b]), int(got[0][2][b])) == (alen, bonus)
        assert np.array_equal(got[0][1][b], path)


@pytest.mark.parametrize("V", [2, 3, 4, 6, 7, 1021, 1022, 1023, 32765, 32766, 32767, 65535])
def test_rows_that_end_anywhere(V):
    """Rows whose last 16-byte piece is whole or straddles the end, and rows shorter than one: nearly all weight on the last four
    tokens, so the bonus tells whether each of them counted once, on both routes and against the oracle.  The logits fill their
    allocation to its last element."""
    import torch
    import paper_2409_00142_amd as D
    print(f"[case] verify_sample row ends V={V}", flush=True)
    B, k, Dm, m = 16, 2, 3, 4
    rng = np.random.default_rng(V)
    lg = rng.standard_normal((B, m + 1, V)).astype(np.float32)
    lg[..., max(V - 4, 0):] += 14.0
    ua, ub = np.full((B, m + 1), 0.999999), np.tile(((np.arange(B) + 0.5) / B)[:, None], (1, m + 1))
    cfg = D.make_config(B, 128, V, k, Dm, m, 0.3)
    ctx = D.ddd_create(cfg)
    got = []
    try:
        tree, t = D.alloc_tree(cfg)
        t["n_sel"].zero_()
        x, a, u = torch.from_numpy(lg).cuda(), torch.from_numpy(ua).cuda(), torch.from_numpy(ub).cuda()
        other = torch.cuda.Stream()
        for stream in (torch.cuda.current_stream(), other):
            out = [torch.full((B,), -7, dtype=torch.int32, device="cuda"),
                   torch.full((B, Dm + 1), -7, dtype=torch.int32, device="cuda"),
                   torch.full((B,), -7, dtype=torch.int32, device="cuda")]
            torch.cuda.synchronize()
            D.ddd_verify_sample(ctx, tree, x, 1.0, a, u, *out, stream=stream.cuda_stream)
            torch.cuda.synchronize()
            got.append([o.cpu().numpy() for o in out])
    finally:
        D.ddd_destroy(ctx)
    for p, q in zip(*got):
        assert np.array_equal(p, q)
    none = np.full(m + 1, -1, np.int32)
    for b in range(B):
        tr = O.Tree(m=m, n_sel=0, sel_node=none[1:], tree_token=none, pos=np.zeros(m + 1, np.int32), parent_idx=none,
                    mask=np.zeros((m + 1, m + 1), np.uint8))
        mg = []
        alen, _, bonus = verify_sample(tr, lg[b], 1.0, ua[b], ub[b], Dm, margins=mg)
        if mg and min(mg) <= MIN_MARGIN:
            continue
        assert (int(got[0][0][b]), int(got[0][2][b])) == (alen, bonus)
