"""ddd_verify_sample's rows' sums have a short exponential for weights of 2^-1000 and more and a long one for the others: both
routes on rows that mix them, against the oracle."""
import numpy as np
import pytest

import synth
from oracle import ddd_oracle as O
from oracle.verify_sample import verify_sample

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [1021, 32000])
@pytest.mark.parametrize("spread", [2.0, 690.0, 800.0, 3.0e38])
def test_rows_of_short_and_long_weights(V, spread):
    """Logits N(0, 2^2), a third of them `spread` lower: 2^-995 of the row's mass, 2^-1154, or masked by the type's lowest value.  A
    decision closer to its threshold than 1e-10 of the row's weight (summation order in fp64: 1e-15) is not compared; the lowest
    uniform, 0, takes the first token that has weight at all."""
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device (an MI355X)")
    import paper_2409_00142_amd as D
    print(f"[case] sample_weights V={V} spread={spread}", flush=True)
    B, k, Dm, m = 4, 4, 4, 10
    rng = np.random.default_rng(V + int(min(spread, 1e6)))
    toks, pars = zip(*(synth.make_random_tree(m, m, k, V, Dm, seed=V + b) for b in range(B)))
    lg = (rng.standard_normal((B, m + 1, V)) * 2).astype(np.float32)
    lg = np.maximum(lg - np.float32(spread) * (rng.random((B, m + 1, V)) < 1 / 3), np.finfo(np.float32).min).astype(np.float32)
    for b in range(B):
        for c in range(1, m + 1):
            if rng.random() < 0.7:
                lg[b, pars[b][c], toks[b][c]] = 12.0
    ua, ub = rng.random((B, m + 1)), rng.random((B, m + 1))
    ub[1] = 0.0
    cfg = D.make_config(B, 128, V, k, Dm, m, 0.3)
    ctx = D.ddd_create(cfg)
    got = []
    try:
        tree, t = D.alloc_tree(cfg)
        t["tree_token"].copy_(torch.from_numpy(np.stack(toks)).view_as(t["tree_token"]))
        t["parent_idx"].copy_(torch.from_numpy(np.stack(pars)).view_as(t["parent_idx"]))
        t["n_sel"].fill_(m)
        x, a, u = torch.from_numpy(lg).cuda(), torch.from_numpy(ua).cuda(), torch.from_numpy(ub).cuda()
        torch.cuda.synchronize()
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
    for b in range(B):
        pos = np.zeros(m + 1, np.int32)
        for i in range(1, m + 1):
            pos[i] = pos[pars[b][i]] + 1
        tr = O.Tree(m=m, n_sel=m, sel_node=np.full(m, -1, np.int32), tree_token=toks[b], pos=pos, parent_idx=pars[b],
                    mask=np.zeros((m + 1, m + 1), np.uint8))
        mg = []
        alen, path, bonus = verify_sample(tr, lg[b], 1.0, ua[b], ub[b], Dm, margins=mg)
        if mg and min(mg) <= 1e-10 and b != 1:
            continue
        assert (int(got[0][0][b]), int(got[0][2][b])) == (alen, bonus)
        assert np.array_equal(got[0][1][b], path)
