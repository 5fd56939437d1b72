"""ddd_verify_sample above 128 MiB of logits: a launch decides at the roots, and only rows below the accepted child are summed up.
Against the oracle and against the walk that makes its own sums (another stream): roots that reject all their children or the first
few, absent trees, small trees with their leaves ahead, and a scratch that other decisions have used."""
import numpy as np
import pytest

import synth
from oracle import ddd_oracle as O
from oracle.verify_sample import verify_sample

pytestmark = pytest.mark.gpu
MIN_MARGIN = 1e-10     # relative distance of a decision from its threshold below which fp64 summation order could matter
MB = 1 << 20


# three, seven and eight parts of a row; two to four chunks a block; m from 32 to 128
@pytest.mark.parametrize("B,V,m,depth", [(33, 10000, 101, 6), (10, 28672, 120, 3), (10, 32000, 128, 6), (9, 32769, 127, 4), (16, 65537, 32, 6),
                                         (10, 98305, 35, 3), (8, 131071, 33, 6)])
def test_only_rows_below_the_accepted_child(B, V, m, depth):
    import torch
    import paper_2409_00142_amd as D
    print(f"[case] verify_sample root B={B} V={V} m={m} depth={depth}", flush=True)
    assert 128 * MB < B * (m + 1) * V * 4 <= 288 * MB or B * (m + 1) <= 1024
    k = 10
    rng = np.random.default_rng(V + m)
    n_sels = ([m, m, m, m, m, 0, 1, min(m, 10 * MB // (B * V * 4))] + [m] * B)[:B]
    toks, pars = zip(*(synth.make_random_tree(m, n, k, V, depth, seed=3 * V + b) for b, n in enumerate(n_sels)))
    g = torch.Generator(device="cuda")
    g.manual_seed(V + m)
    xd = torch.empty(B, m + 1, V, device="cuda").normal_(0, 2, generator=g)
    x = xd.cpu().numpy()
    cfg = D.make_config(B, 128, V, k, depth, m, 0.3)
    ctx = D.ddd_create(cfg)
    try:
        tree, t = D.alloc_tree(cfg)
        t["tree_token"].copy_(torch.from_numpy(np.stack(toks)).view_as(t["tree_token"]))
        t["parent_idx"].copy_(torch.from_numpy(np.stack(pars)).view_as(t["parent_idx"]))
        t["n_sel"].copy_(torch.tensor(n_sels, dtype=torch.int32))
        lens = []
        for call in range(4):
            ua, ub = np.zeros((B, m + 1)), rng.random((B, m + 1))          # every first child is accepted ...
            for b in range(B):
                kids = [i for i in range(1, n_sels[b] + 1) if pars[b][i] == 0]
                refuse = (0, len(kids), 1, 2)[(b + call) % 4]              # ... but for so many of the root's
                ua[b, kids[:refuse]] = 1.0 - 1e-9
            ua[0] = rng.random(m + 1)
            a, u = torch.from_numpy(ua).cuda(), torch.from_numpy(ub).cuda()
            outs = []
            for stream in (torch.cuda.current_stream(), torch.cuda.Stream()):
                stream.wait_stream(torch.cuda.current_stream())
                out = [torch.full((B,), -7, dtype=torch.int32, device="cuda"),
                       torch.full((B, depth + 1), -7, dtype=torch.int32, device="cuda"),
                       torch.full((B,), -7, dtype=torch.int32, device="cuda")]
                torch.cuda.synchronize()
                D.ddd_verify_sample(ctx, tree, xd, 0.8, a, u, *out, stream=stream.cuda_stream)
                torch.cuda.synchronize()
                outs.append([o.cpu().numpy() for o in out])
            for b in range(B):
                pos = np.zeros(m + 1, np.int32)
                for i in range(1, n_sels[b] + 1):
                    pos[i] = pos[pars[b][i]] + 1
                tr = O.Tree(m=m, n_sel=n_sels[b], sel_node=np.full(m, -1, np.int32), tree_token=toks[b], pos=pos,
                            parent_idx=pars[b], mask=np.zeros((m + 1, m + 1), np.uint8))
                mg = []
                o_len, o_path, o_bonus = verify_sample(tr, x[b], float(np.float32(0.8)), ua[b], ub[b], depth, margins=mg)
                if mg and min(mg) <= MIN_MARGIN:
                    continue
                lens.append(o_len)
                for alen, path, bonus in outs:
                    assert (int(alen[b]), int(bonus[b])) == (o_len, o_bonus), (call, b)
                    assert np.array_equal(path[b], o_path), (call, b)
        assert 0 in lens and max(lens) >= 2
    finally:
        D.ddd_destroy(ctx)
