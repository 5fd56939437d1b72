"""Tree attention whose heads are a little more than one step of eight waves per workgroup: up to sixteen chunks of 32 keys in one
pass, and workgroups of a head on one XCD."""
import math

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,nh,m,L", [(1, 32, 60, 1985), (1, 32, 60, 1984), (1, 32, 60, 1983), (1, 32, 63, 2016), (1, 32, 64, 960),
                                      (1, 30, 60, 2047), (1, 32, 2, 2017), (1, 32, 1, 2040), (4, 32, 31, 480), (4, 32, 60, 930),
                                      (3, 40, 20, 900), (1, 32, 127, 900), (1, 128, 60, 992), (2, 16, 127, 300), (5, 16, 127, 700)])
def test_heads_of_one_pass(B, nh, m, L):
    """Against a softmax in 64 bits, trees of different sizes, and twice the same bits.  Tolerance as in the kernel's other tests: the
    weights' two bf16 halves leave 2^-17 and the fast exponential and fp32 sums less, of order-one values: 1e-4."""
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device (an MI355X)")
    import paper_2409_00142_amd as D
    print(f"[case] attention_pass B={B} heads={nh} m={m} L={L}", flush=True)
    T, Tp = m + 1, (m + 32) // 32 * 32
    g = torch.Generator(device="cuda")
    g.manual_seed(L * 131 + m)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g).to(torch.bfloat16)
    q, kt, vt, kp, vp = rnd(B, T, nh, 128), rnd(B, T, nh, 128), rnd(B, T, nh, 128), rnd(B, L, nh, 128), rnd(B, L, nh, 128)
    vtt = torch.zeros(B, nh, 128, Tp, device="cuda", dtype=torch.bfloat16)
    vtt[..., :T] = vt.permute(0, 2, 3, 1)
    mask = torch.zeros(B, T, T, dtype=torch.uint8)
    n_sel = [m - (b * m) // max(B, 2) for b in range(B)]
    for b in range(B):
        mask[b, 0, 0] = 1
        for i in range(1, n_sel[b] + 1):
            mask[b, i] = mask[b, int(torch.randint(0, i, (1,)))]
            mask[b, i, i] = 1
    ctx = D.ddd_create(D.make_config(B, 256, 1000, 4, 4, m, 0.3))
    try:
        tree, t = D.alloc_tree(D.make_config(B, 256, 1000, 4, 4, m, 0.3))
        t["mask"].copy_(mask.view_as(t["mask"]))
        t["n_sel"].copy_(torch.tensor(n_sel, dtype=torch.int32))
        n = B * nh * ((L + 31) // 32) * 4096
        kpk, vpk = (torch.full((n,), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2))
        D.ddd_kv_pack(ctx, kp, vp, L, nh, kpk, vpk)
        ws = torch.full((D.ddd_tree_attention_workspace(ctx, nh, L) // 4,), float("nan"), device="cuda")
        outs = [torch.full((B, T, nh, 128), float("nan"), device="cuda") for _ in range(2)]
        for out in outs:
            D.ddd_tree_attention(ctx, tree, q, kt, vtt, kpk, vpk, L, nh, ws, out)
        torch.cuda.synchronize()
    finally:
        D.ddd_destroy(ctx)
    assert torch.equal(outs[0], outs[1])
    for b in range(B):
        s = n_sel[b] + 1
        K = torch.cat([kp[b], kt[b, :s]]).double().permute(1, 0, 2).contiguous()
        V = torch.cat([vp[b], vt[b, :s]]).double().permute(1, 0, 2).contiguous()
        score = torch.matmul(q[b, :s].double().permute(1, 0, 2).contiguous(), K.transpose(1, 2).contiguous()) / math.sqrt(128.0)
        seen = torch.ones(s, L + s, dtype=torch.bool, device="cuda")
        seen[:, L:] = mask[b, :s, :s].cuda() != 0
        want = torch.matmul(torch.softmax(score.masked_fill(~seen, -math.inf), -1), V).permute(1, 0, 2)
        assert float((outs[0][b, :s].double() - want).abs().max()) <= 1e-4
        assert bool((outs[0][b, s:] == 0).all())


@pytest.mark.parametrize("nh,m,L", [(24, 60, 2496), (16, 60, 4032), (8, 127, 3968), (4, 60, 16320)])
def test_workspace_of_a_longer_prompt(nh, m, L):
    """The workspace never shrinks as the prompt grows, also where the longer prompt takes its chunks in one pass."""
    import paper_2409_00142_amd as D
    ctx = D.ddd_create(D.make_config(1, 256, 1000, 4, 4, m, 0.3))
    try:
        assert D.ddd_tree_attention_workspace(ctx, nh, L) <= D.ddd_tree_attention_workspace(ctx, nh, L + 1)
    finally:
        D.ddd_destroy(ctx)
