"""The draft layer's weight streams with few rows: calls whose rows are all stopped, and gathers by sequence, at a size whose
attention reads the next weights ahead and at one whose does not."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,F", [(4096, 9984), (256, 384)])
@pytest.mark.parametrize("B,k", [(1, 10), (3, 5)])
def test_stopped_calls_leave_no_trace(H, F, B, k):
    """A call without active rows writes nothing and changes nothing that a later call reads; a call with some active writes those
    rows as a call with all of them does, bit for bit (a row's sums do not depend on its neighbours)."""
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device (an MI355X)")
    import paper_2409_00142_amd as D
    print(f"[case] few_rows H={H} F={F} B={B} k={k}", flush=True)
    V, L, R = 500, 40, B * k
    g = torch.Generator(device="cuda")
    g.manual_seed(H + R)

    def rnd(*shape, std=1.0, dtype=torch.bfloat16):
        return torch.empty(shape, dtype=dtype, device="cuda").normal_(0, std, generator=g)

    w = {"E": rnd(V, H), "Wfc": rnd(H, 2 * H, std=(2 * H) ** -0.5), "g1": 1 + 0.1 * rnd(H, dtype=torch.float32),
         "Wqkv": rnd(3 * H, H, std=H ** -0.5), "Wo": rnd(H, H, std=H ** -0.5), "g2": 1 + 0.1 * rnd(H, dtype=torch.float32),
         "Wgu": rnd(2 * F, H, std=H ** -0.5), "Wd": rnd(H, F, std=F ** -0.5)}
    p = {"K": rnd(B, L, H), "V": rnd(B, L, H), "f_root": rnd(B, H),
         "root_token": torch.randint(0, V, (B,), generator=g, device="cuda", dtype=torch.int32)}
    token = torch.randint(0, V, (3, B, k), generator=g, device="cuda", dtype=torch.int32)
    slot = torch.randint(0, k, (3, B, k), generator=g, device="cuda", dtype=torch.int32)
    cfg = D.make_config(B, H, V, k, 4, 60, 0.0, 0)
    body = D.ddd_body_create(D.ddd_body_config(B, k, H, F, V, 4, L))
    some = torch.arange(B, device="cuda") == 0
    try:
        D.ddd_body_bind(body, w, p)

        def call(step, on):
            st, t = D.alloc_state(cfg)
            if step:
                t["beam_token"].copy_(token[step - 1])
                t["beam_parent_slot"].copy_(slot[step - 1] if step > 1 else torch.zeros_like(slot[0]))
                t["row_active"].copy_(on.to(torch.uint8).repeat_interleave(k))
            out = torch.full((B if step == 0 else R, H), -7.0, dtype=torch.bfloat16, device="cuda")
            D.ddd_body_step(body, step, st, out)
            torch.cuda.synchronize()
            return out

        every, none = torch.ones(B, dtype=torch.bool, device="cuda"), torch.zeros(B, dtype=torch.bool, device="cuda")
        call(0, every)
        a1, a2 = call(1, every), call(2, every)
        assert bool((call(1, none) == -7.0).all()) and bool((call(2, none) == -7.0).all())
        assert torch.equal(call(2, every), a2)
        b2 = call(2, some)
        assert torch.equal(b2.view(B, k, H)[some], a2.view(B, k, H)[some])
        assert bool((b2.view(B, k, H)[~some] == -7.0).all())
        call(0, every)
        assert torch.equal(call(1, every), a1) and torch.equal(call(2, every), a2)
        assert bool(torch.isfinite(a2.float()).all())
    finally:
        D.ddd_body_destroy(body)


@pytest.mark.parametrize("N,K", [(4096, 11008), (12292, 8192), (260, 5248), (64, 4096)])
@pytest.mark.parametrize("R", [1, 10, 16])
def test_sums_run_along_k(N, K, R):
    """A product of several K ranges whose weight rows are all alike: every workgroup starts with a range of its own, and yet all
    outputs of an input row are the same bits."""
    import torch
    import paper_2409_00142_amd as D
    print(f"[case] few_rows sums N={N} K={K} R={R}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(N + K + R)
    row = torch.empty(K, device="cuda").normal_(0, K ** -0.5, generator=g).to(torch.bfloat16)
    W = row.expand(N, K).contiguous()
    x = torch.empty(R, K, device="cuda").normal_(0, 1, generator=g).to(torch.bfloat16)
    y = torch.zeros(R, N, device="cuda")
    body = D.ddd_body_create(D.ddd_body_config(1, 16, 1024, 128, 16, 4, 0))
    try:
        D.ddd_body_linear(body, W, N, K, x, R, y)
        torch.cuda.synchronize()
        assert torch.equal(y, y[:, :1].expand(R, N))
        exact = x.double() @ row.double()
        assert bool((y[:, 0].double() - exact).abs().max() < 1e-4)   # fp32 sums of K products of the size K^-1/2
    finally:
        D.ddd_body_destroy(body)


@pytest.mark.parametrize("N,K", [(4096, 8192), (516, 16384), (12, 24576)])   # two ranges; two launches, the second with one or two
@pytest.mark.parametrize("R", [1, 6, 7])
def test_input_rows_behind_the_whole_tile(N, K, R):
    """Weight rows whole 16 KB apart, on either side of the number of input rows up to which these are requested behind all of the first
    tile.  Against 64 bits, and twice with the same bits whatever the result held."""
    import torch
    import paper_2409_00142_amd as D
    print(f"[case] few_rows late N={N} K={K} R={R}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(N + K + R)
    W = torch.empty(N, K, device="cuda").normal_(0, K ** -0.5, generator=g).to(torch.bfloat16)
    x = torch.empty(R, K, device="cuda").normal_(0, 1, generator=g).to(torch.bfloat16)
    y = torch.full((R, N), -7.0, device="cuda")
    again = torch.full((R, N), -7.0, device="cuda")
    body = D.ddd_body_create(D.ddd_body_config(1, 16, 1024, 128, 16, 4, 0))
    try:
        D.ddd_body_linear(body, W, N, K, x, R, y)
        D.ddd_body_linear(body, W, N, K, x, R, again)
        torch.cuda.synchronize()
    finally:
        D.ddd_body_destroy(body)
    assert torch.equal(y, again)
    assert bool((y.double() - x.double() @ W.double().T).abs().max() < 1e-4)   # fp32 sums of K products of the size K^-1/2
