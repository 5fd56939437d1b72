"""GPU tests of the batched (MFMA GEMM) path's own branches: how rows are laid out, listed and handed on."""
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


def _lmhead(torch, D, ctx, W, hid, R, k, V, row_active=None, debug=False):
    tok = torch.full((R, k), -7, dtype=torch.int32, device="cuda")
    lp = torch.zeros(R, k, device="cuda")
    lse = torch.zeros(R, device="cuda")
    dbg = torch.zeros(R, V, device="cuda") if debug else None
    D.ddd_lmhead_topk(ctx, W, hid, R, row_active, tok, lp, lse, dbg)
    torch.cuda.synchronize()
    return tok.cpu().numpy(), lp.cpu().numpy(), lse.cpu().numpy(), None if dbg is None else dbg.cpu().numpy()


@pytest.mark.parametrize("equal", [False, True], ids=["random", "all_equal"])
@pytest.mark.parametrize("V", [16385, 16386, 16387, 16388, 16447])
def test_logits_pitch_of_any_vocabulary(gpu, V, equal):
    """The context's own logits have a padded row pitch, a debug buffer the pitch V: the same results, bit for bit, for
    every remainder of V.  Equal logits (more than 256 groups at the threshold) take the scan of the whole row, which
    reads the padding's pieces too: the winners are the k lowest tokens."""
    torch, D = gpu
    print(f"[case] logits_pitch V={V} equal={equal}", flush=True)
    B, k, H = 7, 5, 256
    rng = np.random.default_rng(V)
    Wb = synth.make_lm_head(V, H, 0.2, V)
    if equal:
        Wb[:] = Wb[0]
    W = torch.from_numpy(Wb.view(np.int16)).cuda().view(torch.bfloat16)
    hid = torch.from_numpy(rng.standard_normal((B * k, H)).astype(np.float32)).cuda().to(torch.bfloat16)
    ctx = D.ddd_create(D.make_config(B, H, V, k, 3, 10, 0.3))
    try:
        a = _lmhead(torch, D, ctx, W, hid, B * k, k, V)
        b = _lmhead(torch, D, ctx, W, hid, B * k, k, V, debug=True)
    finally:
        D.ddd_destroy(ctx)
    for x, y in zip(a[:3], b[:3]):
        assert np.array_equal(x, y)
    want = np.argsort(-b[3], axis=1, kind="stable")[:, :k]     # ties: the lower token first
    assert np.array_equal(a[0], want)
    assert np.all(a[0] < V)


@pytest.mark.parametrize("N,K", [(4, 256), (128, 2048), (1156, 2048), (4096, 512), (516, 11008)])
@pytest.mark.parametrize("R", [17, 32, 33, 64, 65, 321, 640])
def test_split_linear(gpu, N, K, R):
    """ddd_body_linear on the MFMA path where few row tiles of W make it split K (1 to 8 ranges, uneven where the k tiles
    do not divide), one block of rows more or less than a tile: against the product in 64 bits, and twice the same bits.

    Tolerance: products of bf16 numbers are exact in fp32, and K sums of terms of size K^-0.5 round with relative error
    2^-24 each: sqrt(K) * 2^-24 times a few, below 1e-5 for K <= 11008; 1e-4 leaves room for the largest of R * N."""
    torch, D = gpu
    print(f"[case] split_linear N={N} K={K} R={R}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(N * 31 + K * 7 + R)
    W = torch.empty(N, K, dtype=torch.bfloat16, device="cuda").normal_(0, K ** -0.5, generator=g)
    x = torch.empty(R, K, dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    want = x.double() @ W.double().T.contiguous()
    body = D.ddd_body_create(D.ddd_body_config((R + 4) // 5, 5, 256, 256, 10, 2, 0))
    try:
        y = [torch.full((R, N), float("nan"), device="cuda") for _ in range(2)]
        for t in y:
            D.ddd_body_linear(body, W, N, K, x, R, t)
        acc = y[0].clone()
        D.ddd_body_linear(body, W, N, K, x, R, acc, accumulate=True)
        torch.cuda.synchronize()
    finally:
        D.ddd_body_destroy(body)
    assert torch.equal(y[0], y[1])
    assert float((y[0].double() - want).abs().max()) <= 1e-4
    assert float((acc.double() - 2 * want).abs().max()) <= 2e-4
