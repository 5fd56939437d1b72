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
