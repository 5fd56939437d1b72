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
def test_linear_of_any_rows(gpu, N, K, R):
    """ddd_body_linear on the MFMA path, one block of rows more or less than a tile: against the product in 64 bits, and twice
    the same bits.

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


def test_linears_on_two_streams(gpu):
    """ddd_body_linear keeps nothing in the body: calls of one body on two streams may overlap.  Tolerance as above."""
    torch, D = gpu
    print("[case] linears_on_two_streams", flush=True)
    N, K, R = 1024, 8192, 200
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    W = [torch.empty(N, K, dtype=torch.bfloat16, device="cuda").normal_(0, K ** -0.5, generator=g) for _ in range(2)]
    x = [torch.empty(R, K, dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g) for _ in range(2)]
    y = [[torch.full((R, N), float("nan"), device="cuda") for _ in range(20)] for _ in range(2)]
    body = D.ddd_body_create(D.ddd_body_config(50, 4, 256, 256, 10, 2, 0))
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    try:
        for i in range(20):
            for q in range(2):
                D.ddd_body_linear(body, W[q], N, K, x[q], R, y[q][i], stream=streams[q].cuda_stream)
        torch.cuda.synchronize()
    finally:
        D.ddd_body_destroy(body)
    for q in range(2):
        want = x[q].double() @ W[q].double().T.contiguous()
        for t in y[q]:
            assert float((t.double() - want).abs().max()) <= 1e-4


@pytest.mark.parametrize("L", [0, 5, 31, 32, 33, 64, 250, 257, 545, 1024, 1100])
@pytest.mark.parametrize("k", [3, 10, 16])
def test_batched_attention_of_any_prompt_length(gpu, L, k):
    """Draft layer, several sequences per call (batched attention: the prompt on the matrix cores from 32 positions on,
    whole steps of 32 keys or not; one too long for that: one workgroup per row and head) against the same sequences one at a
    time (at most 16 rows: the weight streams).  One sequence stops before the third call.

    Tolerance: both sides round at the same five points of a call, what lies between them is summed in another order,
    and a rounding that falls the other way moves a term by one bf16 ulp (2^-8): 2^-5 of the row's rms, as against the oracle."""
    print(f"[case] batched_attention L={L} k={k}", flush=True)
    _batch_against_single(gpu, 7, k, 256, 384, L, range(7), 1000 * k + L)


# Row counts around the blocks of 32 rows and the column tiles, few rows of W for 256 workgroups: K = 11008 (172 k tiles) in
# eight uneven ranges, 2816 in six or eight, 2048 in six or eight, 1408 in five, 1024 in two or four, 512 in one or two, 256 in
# one.  H = 4096 with 640 rows: tiles of 192 rows of W, whole and split.
@pytest.mark.parametrize("B,k,H,F", [(6, 3, 256, 11008), (8, 4, 256, 2944), (11, 3, 1024, 1408), (13, 5, 256, 11008), (43, 3, 512, 1024),
                                     (65, 5, 256, 11008), (64, 10, 1024, 2816), (64, 10, 4096, 1408)])
def test_split_products_of_the_layer(gpu, B, k, H, F):
    """Draft layer with more than 16 rows: partial sums of K ranges, added up by the norms, the attention and the last launch,
    against the same sequences one at a time (at most 16 rows: whole sums in the weight streams).  Tolerance as above."""
    print(f"[case] split_products B={B} k={k} H={H} F={F}", flush=True)
    _batch_against_single(gpu, B, k, H, F, 33, sorted({0, 2, B // 2, B - 1}), B + F)


# More workgroups than CUs: eight waves each; the sequences alone have sixteen.
@pytest.mark.parametrize("B,k,L", [(7, 20, 300), (7, 20, 513), (9, 16, 1100)])
def test_long_prompts_row_by_row(gpu, B, k, L):
    """Draft layer with one workgroup per row and head and more keys than a pass holds, in a batch and alone.  Tolerance as
    above."""
    print(f"[case] long_prompts_row_by_row B={B} k={k} L={L}", flush=True)
    _batch_against_single(gpu, B, k, 256, 384, L, [0, 2, B - 1], L)


def _batch_against_single(gpu, B, k, H, F, L, check, seed):
    torch, D = gpu
    V, calls = 300, 4
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def normal(*shape, std=1.0, dtype=torch.bfloat16):
        return torch.empty(shape, dtype=dtype, device="cuda").normal_(0, std, generator=g)

    w = {"E": normal(V, H), "Wfc": normal(H, 2 * H, std=(2 * H) ** -0.5), "g1": normal(H, dtype=torch.float32),
         "Wqkv": normal(3 * H, H, std=H ** -0.5), "Wo": normal(H, H, std=H ** -0.5), "g2": normal(H, dtype=torch.float32),
         "Wgu": normal(2 * F, H, std=H ** -0.5), "Wd": normal(H, F, std=F ** -0.5)}
    p = {"K": normal(B, max(L, 1), H), "V": normal(B, max(L, 1), H), "f_root": normal(B, H),
         "root_token": torch.randint(0, V, (B,), generator=g, device="cuda", dtype=torch.int32)}
    tok = torch.randint(0, V, (calls, B, k), generator=g, device="cuda", dtype=torch.int32)
    slot = torch.randint(0, k, (calls, B, k), generator=g, device="cuda", dtype=torch.int32)
    slot[1] = 0

    def layer(seqs):
        n = len(seqs)
        body = D.ddd_body_create(D.ddd_body_config(n, k, H, F, V, calls, L))
        pp = {name: t[seqs].contiguous() for name, t in p.items()}
        D.ddd_body_bind(body, w, pp)
        st, t = D.alloc_state(D.make_config(n, H, V, k, calls, 10, 0.0))
        out = []
        try:
            for s in range(calls):
                t["beam_token"].copy_(tok[s][seqs])
                t["beam_parent_slot"].copy_(slot[s][seqs])
                if s == 2 and n > 1:
                    t["row_active"][2 * k:3 * k] = 0
                h = torch.zeros(n if s == 0 else n * k, H, dtype=torch.bfloat16, device="cuda")
                D.ddd_body_step(body, s, st, h)
                torch.cuda.synchronize()
                out.append(h.float().reshape(n, -1, H))
        finally:
            D.ddd_body_destroy(body)
        return out

    got = layer(list(range(B)))
    for b in check:
        want = layer([b])
        for s in range(calls):
            if b == 2 and s >= 2:
                assert float(got[s][b].abs().max()) == 0.0
                continue
            rms = want[s][0].square().mean(-1, keepdim=True).sqrt()
            assert float(((got[s][b] - want[s][0]).abs() / rms).max()) <= 2 ** -5, (b, s)
