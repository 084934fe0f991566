"""16-bit products with at most 128 result rows, which take tiles of 128 x 256: edges in every direction, short and long contractions, batches, both 16-bit
types and the causal limit, against torch in 64 bits (GPU)."""
import pytest
import torch

pytestmark = pytest.mark.gpu
CAUSAL, PERSISTENT, HALF = 2, 4, 64


@pytest.mark.parametrize("half", [0, 1])
@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("batch,M,N,K", [(1, 128, 256, 32), (1, 1, 256, 96), (9, 64, 300, 320), (3, 100, 777, 800), (8, 127, 1024, 1024), (2, 129, 512, 512), (1, 128, 255, 64), (33, 64, 2048, 64)])
def test_against_64_bits(lib, batch, M, N, K, causal, half):
    ctx = lib.Context()
    g = torch.Generator(device="cuda"); g.manual_seed(M + N + K)
    dt = torch.float16 if half else torch.bfloat16
    A = torch.randn(batch, M, K, generator=g, device="cuda").to(dt)
    B = torch.randn(batch, N, K, generator=g, device="cuda").to(dt)
    if causal:      # column n of the result takes k up to n, rounded up to the tile
        B = B * (torch.arange(K, device="cuda")[None, :] <= torch.arange(N, device="cuda")[:, None])
    B = B.contiguous()
    a, b = A.double(), B.double().transpose(1, 2).contiguous()
    want, size = a @ b, a.abs() @ b.abs()
    flags = PERSISTENT | (CAUSAL if causal else 0) | (HALF if half else 0)
    got = ctx.gemm_bf16_nt(A.view(torch.bfloat16), B.view(torch.bfloat16), flags=flags)
    assert bool(((got.double() - want).abs() <= (K + 2) * 2.0 ** -24 * size).all())      # one rounding a product in 32 bits at most
    got16 = ctx.gemm_bf16_nt(A.view(torch.bfloat16), B.view(torch.bfloat16), out_dtype=torch.bfloat16, flags=flags).view(dt)
    assert bool(((got16.double() - want).abs() <= (K + 2) * 2.0 ** -24 * size + (2.0 ** -11 if half else 2.0 ** -8) * want.abs() + 2.0 ** -24).all())
    ctx.close()


def attention(X, Wq, Wk, Wv, hq, hkv, dh, cut=lambda name, t: t):
    """Concatenated attention outputs [S L, hq dh] in 64 bits; cut("v" or "a", t): what is done to values and probabilities."""
    S, L, d = X.shape
    mask = torch.ones(L, L, dtype=torch.bool, device=X.device).triu(1)
    out = torch.empty(S, L, hq * dh, dtype=torch.float64, device=X.device)
    for s in range(S):
        for h in range(hq):
            g = h * hkv // hq
            q, k, v = X[s] @ Wq[h * dh:(h + 1) * dh].T, X[s] @ Wk[g * dh:(g + 1) * dh].T, X[s] @ Wv[g * dh:(g + 1) * dh].T
            a = torch.softmax((q @ k.T / dh ** 0.5).masked_fill(mask, float("-inf")), 1)
            out[s, :, h * dh:(h + 1) * dh] = cut("a", a) @ cut("v", v)
    return out.reshape(S * L, hq * dh)


@pytest.mark.parametrize("L,hq,hkv,dh", [(256, 4, 2, 64), (512, 3, 1, 128), (256, 2, 1, 96), (264, 2, 1, 128), (288, 2, 2, 104), (328, 4, 4, 64)])
def test_values_times_probabilities_by_segments(lib, L, hq, hkv, dh):
    """The form in which attention outputs are taken: three segments or pairs of (hi, lo) operands with a causal limit each, a two-level batch, a (hi, lo) result; from the
    fused probabilities (whole 256s) and from stored ones.  Values have a common part and probabilities are nearly equal, so that what a missing or a
    wrong segment leaves out (2^-12 of an operand) does not average out: the oracle without the low part of either operand fails the bound."""
    S, d = 2, 64
    g = torch.Generator(device="cuda"); g.manual_seed(L + dh)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")
    xf = r(S, L, d); xf[..., 0] = 1.0
    X, Xf = (xf + 0.02 * r(S, L, d)).bfloat16(), xf.bfloat16()
    X[..., 0] = 1.0
    W = [0.002 * r(hq * dh, d), 0.002 * r(hkv * dh, d), 0.002 * r(hkv * dh, d)]
    W[2][:, 0] = 0.3 + 0.7 * torch.rand(hkv * dh, generator=g, device="cuda")
    Wb = [w.bfloat16() for w in W]
    ctx = lib.Context()
    H, R = ctx.build_hessian_out_proj(X, Xf, *W, *Wb, hq, hkv, dh, alpha=0.25)
    ctx.close()
    W64, Wb64 = [w.double() for w in W], [w.double() for w in Wb]
    O, Of = attention(X.double(), *W64, hq, hkv, dh), attention(Xf.double(), *Wb64, hq, hkv, dh)
    size = O.norm(dim=0)[:, None] * O.norm(dim=0)[None, :]
    # a query's probabilities are divided by their sum in fp32: L nearly equal numbers, each addition off by 2^-24 of the sum so far at most, together L / 2 of the whole
    # sum's; twice that in H, that of either path in R; they do not all round the same way in every binade: a quarter of it
    bound = L * 2.0 ** -26
    assert float(((H.double() - O.T @ O).abs() / size).max()) <= bound
    assert float(((R.double() - 0.25 * (O - Of).T @ O).abs() / size).max()) <= 0.25 * bound
    for x, w, n in ((X, W64, "v"), (X, W64, "a"), (Xf, Wb64, "v")):
        cut = attention(x.double(), *w, hq, hkv, dh, lambda m, t: t.half().double() if m == n else t)
        wrong = cut.T @ cut - O.T @ O if x is X else (Of - cut).T @ O
        assert float((wrong.abs() / size).max()) > bound
