"""Attention outputs of the fused kernel (forward pass, W_O Hessian) against fp64: every head width it has, lengths around its tiles (8 keys, 32, 64, 128 and 256 queries, +- 8), blocked and
row-major operands (lengths that are multiples of 16 or only of 8), with and without the causal mask, few heads and many; undefined activations."""
import math

import pytest
import torch

from paper_2602_04929_amd import synth

pytestmark = pytest.mark.gpu

CASES = [(32, 4, 2, 1, 8, 1), (64, 2, 1, 2, 24, 1), (128, 2, 2, 1, 32, 1), (96, 3, 1, 2, 40, 0), (64, 4, 4, 1, 64, 0), (128, 4, 2, 2, 72, 1), (32, 2, 2, 3, 128, 1), (128, 2, 1, 1, 136, 1),
         (96, 2, 2, 1, 256, 1), (64, 3, 3, 2, 264, 1), (128, 2, 2, 1, 520, 0), (128, 4, 4, 2, 1000, 1), (64, 32, 8, 16, 64, 1), (128, 64, 64, 8, 40, 1), (32, 16, 4, 8, 1032, 1)]


def block(dh, hq, hkv, S, L):
    cfg = synth.scaled(synth.CONFIGS["llama2-7b"], d_model=192, n_q_heads=hq, n_kv_heads=hkv, head_dim=dh, n_seqs=S, seq_len=L, n_outlier=2)
    return synth.make_block(cfg, seed=L + dh + hq, device="cuda")


def attention(X, Wq, Wk, Wv, hq, hkv, dh, causal):
    X, Wq, Wk, Wv = (t.double() for t in (X, Wq, Wk, Wv))
    S, L, _ = X.shape
    out = torch.empty(S, L, hq * dh, dtype=torch.float64, device="cuda")
    for s in range(S):
        for h in range(hq):
            g = slice(h // (hq // hkv) * dh, (h // (hq // hkv) + 1) * dh)
            sc = (X[s] @ Wq[h * dh:(h + 1) * dh].T) @ (X[s] @ Wk[g].T).T / math.sqrt(dh)
            if causal:
                sc = sc.masked_fill(torch.ones_like(sc, dtype=torch.bool).triu(1), -math.inf)
            out[s, :, h * dh:(h + 1) * dh] = torch.softmax(sc, -1) @ (X[s] @ Wv[g].T)
    return out


@pytest.mark.parametrize("dh,hq,hkv,S,L,causal", CASES)
def test_forward(lib, dh, hq, hkv, S, L, causal):
    print("attention_forward", dh, hq, hkv, S, L, causal, flush=True)
    b = block(dh, hq, hkv, S, L)
    ctx = lib.Context()
    got = ctx.attention_forward(b["X"], b["Wq"], b["Wk"], b["Wv"], hq, hkv, dh, causal=bool(causal)).double()
    ctx.close()
    want = attention(b["X"], b["Wq"], b["Wk"], b["Wv"], hq, hkv, dh, causal)
    # stored in bf16: half a unit of at most 2^-7 |value| each, 2^-7 / sqrt(12) as root mean square.  Beyond that what the operands' 16 bits leave of a score (2^-17 |q||k| / d_h, scores up to
    # 9e3 here) moves between keys: 2.5e-5 of the largest value at most as measured; of half pairs (whole 256s, causal), 22 bits, 1e-9
    slack = 1e-6 if L % 256 == 0 and causal else 1e-4
    assert ((got - want).abs() <= 2.0 ** -8 * want.abs() + slack * want.abs().max()).all()
    assert torch.linalg.norm(got - want) <= 2.0 ** -7 / math.sqrt(12.0) * torch.linalg.norm(want)


@pytest.mark.parametrize("value", [float("nan"), float("inf"), -float("inf")])
@pytest.mark.parametrize("dh,hq,hkv,S,L,causal", [(64, 2, 1, 2, 24, 1), (128, 4, 2, 2, 72, 1), (64, 4, 4, 2, 64, 0), (32, 16, 4, 8, 1032, 1), (128, 2, 2, 2, 256, 1), (96, 2, 2, 2, 512, 1)])
def test_undefined_activations(lib, dh, hq, hkv, S, L, causal, value):
    """One entry of one token that is no number: undefined outputs for that token and all that attend to it, right ones for the other sequences and for tokens before its block of 32 keys."""
    print("attention_forward", dh, hq, hkv, S, L, causal, value, flush=True)
    b = block(dh, hq, hkv, S, L)
    want = attention(b["X"], b["Wq"], b["Wk"], b["Wv"], hq, hkv, dh, causal)
    t0 = L // 2
    X = b["X"].clone()
    X[-1, t0, 3] = value
    ctx = lib.Context()
    got = ctx.attention_forward(X, b["Wq"], b["Wk"], b["Wv"], hq, hkv, dh, causal=bool(causal)).double()
    ctx.close()
    assert not torch.isfinite(got[-1, t0 if causal else 0:]).any()
    # (values and probabilities are bf16 pairs then, 16 bits each)
    near = lambda g, w: ((g - w).abs() <= 2.0 ** -8 * w.abs() + 1e-3 * want.abs().max()).all()  # noqa: E731
    assert near(got[:-1], want[:-1])
    if causal:
        assert near(got[-1, :t0 // 32 * 32], want[-1, :t0 // 32 * 32])


@pytest.mark.parametrize("dh,hq,hkv,S,L", [(64, 2, 1, 2, 24), (128, 4, 2, 2, 72), (96, 2, 2, 3, 256), (32, 4, 4, 2, 264), (64, 32, 8, 16, 64)])
def test_hessian_of_the_output_projection(lib, dh, hq, hkv, S, L):
    """Both paths side by side: H and R against fp64, and H with the same bits as without the second path."""
    print("build_hessian_out_proj", dh, hq, hkv, S, L, flush=True)
    b = block(dh, hq, hkv, S, L)
    w = {k: b[k].float() * 1.01 for k in ("Wq", "Wk", "Wv")}
    ctx = lib.Context()
    H, R = ctx.build_hessian_out_proj(b["X"], b["X_fp"], w["Wq"], w["Wk"], w["Wv"], b["Wq"], b["Wk"], b["Wv"], hq, hkv, dh, alpha=0.25)
    H1, _ = ctx.build_hessian_out_proj(b["X"], None, w["Wq"], w["Wk"], w["Wv"], None, None, None, hq, hkv, dh)
    ctx.close()
    assert torch.equal(H, H1)
    o = attention(b["X"], w["Wq"], w["Wk"], w["Wv"], hq, hkv, dh, 1).flatten(0, 1)
    of = attention(b["X_fp"], b["Wq"], b["Wk"], b["Wv"], hq, hkv, dh, 1).flatten(0, 1)
    want, dev = o.T @ o, 0.25 * ((o - of).T @ o)
    bar = 2e-3 if L % 256 else 2e-6
    assert torch.linalg.norm(H - want) <= bar * torch.linalg.norm(want)
    assert torch.linalg.norm(R - dev) <= 10 * bar * torch.linalg.norm(dev)


@pytest.mark.parametrize("up", [6, 10, 14])
@pytest.mark.parametrize("dh,hq,hkv,S,L,causal", [(128, 4, 2, 2, 72, 1), (64, 4, 4, 2, 264, 0), (128, 2, 2, 2, 256, 1), (96, 2, 2, 2, 512, 1)])
def test_large_scores(lib, dh, hq, hkv, S, L, causal, up):
    """Scores of 1e7, 1e9 and 1e12, of which fp32 leaves units of 1, 64 and 65536 (correlated channels with heavy-tailed tokens reach 1e8): a softmax that picks one key.  Where the two largest scores
    of a query are further apart than what the operands' 16 bits and fp32 sums leave of them, the output is the value of the larger; no output is undefined or larger than the values."""
    print("attention_forward", dh, hq, hkv, S, L, causal, up, flush=True)
    b = block(dh, hq, hkv, S, L)
    wq, wk = b["Wq"] * 2.0 ** up, b["Wk"] * 2.0 ** up
    ctx = lib.Context()
    got = ctx.attention_forward(b["X"], wq, wk, b["Wv"], hq, hkv, dh, causal=bool(causal)).double().view(S, L, hq, dh)
    ctx.close()
    X, rep = b["X"].double(), hq // hkv
    q, k, v = ((X @ w.double().T).view(S, L, -1, dh).transpose(1, 2) for w in (wq, wk, b["Wv"]))
    k, v = k.repeat_interleave(rep, 1), v.repeat_interleave(rep, 1)
    sc = torch.matmul(q, k.transpose(2, 3).contiguous()) / math.sqrt(dh)
    if causal:
        sc = sc.masked_fill(torch.ones(L, L, dtype=torch.bool, device="cuda").triu(1), -math.inf)
    two, at = sc.topk(2, -1)
    want = torch.gather(v, 2, at[..., :1].expand(-1, -1, -1, dh)).transpose(1, 2)
    decided = (two[..., 0] - two[..., 1] > 2.0 ** -13 * q.norm(dim=-1) * k.norm(dim=-1).amax(-1, keepdim=True) / math.sqrt(dh) + 40.0).transpose(1, 2)
    assert decided.double().mean() > 0.25
    assert got.abs().amax() <= 1.01 * v.abs().amax()      # (no NaN either)
    assert ((got - want).abs() <= 2.0 ** -8 * want.abs() + 1e-4 * want.abs().max())[decided].all()
