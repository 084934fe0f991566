"""bf16 Hessian builds whose sequence length or token count is no multiple of 32 (the products run over columns padded with zeros), against the
oracle.  Bounds: the exact-input sums (H_in, R of W_Q / W_K and of a linear layer) at fp32 accumulation, 2e-6 of the largest entry; the
W_V Hessian of these shapes takes single 16-bit probabilities and Y (5e-4 / 5e-3), the W_O Hessian pairs (1e-5, its deviation term
from scores of 16 bits: 1e-3)."""
import numpy as np
import pytest
import torch

from oracle import turboboa_ref as O
from paper_2602_04929_amd import synth

pytestmark = pytest.mark.gpu


def worst(got, want):
    return np.abs(got.double().cpu().numpy() - want).max() / np.abs(want).max()


@pytest.mark.parametrize("S,L,d,hq,hkv,dh,causal", [(1, 8, 64, 2, 1, 32, 1), (3, 40, 64, 2, 2, 32, 1), (2, 104, 96, 2, 1, 40, 0), (2, 248, 256, 2, 2, 64, 1),
                                                    (1, 264, 128, 2, 1, 64, 1), (2, 1000, 64, 1, 1, 32, 1), (1, 2056, 64, 1, 1, 32, 1), (2, 2056, 40, 1, 1, 24, 0)])
def test_ragged_sequences(lib, S, L, d, hq, hkv, dh, causal):
    cfg = synth.scaled(synth.CONFIGS["llama2-7b"], d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=dh, n_seqs=S, seq_len=L, n_outlier=2)
    b = synth.make_block(cfg, seed=L, device="cuda")
    f = lambda t: t.float().cpu().numpy().astype(np.float64)
    ctx = lib.Context()
    # a call of another shape first: its values are what lies in the workspace where this one's padding is
    ctx.build_hessian_linear(torch.full((2048, 512), 3e4, device="cuda").bfloat16())
    args = (hq, hkv, dh)
    got = ctx.build_hessians(b["X"], b["X_fp"], b["Wq"], b["Wk"], b["Wv"], b["Wo"], *args, alpha=0.25, causal=bool(causal))
    ref = O.build_hessians(f(b["X"]), f(b["X_fp"]), f(b["Wq"]), f(b["Wk"]), f(b["Wv"]), f(b["Wo"]), *args, alpha=0.25, causal=bool(causal))
    for k, tol in (("Hin_qk", 2e-6), ("R_qk", 2e-6), ("Hout_q", 2e-6), ("Hout_k", 2e-6), ("Hout_v", 2e-6), ("Hin_v", 5e-4), ("R_v", 5e-3)):
        assert worst(got[k], ref[k]) <= tol, k
    dq = [(f(b[w]) * 64).round() / 64 for w in ("Wq", "Wk", "Wv")]
    deq = [torch.from_numpy(w.astype(np.float32)).cuda() for w in dq]
    H, R = ctx.build_hessian_out_proj(b["X"], b["X_fp"], *deq, b["Wq"], b["Wk"], b["Wv"], *args, alpha=0.25, causal=bool(causal))
    Hr, Rr = O.build_hessian_out_proj(f(b["X"]), f(b["X_fp"]), *dq, f(b["Wq"]), f(b["Wk"]), f(b["Wv"]), *args, alpha=0.25, causal=bool(causal))
    assert worst(H, Hr) <= 1e-5 and worst(R, Rr) <= 1e-3
    ctx.close()


@pytest.mark.parametrize("T,n", [(8, 8), (40, 72), (264, 40), (1000, 264), (2056, 96), (4096, 520)])
def test_ragged_tokens_of_a_linear_layer(lib, T, n):
    g = torch.Generator(device="cuda"); g.manual_seed(T)
    x = torch.randn(T, n, generator=g, device="cuda")
    X, Xf = (x + 0.05 * torch.randn(T, n, generator=g, device="cuda")).bfloat16(), x.bfloat16()
    ctx = lib.Context()
    H, R = ctx.build_hessian_linear(X, Xf, 0.25)
    f = lambda t: t.float().cpu().numpy().astype(np.float64)
    Hr, Rr = O.build_hessian_linear(f(X), f(Xf), 0.25)
    assert worst(H, Hr) <= 2e-6 and worst(R, Rr) <= 2e-6
    H1, _ = ctx.build_hessian_linear(X)
    assert torch.equal(H, H1)
    ctx.close()
