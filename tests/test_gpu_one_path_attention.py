"""Fused causal probabilities of one score matrix (attention forward; Hessians without the full-precision path): tiles of 128 keys, whose two halves
different wavefronts take, at every head width the kernel has and from one to three diagonal blocks of 256, grouped-query heads included."""
import numpy as np
import pytest
import torch

from oracle import turboboa_ref as O
from paper_2602_04929_amd import synth

pytestmark = pytest.mark.gpu


def f64(t):
    return t.detach().float().cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("dh,hq,hkv,L", [(32, 4, 2, 256), (64, 2, 2, 768), (96, 3, 1, 512), (128, 2, 1, 512), (32, 16, 8, 256)])
def test_one_path(lib, dh, hq, hkv, L):
    cfg = synth.scaled(synth.CONFIGS["llama2-7b"], d_model=160, n_q_heads=hq, n_kv_heads=hkv, head_dim=dh, n_seqs=2, seq_len=L, n_outlier=2)
    b = synth.make_block(cfg, seed=L + dh, device="cuda")
    ctx = lib.Context()
    Og = ctx.attention_forward(b["X"], b["Wq"], b["Wk"], b["Wv"], hq, hkv, dh)
    want = O.attention_output(f64(b["X"]), f64(b["Wq"]), f64(b["Wk"]), f64(b["Wv"]), hq, hkv, dh)
    # stored in bf16: half an ulp of the value; 16-bit pairs before that (as in the other forward tests)
    assert (np.abs(f64(Og) - want) <= 2.0 ** -8 * np.abs(want) + 1e-5 * np.abs(want).max()).all()
    a = (b["Wq"], b["Wk"], b["Wv"], b["Wo"], hq, hkv, dh)
    H1 = ctx.build_hessians(b["X"], None, *a)["Hin_v"]
    H2 = ctx.build_hessians(b["X"], b["X_fp"], *a, alpha=0.25)["Hin_v"]
    # the same scores; fp32 sums of exponentials in another order, L 2^-24 at the most, twice in the product A^T A
    assert (H1 - H2).abs().max() <= 2 * L * 2.0 ** -24 * H2.abs().max()


@pytest.mark.parametrize("dh,hq,hkv,L", [(32, 8, 2, 256), (64, 6, 3, 768), (96, 3, 1, 512), (128, 8, 4, 1280)])
def test_one_path_takes_the_keys_in_the_order_of_two(lib, dh, hq, hkv, L):
    """Maximum and sum of a query go through its keys in the same order with one score matrix as with two, and the rounding of a sum shows its
    order: W_V's Hessian has the same bits with and without the full-precision path."""
    cfg = synth.scaled(synth.CONFIGS["llama2-7b"], d_model=256, n_q_heads=hq, n_kv_heads=hkv, head_dim=dh, n_seqs=2, seq_len=L, n_outlier=2)
    b = synth.make_block(cfg, seed=L + dh, device="cuda")
    ctx = lib.Context()
    a = (b["Wq"], b["Wk"], b["Wv"], b["Wo"], hq, hkv, dh)
    one = ctx.build_hessians(b["X"], None, *a)["Hin_v"]
    two = ctx.build_hessians(b["X"], b["X_fp"], *a, alpha=0.25)["Hin_v"]
    assert torch.equal(one, two)
    ctx.close()
