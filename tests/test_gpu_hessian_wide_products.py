"""H_out of W_Q and W_K where the product of the stacked weights with H_in runs as a product of residues: ragged widths, all heads or few KV heads, fewer rows than columns, sequences so short
that the residues outgrow the other buffers; one shape on the fp64 side of the line; channels so small that their squares vanish in fp32.

Against fp64 from the H_in that the call returns: what is left is the result's rounding to fp32, 2^-24 of each entry, and the fp64 sums' own."""
import pytest
import torch

from paper_2602_04929_amd import synth

pytestmark = pytest.mark.gpu


def check(lib, cfg, hq, hkv, dh, seed, tiny=None):
    d = cfg.d_model
    b = synth.make_block(cfg, seed=seed, device="cuda")
    if tiny is not None:
        b["X"][..., 5::97] *= tiny
        b["X_fp"][..., 5::97] *= tiny
    ctx = lib.Context()
    got = ctx.build_hessians(b["X"], b["X_fp"], b["Wq"], b["Wk"], b["Wv"], b["Wo"], hq, hkv, dh, alpha=0.25)
    ctx.close()
    H, rep = got["Hin_qk"].double(), hq // hkv
    assert torch.equal(H, H.T.contiguous())
    if tiny is not None:
        assert (H.diagonal()[5::97] == 0.0).any() and (H[5::97, 6] != 0.0).all()

    def sums(W, heads):
        w = W.double().view(heads, dh, d)
        return torch.stack([(m @ H) @ m.T for m in w])
    want = {"Hout_q": sums(b["Wk"], hkv).repeat_interleave(rep, 0), "Hout_k": sums(b["Wq"], hq).view(hkv, rep, dh, dh).sum(1)}
    for k, w in want.items():
        g = got[k].double()
        size = w.diagonal(dim1=1, dim2=2).sqrt()
        assert ((g - w).abs() <= 2.0 ** -24 * w.abs() + 2.0 ** -40 * size[:, :, None] * size[:, None, :]).all(), k


@pytest.mark.parametrize("d,hq,hkv,dh,S,L", [(1544, 12, 3, 128, 2, 264), (1536, 12, 12, 128, 1, 64), (2056, 8, 8, 64, 3, 1000), (2312, 6, 2, 72, 2, 256), (3000, 8, 4, 64, 1, 40), (1024, 8, 2, 128, 2, 256)])
def test_against_fp64(lib, d, hq, hkv, dh, S, L):
    check(lib, synth.scaled(synth.CONFIGS["llama2-7b"], d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=dh, n_seqs=S, seq_len=L, n_outlier=4), hq, hkv, dh, d + L)


@pytest.mark.parametrize("d,hq,hkv,dh,S,L", [(1544, 12, 3, 128, 2, 264), (1536, 12, 12, 128, 1, 64)])
def test_channels_whose_squares_vanish(lib, d, hq, hkv, dh, S, L):
    """Zeros on H_in's diagonal beside entries that are none: such a channel is no channel without activations."""
    check(lib, synth.scaled(synth.CONFIGS["llama2-7b"], d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=dh, n_seqs=S, seq_len=L, n_outlier=4), hq, hkv, dh, d + L, tiny=1e-26)
