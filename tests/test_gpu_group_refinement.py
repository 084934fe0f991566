"""Group-wise scale refinement and the column sweep at the sizes where their kernels change path: few and many groups per wavefront, ragged heads,
several sweeps, and heads with so many scales that the diagonals, or the numerators too, no longer fit the LDS beside them."""
import numpy as np
import pytest
import torch

from oracle import turboboa_ref as O
from tests.parity import compare_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,heads,dh,group,iters,bits", [(64, 2, 5, 64, 1, 3), (96, 1, 7, 32, 2, 2), (512, 2, 9, 32, 1, 4), (1280, 1, 6, 16, 2, 3), (130, 2, 9, 2, 1, 2)])
def test_group_refinement_against_oracle(lib, n, heads, dh, group, iters, bits):
    rng = np.random.default_rng(n + dh)
    X = rng.standard_normal((3 * n, n)); X[:, : n // 16 + 1] *= 6
    Xf = X + 0.05 * rng.standard_normal(X.shape)
    H = (X.T @ X).astype(np.float32); R = (0.25 * (X - Xf).T @ X).astype(np.float32)
    K = rng.standard_normal((heads, 3 * dh, dh)); Ho = np.stack([k.T @ k for k in K]).astype(np.float32)
    W = (0.02 * rng.standard_normal((heads * dh, n))).astype(np.float32)
    ctx = lib.Context()
    d = lambda a: torch.from_numpy(a).cuda()
    got = ctx.quantize_layer(d(W), d(H), d(Ho), d(R), heads, bits, 4, group=group, cd_iters=iters)
    ref = O.quantize_layer(W.astype(np.float64), H.astype(np.float64), Ho.astype(np.float64), R.astype(np.float64), heads, bits=bits, block=4, group=group, cd_iters=iters)
    compare_layer(got, ref, min_code_match=1.0, rtol=1e-6)      # fp64 on both sides, fp32 results
    ctx.close()


@pytest.mark.parametrize("heads,dh,ng", [(1, 128, 157), (1, 64, 300), (1, 40, 64), (2, 128, 158), (3, 145, 140)])
def test_many_scales_per_head(lib, heads, dh, ng):
    """20480 doubles of LDS.  (40, 64): the scales, the numerators with a column of H_out and the diagonals fit; (128, 157), (64, 300): the diagonals do not;
    (128, 158), (145, 140): nothing does beside the scales, numerators and H_out are read from memory, a row of numerators per head.  The refinement must not
    depend on where they live: the result is that of the oracle's coordinate descent on the same codes."""
    group, bits = 2, 2
    n = group * ng
    rng = np.random.default_rng(dh)
    X = rng.standard_normal((2 * n, n)); H = (X.T @ X).astype(np.float32)
    K = rng.standard_normal((heads, 2 * dh, dh)); Ho = np.stack([k.T @ k for k in K]).astype(np.float32)
    W = (0.02 * rng.standard_normal((heads * dh, n))).astype(np.float32)
    ctx = lib.Context()
    d = lambda a: torch.from_numpy(a).cuda()
    raw = ctx.quantize_layer(d(W), d(H), d(Ho), None, heads, bits, dh, group=group, cd_iters=0)
    got = ctx.quantize_layer(d(W), d(H), d(Ho), None, heads, bits, dh, group=group, cd_iters=1)
    assert torch.equal(raw["codes"], got["codes"])
    z = got["zeros"].cpu().numpy().astype(np.float64)
    wbar = got["codes"].cpu().numpy().astype(np.float64) - np.repeat(z, group, axis=1)
    s = raw["scales"].cpu().numpy().astype(np.float64)
    Hd = O.damp_hessian(H.astype(np.float64), 0.01)
    # the sequence of the method on Gram products: one d_h vector per (row, group) instead of the oracle's full rows (same steps)
    W64 = W.astype(np.float64); Q = np.repeat(s, group, axis=1) * wbar
    V = (W64 - Q) @ Hd
    for h in range(heads):
        Hod, rows = O.damp_hessian(Ho[h].astype(np.float64), 0.01), slice(h * dh, (h + 1) * dh)
        for j in range(dh):
            for g in range(ng):
                G, r = slice(g * group, (g + 1) * group), h * dh + j
                num = wbar[r, G] @ (V[rows, G].T @ Hod[:, j])
                den = wbar[r, G] @ Hd[G, G] @ wbar[r, G] * Hod[j, j]
                if den > 0:
                    step = num / den
                    s[r, g] += step
                    V[r] -= step * (wbar[r, G] @ Hd[G])
    got_s = got["scales"].cpu().numpy().astype(np.float64)
    # the start values are the library's fp32 scales (2^-24 relative); the descent is a contraction on them
    assert np.abs(got_s - s).max() <= 2e-6 * np.abs(s).max()
    ctx.close()
