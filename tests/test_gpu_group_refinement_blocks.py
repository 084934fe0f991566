"""Group-wise scale refinement where a head's rows go in blocks of 16: heads of 15, 16, 17 and 33 rows, 64 groups (a lane each) and 65 (the general recurrence), several sweeps; a group
without weights keeps its scale."""
import numpy as np
import pytest
import torch

from oracle import turboboa_ref as O
from tests.parity import compare_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,heads,dh,group,iters,bits", [(264, 2, 15, 8, 2, 3), (512, 2, 16, 8, 1, 2), (520, 1, 17, 8, 2, 3), (96, 3, 33, 32, 2, 4)])
def test_blocks_of_rows_against_oracle(lib, n, heads, dh, group, iters, bits):
    rng = np.random.default_rng(n + dh)
    X = rng.standard_normal((3 * n, n)); X[:, : n // 16 + 1] *= 6
    Xf = X + 0.05 * rng.standard_normal(X.shape)
    H = (X.T @ X).astype(np.float32); R = (0.25 * (X - Xf).T @ X).astype(np.float32)
    K = rng.standard_normal((heads, 3 * dh, dh)); Ho = np.stack([k.T @ k for k in K]).astype(np.float32)
    W = (0.02 * rng.standard_normal((heads * dh, n))).astype(np.float32)
    W[3, group:2 * group] = 0.0
    ctx = lib.Context()
    d = lambda a: torch.from_numpy(a).cuda()
    got = ctx.quantize_layer(d(W), d(H), d(Ho), d(R), heads, bits, dh, group=group, cd_iters=iters)
    ref = O.quantize_layer(W.astype(np.float64), H.astype(np.float64), Ho.astype(np.float64), R.astype(np.float64), heads, bits=bits, block=dh, group=group, cd_iters=iters)
    compare_layer(got, ref, min_code_match=1.0, rtol=1e-6)      # fp64 on both sides, fp32 results
    ctx.close()
