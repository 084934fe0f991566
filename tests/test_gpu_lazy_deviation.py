"""The column sweep with the deviation term taken through R and the diagonal blocks of R U^T (few rows per wide H_in) against the oracle, which forms P:
the widths end a group of 512 columns exactly, one panel into the next, and in the middle of a panel; heads with a Hessian each and a shared one."""
import numpy as np
import pytest
import torch

from oracle import turboboa_ref as O
from tests.parity import compare_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,heads,dh,block,per_head,coupled", [(1088, 2, 9, 4, 1, 1), (1536, 1, 20, 7, 0, 1), (1600, 3, 10, 10, 0, 1), (1090, 1, 24, 24, 0, 0), (1201, 2, 5, 2, 1, 1)])
def test_lazy_deviation_term(lib, n, heads, dh, block, per_head, coupled):
    rng = np.random.default_rng(n)
    nh = heads if per_head else 1
    H, R = [], []
    for _ in range(nh):
        X = rng.standard_normal((n + n // 2, n)); X[:, :8] *= 10
        Xf = X + 0.1 * rng.standard_normal(X.shape)
        H.append((X.T @ X).astype(np.float32)); R.append((0.25 * (X - Xf).T @ X).astype(np.float32))
    H, R = (np.stack(H), np.stack(R)) if per_head else (H[0], R[0])
    K = rng.standard_normal((heads, 3 * dh, dh)); Ho = np.stack([k.T @ k for k in K]).astype(np.float32) if coupled else None
    W = (0.02 * rng.standard_normal((heads * dh, n))).astype(np.float32)
    ctx = lib.Context()
    d = lambda a: None if a is None else torch.from_numpy(a).cuda()
    f = lambda a: None if a is None else a.astype(np.float64)
    got = ctx.quantize_layer(d(W), d(H), d(Ho), d(R), heads, 3, block)
    ref = O.quantize_layer(f(W), f(H), f(Ho), f(R), heads, bits=3, block=block)
    compare_layer(got, ref, min_code_match=1.0, rtol=1e-6)      # fp64 on both sides, fp32 results
    ctx.close()
