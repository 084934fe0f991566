"""The column sweep at the edges of its sub-panels (16 columns), tiles (16 rows) and groups (512 columns), with and without the deviation term, shared and
per-head Hessians, grid groups narrower than, equal to and wider than a sub-panel; and columns that lie on the border between two codes."""
import numpy as np
import pytest
import torch

from oracle import turboboa_ref as O
from tests.parity import compare_layer

pytestmark = pytest.mark.gpu


def run(lib, W, H, R, Ho, heads, bits, block, **kw):
    ctx = lib.Context()
    d = lambda a: None if a is None else torch.from_numpy(a).cuda()
    f = lambda a: None if a is None else a.astype(np.float64)
    got = ctx.quantize_layer(d(W), d(H), d(Ho), d(R), heads, bits, block, **kw)
    ref = O.quantize_layer(f(W), f(H), f(Ho), f(R), heads, bits=bits, block=block, **kw)
    compare_layer(got, ref, min_code_match=1.0, rtol=1e-6)      # fp64 on both sides, fp32 results
    ctx.close()


@pytest.mark.parametrize("n,heads,dh,block,per_head,dev,kw", [
    (15, 1, 1, 1, 0, 1, {}), (16, 2, 8, 8, 0, 0, {}), (17, 3, 17, 17, 1, 1, {}), (33, 5, 7, 3, 0, 1, {}), (511, 1, 16, 16, 0, 1, {}), (512, 2, 9, 4, 1, 0, {}),
    (513, 1, 33, 33, 0, 1, {}), (529, 3, 11, 5, 0, 1, {}), (1024, 2, 20, 20, 1, 1, {}), (96, 2, 6, 3, 0, 1, dict(group=8)), (128, 1, 6, 6, 0, 1, dict(group=16)),
    (128, 2, 5, 5, 0, 1, dict(group=8, adaptive_grid=False)), (576, 1, 18, 9, 0, 1, dict(group=192)), (640, 1, 18, 9, 0, 0, dict(group=32, adaptive_grid=False)),
    (768, 2, 4, 2, 0, 1, dict(group=128))])
def test_sweep_edges(lib, n, heads, dh, block, per_head, dev, kw):
    rng = np.random.default_rng(n + dh)
    H, R = [], []
    for _ in range(heads if per_head else 1):
        X = rng.standard_normal((2 * n + 16, n)); X[:, : n // 16 + 1] *= 8
        Xf = X + 0.1 * rng.standard_normal(X.shape)
        H.append((X.T @ X).astype(np.float32)); R.append((0.25 * (X - Xf).T @ X).astype(np.float32))
    H, R = (np.stack(H), np.stack(R)) if per_head else (H[0], R[0])
    K = rng.standard_normal((heads, 3 * dh, dh)); Ho = np.stack([k.T @ k for k in K]).astype(np.float32)
    W = (0.02 * rng.standard_normal((heads * dh, n))).astype(np.float32)
    run(lib, W, H, R if dev else None, Ho, heads, 3, block, **kw)


def test_columns_on_the_border_between_codes(lib):
    """Independent channels (no column changes before its turn), weights at whole and half multiples of their row's step: w / s rounds to a half-integer where
    w (1 / s) may not, and the code is that of the division."""
    rng = np.random.default_rng(3)
    n, rows = 160, 24
    step = (0.01 * (1 + np.arange(rows)) / 3).astype(np.float32).astype(np.float64)
    k = rng.integers(0, 15, size=(rows, n)) / 2.0 - 3.5
    k[:, 0], k[:, 1] = -3.5, 3.5
    W = (step[:, None] * k).astype(np.float32)
    H = np.diag(rng.uniform(1, 4, n)).astype(np.float32)
    run(lib, W, H, None, None, 1, 3, rows, damp=0.0)
