"""The column sweep at the edges of its sub-panels (16 columns), tiles (16 rows) and groups (512 columns), with and without the deviation term, shared and
per-head Hessians, grid groups narrower than, equal to and wider than a sub-panel; and columns that lie on the border between two codes."""
import ctypes as C

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


@pytest.mark.parametrize("n,rows,dev,kw", [(40, 20, 0, {}), (40, 20, 1, {}), (1100, 8, 1, {}), (528, 6, 0, {}), (96, 6, 1, dict(group=32, adaptive_grid=False))])
@pytest.mark.parametrize("where", ["first", "in a sub-panel", "end of a sub-panel", "last"])
def test_an_undefined_weight_touches_later_columns_only(lib, n, rows, dev, kw, where):
    """An undefined weight leaves the columns before it, and the other rows, as they are without it (the grids have one candidate each, whose range it
    does not enter).  Asked for no loss, the call reports nothing."""
    col = {"first": 0, "in a sub-panel": 23, "end of a sub-panel": 31, "last": n - 1}[where]
    g = torch.Generator(device="cuda"); g.manual_seed(n + col)
    X = torch.randn(2 * n, n, generator=g, device="cuda", dtype=torch.float64)
    H = (X.T @ X).float()
    R = (0.05 * X.T @ torch.randn(2 * n, n, generator=g, device="cuda", dtype=torch.float64)).float() if dev else None
    W = 0.02 * torch.randn(rows, n, generator=g, device="cuda")
    ctx = lib.Context()
    ng = n // kw["group"] if kw else 1

    def codes(bad):
        w = W.clone(); w[2, col] = bad
        d = ctx.layer_desc(w, H, 1, 4, rows, grid_points=100, max_shrink=0.01, cd_iters=0, **kw)
        out = [torch.empty(rows, n, dtype=torch.uint8, device="cuda"), torch.empty(rows, ng, device="cuda"), torch.empty(rows, ng, device="cuda"), torch.empty(rows, n, device="cuda")]
        p = lib.binding._ptr
        ctx._check(lib.binding._lib.tboa_quantize_layer(ctx._h, C.byref(d), p(w), p(H), None, p(R), *[p(t) for t in out], None, None))
        return out
    got, want = codes(float("nan")), codes(0.0)
    for a, b in zip((got[0], got[3]), (want[0], want[3])):
        assert torch.equal(a[2, :col], b[2, :col])
        assert torch.equal(a[[i for i in range(rows) if i != 2]], b[[i for i in range(rows) if i != 2]])
    ctx.close()
