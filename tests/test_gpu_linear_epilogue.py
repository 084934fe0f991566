"""Linear and gated projections through integer-form weights: steps, residual, SiLU and rounding in the product's epilogue.  Widths at the edges of its
rules (multiples of 32 or not, rows in registers up to 4096 and 16384 columns) and of the 256 x 256 tiles, against 64 bits."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def grid_weights(rows, n, g):
    """fp32 weights on a 4-bit grid of one step per row"""
    k = torch.randint(0, 16, (rows, n), generator=g, device="cuda") - 7
    k[:, 0] = 1                                       # (the step itself is in every row)
    return (0.01 + 0.02 * torch.rand(rows, 1, generator=g, device="cuda")) * k


def setup(T, d, seed):
    g = torch.Generator(device="cuda"); g.manual_seed(seed)
    return g, torch.randn(T, d, generator=g, device="cuda").bfloat16()


def check(got, want, absum, d):
    """half an ulp of bf16, and fp32 sums of d terms of magnitude absum in all (their worst case), with 2^-22 for the fitted steps"""
    assert (np.abs(got.double().cpu().numpy() - want) <= 2.0 ** -8 * np.abs(want) + (d * 2.0 ** -24 + 2.0 ** -22) * absum + 1e-30).all()


@pytest.mark.parametrize("T,d,dout", [(8, 32, 8), (264, 64, 256), (257, 96, 264), (120, 40, 72), (24, 4096, 40), (24, 4128, 40), (16, 16416, 24)])
@pytest.mark.parametrize("res", [0, 1, 2])
def test_linear(lib, T, d, dout, res):
    g, X = setup(T, d, d + dout)
    W = grid_weights(dout, d, g)
    R = torch.randn(T, dout, generator=g, device="cuda").bfloat16() if res else None
    W = W.bfloat16() if res == 2 else W               # 16-bit weights: no steps
    ctx = lib.Context()
    n = ctx.counter(4)
    Y = ctx.linear_forward(X, W, residual=R)
    assert ctx.counter(4) - n == (res != 2)
    x, w = X.double().cpu().numpy(), W.double().cpu().numpy()
    r = R.double().cpu().numpy() if res else 0.0
    check(Y, x @ w.T + r, np.abs(x) @ np.abs(w).T + np.abs(r), d)


def test_linear_result_over_its_input(lib):
    """a result that takes the input's place, as the products with a pass behind them allow"""
    from paper_2602_04929_amd import binding as B
    g, X = setup(520, 256, 3)
    W = grid_weights(256, 256, g)
    ctx = lib.Context()
    want = ctx.linear_forward(X, W)
    ctx._check(B._lib.tboa_linear_forward(ctx._h, 520, 256, 256, B._dtype_code(X), B._ptr(X), B._dtype_code(W), B._ptr(W), None, B._ptr(X)))
    assert torch.equal(X, want)


@pytest.mark.parametrize("T,d,dff", [(8, 32, 32), (264, 64, 128), (257, 96, 160), (120, 32, 72), (120, 40, 64), (300, 128, 416)])
def test_swiglu(lib, T, d, dff):
    g, X = setup(T, d, d + dff)
    Wg, Wu = grid_weights(dff, d, g), grid_weights(dff, d, g)
    ctx = lib.Context()
    act = ctx.swiglu_forward(X, Wg, Wu)
    x, a, b = (t.double().cpu().numpy() for t in (X, Wg, Wu))
    G, U = x @ a.T, x @ b.T
    sg = G / (1 + np.exp(-G))
    # |silu'| < 1.1, silu(v) <= |v|; __expf and the division: 2^-20 relative
    absum = 1.1 * (np.abs(x) @ np.abs(a).T) * np.abs(U) + np.abs(sg) * (np.abs(x) @ np.abs(b).T)
    check(act, sg * U, absum + 2.0 ** 4 * np.abs(sg * U) / d, d)
