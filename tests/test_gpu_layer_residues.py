"""Layers whose large products run on the integer matrix cores against the same rows quantized by themselves, whose products stay in fp64 (few rows do not repay the operands' preparation).

Heads do not depend on each other, and without H_out rows do not: the slices must agree.  The paths differ in rounding only, 2^-55 of a product's operands each: whole numbers are
compared for equality (no decision of these inputs lies that close to a tie), scales with fp32's spacing, losses with 1e-10."""
import pytest
import torch

pytestmark = pytest.mark.gpu

# name, rows, columns, heads, H_out, R, options: every kind of product, with the others and alone; whole and ragged widths; more rows than one set of residues holds
CASES = [
    ("rows", 4104, 2950, 1, False, True, dict(bits=2, block=4104)),
    ("rows-int8-cd3", 2048, 2944, 1, False, True, dict(bits=8, block=2048, cd_iters=3)),
    ("rows-no-cd", 3000, 2888, 1, False, False, dict(bits=4, block=3000, cd_iters=0)),
    ("rows-group", 2048, 2944, 1, False, True, dict(bits=3, block=2048, group=128)),
    ("rows-past-8192", 8450, 2560, 1, False, True, dict(bits=2, block=8450)),
    ("heads", 4096, 2950, 64, True, True, dict(bits=2, block=16)),
    ("heads-wide-block", 2112, 2948, 33, True, True, dict(bits=2, block=64)),
    ("heads-noR", 2112, 2950, 33, True, False, dict(bits=3, block=32)),
    ("heads-no-cd", 2112, 2944, 33, True, True, dict(bits=2, block=16, cd_iters=0, adaptive_grid=False)),
    ("heads-group", 4096, 2944, 64, True, True, dict(bits=4, block=32, group=128)),
    ("heads-fp64-grid", 2112, 2944, 33, True, True, dict(bits=2, block=32, grid_guard=-1.0)),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_slice_of_a_layer(lib, case):
    name, rows, n, heads, with_out, with_R, kw = case
    g = torch.Generator(device="cuda").manual_seed(len(name) * 1009 + rows + n)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)  # noqa: E731
    dh, T = rows // heads, 4096
    X = rnd(T, n) + 0.5 * rnd(T, 1)
    X[:, ::97] *= 10.0
    Hin = X.T @ X
    R = (0.025 * (rnd(T, n).T @ X)).contiguous() if with_R else None
    W = 0.02 * rnd(rows, n)
    G = rnd(heads, 512, dh) + 0.7 * rnd(heads, 512, 1)
    Hout = torch.matmul(G.transpose(1, 2).contiguous(), G).contiguous() if with_out else None
    ctx = lib.Context()
    whole = ctx.quantize_layer(W, Hin, Hout, R, heads, **kw)
    picks = [0, heads - 1] if with_out else [0, 1]
    for p in picks:
        r0, r1 = (p * dh, (p + 1) * dh) if with_out else ((0, 40) if p == 0 else (rows - 24, rows))
        part = ctx.quantize_layer(W[r0:r1].contiguous(), Hin, Hout[p:p + 1].contiguous() if with_out else None, R, 1, **dict(kw, block=min(kw["block"], r1 - r0)))
        assert torch.equal(whole["codes"][r0:r1], part["codes"])
        assert torch.equal(whole["zeros"][r0:r1], part["zeros"])
        torch.testing.assert_close(whole["scales"][r0:r1], part["scales"], rtol=2.0 ** -22, atol=0.0)
        torch.testing.assert_close(whole["W_deq"][r0:r1], part["W_deq"], rtol=2.0 ** -22, atol=0.0)
        if with_out:
            for a, b in zip(whole["loss_per_head_terms"][p], part["loss_per_head_terms"][0]):
                assert abs(a - b) <= 1e-10 * max(abs(a), abs(b), part["loss_quad"])
    ctx.close()


@pytest.mark.parametrize("rows,n,heads,kw", [(4096, 2950, 64, dict(bits=2, block=16)), (2112, 2948, 33, dict(bits=8, block=64)), (4096, 2944, 64, dict(bits=4, block=32, group=128))])
def test_weights_that_fall_as_their_channels_grow(lib, rows, n, heads, kw):
    """Channels of 1e-4 .. 1e4 and weights that fall as their channel grows: in a sum over channels every one counts alike, and the sum is known to fp64's rounding only where the product takes
    the sizes out.  The loss of the deviation, 2 tr(H_out W R D^T), shows W R to 64 bits: 2^-54 of the sum of its terms' magnitudes, some 2^8 - 2^12 of it (random signs), and as much
    again from H_out; compared with 2^-38.  In units of the largest channels it was off by 2^-28 - 2^-33."""
    g = torch.Generator(device="cuda").manual_seed(rows + n)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)  # noqa: E731
    dh, T = rows // heads, 4096
    s = 10.0 ** (8.0 * torch.rand(n, device="cuda", generator=g) - 4.0)
    X = ((rnd(T, n) + 0.5 * rnd(T, 1)) * s).double()
    Hin, R = (X.T @ X).float(), (0.0125 * ((rnd(T, n) * s).double().T @ X)).float().contiguous()
    W = 0.02 * rnd(rows, n) / s
    G = rnd(heads, 512, dh) + 0.7 * rnd(heads, 512, 1)
    Hout = torch.matmul(G.transpose(1, 2).contiguous(), G).contiguous()
    ctx = lib.Context()
    whole = ctx.quantize_layer(W, Hin, Hout, R, heads, **kw)
    for p in (0, heads - 1):
        part = ctx.quantize_layer(W[p * dh:(p + 1) * dh].contiguous(), Hin, Hout[p:p + 1].contiguous(), R, 1, **kw)
        assert torch.equal(whole["codes"][p * dh:(p + 1) * dh], part["codes"])
        (a, ac), (b, bc) = whole["loss_per_head_terms"][p], part["loss_per_head_terms"][0]
        assert abs(a - b) <= 2.0 ** -40 * b and abs(ac - bc) <= 2.0 ** -38 * abs(bc)
    ctx.close()


@pytest.mark.parametrize("rows,n", [(4096, 2944), (5000, 2816)])
def test_updates_of_channels_that_the_damping_holds(lib, rows, n):
    """Groups of channels of very different size, with weights to match and a grid for each: in the small ones, which the damping makes as large as 1e-2 of the mean, U is little else than
    diagonal, and what the sweep takes from earlier columns is as small as their weights are.  Their codes are those of the same rows by themselves, whose updates run in fp64;
    with updates rounded in units of U's diagonal some of them were not."""
    g = torch.Generator(device="cuda").manual_seed(rows + n)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)  # noqa: E731
    s = (10.0 ** (14.0 * torch.rand(n // 128, device="cuda", generator=g) - 7.0)).repeat_interleave(128)
    X = ((rnd(4096, n) + 0.5 * rnd(4096, 1)) * s).double()
    Hin, R, W = (X.T @ X).float(), (0.0125 * ((rnd(4096, n) * s).double().T @ X)).float().contiguous(), 0.02 * rnd(rows, n) * s
    ctx = lib.Context()
    whole = ctx.quantize_layer(W, Hin, None, R, 1, bits=4, block=rows, group=128)
    part = ctx.quantize_layer(W[:40].contiguous(), Hin, None, R, 1, bits=4, block=40, group=128)
    ctx.close()
    assert torch.equal(whole["codes"][:40], part["codes"])


@pytest.mark.parametrize("rows,n,heads,kw", [(4096, 2950, 64, dict(bits=2, block=16)), (2112, 2948, 33, dict(bits=8, block=64))])
def test_channels_without_deviation(lib, rows, n, heads, kw):
    """Rows of R that are zero, beside others of 1e-13: what the weights are in those channels does not count in the products with R."""
    g = torch.Generator(device="cuda").manual_seed(rows * 3 + n)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)  # noqa: E731
    dh, T = rows // heads, 4096
    X = 1e-8 * (rnd(T, n) + 0.5 * rnd(T, 1)).double()
    dev = 1e-8 * rnd(T, n).double()
    dev[:, ::31] = 0.0
    Hin, R = (X.T @ X).float(), (0.0125 * (dev.T @ X)).float().contiguous()
    W = 0.02 * rnd(rows, n)
    G = rnd(heads, 512, dh)
    Hout = torch.matmul(G.transpose(1, 2).contiguous(), G).contiguous()
    ctx = lib.Context()
    whole = ctx.quantize_layer(W, Hin, Hout, R, heads, **kw)
    part = ctx.quantize_layer(W[:dh].contiguous(), Hin, Hout[:1].contiguous(), R, 1, **kw)
    ctx.close()
    assert torch.equal(whole["codes"][:dh], part["codes"])
    (a, ac), (b, bc) = whole["loss_per_head_terms"][0], part["loss_per_head_terms"][0]
    assert abs(a - b) <= 2.0 ** -40 * b and abs(ac - bc) <= 2.0 ** -38 * abs(bc)
