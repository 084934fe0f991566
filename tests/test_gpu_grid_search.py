"""The two-phase grid search against the same layer with fp64 costs for every candidate (grid_guard < 0): same codes, scales and zeros,
and no call that had to be repeated.  The search returns the fp64 argmin either way, so nothing may differ; the widths sit at the
edges of the operands' 32-column padding and of the 256-tiles, the Hessians need one half term (independent channels) or two."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def layer(n, heads, dh, seed, corr, per_head, tokens=0):
    g = torch.Generator(device="cuda"); g.manual_seed(seed)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda", dtype=torch.float64)

    def hessian():
        x = rnd(tokens or 4 * n, n)
        x[:, torch.randperm(n, generator=g, device="cuda")[:4]] *= 20
        if corr:
            x = x + 0.3 * (x @ rnd(n, 4)) @ rnd(4, n)
        return (x.T @ x).float()
    H = torch.stack([hessian() for _ in range(heads)]) if per_head else hessian()
    k = rnd(heads, 3 * dh, dh)
    Ho = torch.stack([a.T @ a for a in k]).float().contiguous()
    return (rnd(heads * dh, n) * 0.02).float(), H, Ho


def same(a, b):
    for k in ("codes", "scales", "zeros", "W_deq"):
        assert torch.equal(a[k], b[k]), k


@pytest.mark.parametrize("corr", [0, 1])
@pytest.mark.parametrize("bits", [2, 3, 4, 8])
@pytest.mark.parametrize("n,heads,dh,per_head", [(256, 3, 20, 0), (257, 1, 33, 0), (288, 2, 16, 1), (300, 5, 30, 0), (511, 2, 24, 1), (544, 2, 24, 0), (1001, 1, 40, 0)])
def test_two_phase_search_equals_exact(lib, n, heads, dh, per_head, bits, corr):
    W, H, Ho = layer(n, heads, dh, n + bits, corr, per_head)
    ctx = lib.Context()
    fast = ctx.quantize_layer(W, H, Ho, None, heads, bits, 16)
    passes, again = ctx.counter(0), ctx.counter(1)
    assert passes > 0 and again == 0
    same(fast, ctx.quantize_layer(W, H, Ho, None, heads, bits, 16, grid_guard=-1.0))
    assert ctx.counter(0) == passes
    ctx.close()


@pytest.mark.parametrize("corr", [0, 1])
def test_a_guard_that_cannot_be_met_ends_in_exact_costs(lib, corr):
    """A guard below what any rounding gives: the call is run again (independent channels: with two half terms first, twice the passes) and at
    last exactly, once by the counter."""
    W, H, Ho = layer(320, 2, 32, 5, corr, 0, tokens=0 if corr else 160 * 320)      # (one term: independent channels over so many tokens)
    ctx = lib.Context()
    got = ctx.quantize_layer(W, H, Ho, None, 2, 2, 32, grid_guard=1e-12)
    assert ctx.counter(1) == 1 and ctx.counter(0) == (2 if not corr else 1)
    same(got, ctx.quantize_layer(W, H, Ho, None, 2, 2, 32, grid_guard=-1.0))
    ctx.close()


def test_channels_of_very_different_variance(lib):
    """Variances over 2^40: beyond the spread of the half exponents the small channels share one (their part of the cost is nothing)."""
    W, H, Ho = layer(320, 2, 32, 6, 0, 0)
    d = torch.logspace(-6, 6, 320, device="cuda", dtype=torch.float64)
    H = (H.double() * d[:, None] * d[None, :]).float()
    ctx = lib.Context()
    fast = ctx.quantize_layer(W, H, Ho, None, 2, 3, 32)
    same(fast, ctx.quantize_layer(W, H, Ho, None, 2, 3, 32, grid_guard=-1.0))
    ctx.close()


def test_rows_of_zeros(lib):
    """Every candidate of a row of zeros costs 0, approximately and exactly: no deviation, no run again; the first candidate wins as in the exact search."""
    W, H, _ = layer(320, 2, 32, 8, 0, 0, tokens=160 * 320)
    W[3] = 0; W[40] = 0
    ctx = lib.Context()
    fast = ctx.quantize_layer(W, H, None, None, 2, 2, 32)
    assert ctx.counter(1) == 0 and ctx.counter(6) == 0
    same(fast, ctx.quantize_layer(W, H, None, None, 2, 2, 32, grid_guard=-1.0))
    ctx.close()


def test_weights_on_a_grid_go_to_exact_costs_at_once(lib):
    """Weights that one candidate meets up to fp32 rounding: its cost is nothing but that rounding, which no number of terms of H brings out; one
    approximate run, then the exact one."""
    W, H, _ = layer(320, 2, 32, 9, 0, 0, tokens=160 * 320)
    q = torch.randint(0, 4, W.shape, device="cuda"); q[:, 0] = 0; q[:, 1] = 3
    W = (q - 1) * (0.01 + W.abs().amax(1, keepdim=True))
    ctx = lib.Context()
    got = ctx.quantize_layer(W, H, None, None, 2, 2, 32)
    assert ctx.counter(0) == 1 and ctx.counter(1) == 1 and ctx.counter(6) == 0
    same(got, ctx.quantize_layer(W, H, None, None, 2, 2, 32, grid_guard=-1.0))
    ctx.close()


def test_runs_with_two_terms_are_counted(lib):
    W, H, Ho = layer(320, 2, 32, 5, 0, 0, tokens=160 * 320)
    ctx = lib.Context()
    ctx.quantize_layer(W, H, Ho, None, 2, 2, 32, grid_guard=1e-12)
    assert ctx.counter(0) == 2 and ctx.counter(1) == 1 and ctx.counter(6) == 1
    ctx.close()


@pytest.mark.parametrize("bits", [2, 3, 4, 8])
@pytest.mark.parametrize("n,tokens", [(320, 1280), (1000, 2000), (1024, 32768)])
def test_approximate_costs_of_independent_channels(lib, bits, n, tokens):
    """Few tokens correlate independent channels by chance, and a cost takes up the rounding of H by that much.  Costs from (hi, lo) pairs of H are within 5e-6
    of the exact ones here; a guard at 1.5e-5 holds however many terms are taken."""
    W, H, _ = layer(n, 2, 32, n, 0, 0, tokens=tokens)
    ctx = lib.Context()
    ctx.quantize_layer(W, H, None, None, 2, bits, 32, grid_guard=1.5e-5 / 2e-3)
    assert ctx.counter(0) > 0 and ctx.counter(1) == 0 and ctx.counter(6) == 0
    ctx.close()


@pytest.mark.parametrize("bits", [2, 3, 4, 8])
@pytest.mark.parametrize("n,heads,dh,per_head", [(257, 1, 33, 0), (288, 2, 16, 1), (544, 2, 24, 0)])
def test_one_term_search_equals_exact(lib, n, heads, dh, per_head, bits):
    """Independent channels over many tokens: H_in as one half term (except with 8 bits)."""
    W, H, Ho = layer(n, heads, dh, n + bits, 0, per_head, tokens=200000)
    ctx = lib.Context()
    fast = ctx.quantize_layer(W, H, Ho, None, heads, bits, 16)
    assert ctx.counter(0) > 0 and ctx.counter(1) == 0 and ctx.counter(6) == 0
    same(fast, ctx.quantize_layer(W, H, Ho, None, heads, bits, 16, grid_guard=-1.0))
    ctx.quantize_layer(W, H, Ho, None, heads, bits, 16, grid_guard=1e-12)      # what cannot be met tells whether there was one term
    assert ctx.counter(6) == (bits != 8)
    ctx.close()


@pytest.mark.parametrize("bits", [3, 4, 8])
@pytest.mark.parametrize("seed", [1, 2])
def test_approximate_costs_of_fine_grids(lib, bits, seed):
    """Strongly correlated wide channels: costs from pairs of delta are within 1.5e-5 of the exact ones (22 bits on both sides, fp32 sums), those from codes
    and weights that are subtracted are off by 7e-5 and more; a guard at 4e-5 tells which it was."""
    W, H, _ = layer(2304, 4, 64, seed, 1, 0)
    ctx = lib.Context()
    ctx.quantize_layer(W, H, None, None, 4, bits, 64, grid_guard=4e-5 / 2e-3)
    assert ctx.counter(0) > 0 and ctx.counter(1) == 0 and ctx.counter(6) == 0
    ctx.close()


@pytest.mark.parametrize("n", [2048, 2049])
def test_both_operands_of_3_bits_equal_exact(lib, n):
    """The widths on either side of the rule that chooses codes or pairs of delta."""
    W, H, Ho = layer(n, 2, 16, n, 0, 0)
    ctx = lib.Context()
    fast = ctx.quantize_layer(W, H, Ho, None, 2, 3, 16)
    assert ctx.counter(0) > 0 and ctx.counter(1) == 0
    same(fast, ctx.quantize_layer(W, H, Ho, None, 2, 3, 16, grid_guard=-1.0))
    ctx.close()
