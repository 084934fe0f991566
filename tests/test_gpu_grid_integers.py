"""The integer form of the grid search's products (2 bits, 3 bits up to 2048 columns): products of bytes by digits against 64-bit sums, at the edges of its
256-column padding and of its two and three digits, through layers whose results must be those of exact costs (GPU)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def layer(n, rows, seed, kind):
    g = torch.Generator(device="cuda"); g.manual_seed(seed)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda", dtype=torch.float64)
    x = rnd(2 * n, n)
    if kind == "factors":          # a few common factors: costs far below the trace
        x = x + 3.0 * rnd(2 * n, 4) @ rnd(4, n)
    elif kind == "one channel":    # one channel holds nearly all of the variance
        x[:, n // 3] *= 3e3
    elif kind == "signs":          # entries of T of one sign and one size: the sums that the step of a row has to bound
        x = 1.0 + 1e-2 * x
    return (rnd(rows, n) * 0.02).float(), (x.T @ x).float()


@pytest.mark.parametrize("kind", ["independent", "factors", "one channel", "signs"])
@pytest.mark.parametrize("bits,n,rows", [(2, 256, 16), (2, 511, 33), (2, 513, 130), (3, 768, 40), (3, 2048, 20), (2, 3000, 24)])
def test_equals_exact(lib, bits, n, rows, kind):
    W, H = layer(n, rows, n + bits, kind)
    ctx = lib.Context()
    fast = ctx.quantize_layer(W, H, None, None, 1, bits, rows)
    assert ctx.counter(0) > 0 and ctx.counter(1) == 0 and ctx.counter(6) == 0
    exact = ctx.quantize_layer(W, H, None, None, 1, bits, rows, grid_guard=-1.0)
    for k in ("codes", "scales", "zeros", "W_deq"):
        assert torch.equal(fast[k], exact[k]), k
    ctx.close()


@pytest.mark.parametrize("block", [4, 15, 16])
def test_few_rows_a_step(lib, block):
    """Steps of fewer than 16 rows take exact costs at once; the results are those of either."""
    W, H = layer(320, 32, 3, "independent")
    ctx = lib.Context()
    Ho = torch.eye(32, device="cuda")[None] * 2 + 0.1
    fast = ctx.quantize_layer(W, H, Ho, None, 1, 2, block)
    assert (ctx.counter(0) > 0) == (block >= 16)
    exact = ctx.quantize_layer(W, H, Ho, None, 1, 2, block, grid_guard=-1.0)
    for k in ("codes", "scales", "zeros", "W_deq"):
        assert torch.equal(fast[k], exact[k]), k
    ctx.close()


@pytest.mark.parametrize("bits,n", [(2, 320), (3, 768)])
def test_rows_that_lie_on_a_candidate_s_grid(lib, bits, n):
    """A row on a grid, a constant row and a row of a single weight, sampled by the guard (every eighth row) and not, among ordinary rows: the least cost of such a row is
    rounding, which its approximation does not resolve.  Its candidates get exact costs; the layer is not run again."""
    W, H = layer(n, 64, n, "independent")
    q = torch.randint(0, 2 ** bits, (2, n), device="cuda", generator=torch.Generator(device="cuda").manual_seed(1)); q[:, 0] = 0; q[:, 1] = 2 ** bits - 1
    W[[8, 13]] = (q - 1).float() * 0.0123
    W[16] = 0.0457
    W[24] = 0; W[24, n // 2] = -0.031
    W[37] = 0; W[37, 5] = 0.77
    ctx = lib.Context()
    fast = ctx.quantize_layer(W, H, None, None, 1, bits, 64)
    assert ctx.counter(0) == 1 and ctx.counter(1) == 0 and ctx.counter(6) == 0
    exact = ctx.quantize_layer(W, H, None, None, 1, bits, 64, grid_guard=-1.0)
    for k in ("codes", "scales", "zeros", "W_deq"):
        assert torch.equal(fast[k], exact[k]), k
    ctx.close()


@pytest.mark.parametrize("guard,again", [(0.0, 0), (0.25, 0), (0.5, 0), (0.125, 1)])
def test_the_guard_is_the_caller_s(lib, guard, again):
    """One direction holds nearly all of the variance and little damping hides it: the largest deviation of this layer's approximate costs lies between 2.5e-4 and
    5e-4, which a guard of 0.25 (the default) or more lets pass and one of 0.125 does not.  The results are those of exact costs."""
    g = torch.Generator(device="cuda"); g.manual_seed(1)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda", dtype=torch.float64)
    x = 1.0 + 1e-2 * rnd(1024, 512)
    W, H = (rnd(64, 512) * 0.02).float(), (x.T @ x).float()
    ctx = lib.Context()
    fast = ctx.quantize_layer(W, H, None, None, 1, 2, 64, damp=1e-6, grid_guard=guard)
    assert ctx.counter(0) > 0 and ctx.counter(1) + ctx.counter(6) == again
    exact = ctx.quantize_layer(W, H, None, None, 1, 2, 64, damp=1e-6, grid_guard=-1.0)
    for k in ("codes", "scales", "zeros", "W_deq"):
        assert torch.equal(fast[k], exact[k]), k
    ctx.close()


@pytest.mark.parametrize("bits,tokens", [(2, 16384), (3, 65536)])
def test_two_digits_only_where_one_half_term_did(lib, bits, tokens):
    """Independent channels over so many tokens that two digits would be off by no more than 6e-7 by expectation, but too few for one half term of H_in: costs from pairs of
    half terms are within 2.4e-7 of the exact ones, from two digits 5e-7 - 1e-6, from three, which are taken, 2e-8."""
    g = torch.Generator(device="cuda"); g.manual_seed(1024 + bits)
    x = torch.randn(tokens, 1024, generator=g, device="cuda", dtype=torch.float64)
    W, H = (torch.randn(64, 1024, generator=g, device="cuda") * 0.02), (x.T @ x).float()
    ctx = lib.Context()
    ctx.quantize_layer(W, H, None, None, 1, bits, 64, grid_guard=2.4e-7 / 2e-3)
    assert ctx.counter(0) == 1 and ctx.counter(1) == 0 and ctx.counter(6) == 0
    ctx.close()
