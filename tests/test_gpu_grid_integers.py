"""The integer form of the grid search's products (2 bits, 3 bits up to 2048 columns): products of bytes by digits against 64-bit sums, at the edges of its
256-column padding and of its two and three digits, through layers whose results must be those of exact costs (GPU)."""
import numpy as np
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


def test_a_row_whose_costs_the_integers_do_not_resolve(lib):
    """H = 1 1^T + 2^-23 I, whose rows of T' are all off by the same factor: a row is made (on the CPU, with the costs of T') of which two candidates cost next to nothing,
    the dearer of them less than nothing by its approximation.  What is so far off is no row on a candidate's grid: the call goes to exact costs."""
    n, rng = 4096, np.random.default_rng(0)
    v = np.maximum(3.0 * np.arange(n) / (2147483000.0 - 1.5 * n), 1.0 / 8.3e6)
    T = np.rint(1.0 / v) * v

    def costs(w):      # of T', of H, and the sums of delta
        lo, hi, p = min(w.min(), 0.0), max(w.max(), 0.0), 1.0 - np.arange(80) / 100.0
        s = (p * hi - p * lo) / 3.0
        z = np.rint(-(p * lo) / s)
        d = s[:, None] * (np.clip(np.rint(w / s[:, None]) + z[:, None], 0, 3) - z[:, None]) - w
        before, sq = np.cumsum(d, 1) - d, (1.0 + 2.0 ** -23) * d * d
        return (2 * d * T * before + sq).sum(1), (2 * d * before + sq).sum(1), d.sum(1)

    def draw():
        return (0.02 * rng.standard_normal(n)).astype(np.float32).astype(np.float64)

    def misled():
        while True:
            w = draw()
            sums = costs(w)[2]
            order = np.argsort(sums)
            for g in np.argsort(np.diff(sums[order]))[:6]:
                if abs(sums[order[g]]) > 0.08: continue
                for f in (0.0, 0.25, 0.5, 0.75, 1.0):
                    u, c = w.copy(), np.argsort(np.abs(w))[n // 4: 3 * n // 4]
                    for _ in range(3):      # every sum falls by the same as long as no code changes
                        sums_u = costs(u)[2]
                        u[c] += (sums_u[order[g]] * f + sums_u[order[g + 1]] * (1 - f)) / len(c)
                        u = u.astype(np.float32).astype(np.float64)
                    a, e, _ = costs(u)
                    if a.min() < 0 and a.argmin() != e.argmin() and a[e.argmin()] > 0: return u
    rows = []
    while len(rows) < 15:      # rows that the integers resolve
        w = draw()
        if np.sort(costs(w)[1])[0] > 2e-3: rows.append(w)
    rows.insert(3, misled())
    W = torch.from_numpy(np.stack(rows).astype(np.float32)).cuda()
    H = torch.ones(n, n, device="cuda")
    H.diagonal().add_(2.0 ** -23)
    ctx = lib.Context()
    fast = ctx.quantize_layer(W, H, None, None, 1, 2, 16, damp=0.0)
    assert ctx.counter(0) > 0
    exact = ctx.quantize_layer(W, H, None, None, 1, 2, 16, damp=0.0, grid_guard=-1.0)
    for k in ("codes", "scales", "zeros", "W_deq"):
        assert torch.equal(fast[k], exact[k]), k
    assert ctx.counter(1) == 1
    ctx.close()
