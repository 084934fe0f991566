"""Hessians of a linear layer whose sums over the tokens are folded in registers: edges of the tiles, both operand layouts, lengths that are no
multiple of the fold, against torch in 64 bits; and inputs that are not finite (GPU)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tokens,d_in", [(2000, 1800), (2000, 1808), (1024, 4096), (4104, 2056), (1536, 3088)])
def test_against_64_bits(lib, tokens, d_in):
    ctx = lib.Context()
    g = torch.Generator(device="cuda"); g.manual_seed(tokens + d_in)
    xf = torch.randn(tokens, d_in, generator=g, device="cuda") * (1 + 20 * (torch.arange(d_in, device="cuda") % 97 == 0))
    X, Xf = (xf + 0.05 * torch.randn(tokens, d_in, generator=g, device="cuda")).bfloat16(), xf.bfloat16()
    H, R = ctx.build_hessian_linear(X, Xf, 0.25)
    a, d = X.double(), X.double() - Xf.double()
    # entry by entry, the worst case: a sum of at most 32 x 32 products is taken in fp32 (one rounding per product at most), the pair (hi, lo) of the difference
    # holds 16 bits of it; the folded sums and the result round once more each
    for got, l, r, scale, rep in ((H, a, a, 1.0, 0.0), (R, d, a, 0.25, 2.0 ** -16)):
        bound = scale * (1040 * 2.0 ** -24 + rep) * (l.abs().T @ r.abs())
        assert bool(((got.double() - scale * (l.T @ r)).abs() <= bound).all())
    assert torch.equal(H, H.T)
    H2, R2 = ctx.build_hessian_linear(X, Xf, 0.25)
    assert torch.equal(H, H2) and torch.equal(R, R2)
    ctx.close()


def test_not_finite(lib):
    """What is infinite or undefined in the sum of 64 bits, rounded to 32, is so here, and nothing else."""
    ctx = lib.Context()
    g = torch.Generator(device="cuda"); g.manual_seed(5)
    X = torch.randn(2048, 2048, generator=g, device="cuda").bfloat16()
    X[1500, 7] = float("inf"); X[3, 900] = float("nan"); X[10, 40] = 3e38
    H, _ = ctx.build_hessian_linear(X)
    want = (X.double().T @ X.double()).float()
    assert torch.equal(torch.isfinite(H), torch.isfinite(want)) and torch.equal(torch.isnan(H), torch.isnan(want))
    ctx.close()


@pytest.mark.parametrize("tokens,d_in", [(8192, 4096), (16384, 4096), (8192, 4104), (4096, 5136)])
def test_running_sums_of_one_sign_lose_nothing(lib, tokens, d_in):
    """Positive whole numbers of which 512 products, and the remainders of the running sums with them, stay below 2^24 in sum (the sums of 1024 do not): nothing
    is rounded but the result."""
    ctx = lib.Context()
    g = torch.Generator(device="cuda"); g.manual_seed(tokens)
    x = torch.randint(128, 181, (tokens, d_in), generator=g, device="cuda").double()
    dev = torch.randint(128, 181, (tokens, d_in), generator=g, device="cuda").double()
    H, R = ctx.build_hessian_linear(x.bfloat16(), (x - dev).bfloat16(), 0.25)
    assert torch.equal(H, (x.T @ x).float()) and torch.equal(R, (0.25 * (dev.T @ x)).float())
    ctx.close()


def test_a_chunk_larger_than_the_running_sum(lib):
    """0.5, then 2^24, then 0.75, 512 tokens apart: the fold of the larger chunk may lose one rounding of it (2^-24 of 2^24), and the result rounds."""
    ctx = lib.Context()
    x = torch.zeros(8192, 4096, device="cuda", dtype=torch.float64)
    x[[0, 512, 1024], 7] = torch.tensor([0.5, 4096.0, 0.75], device="cuda", dtype=torch.float64)
    x[[0, 512, 1024], 3] = torch.tensor([1.0, 4096.0, 1.0], device="cuda", dtype=torch.float64)
    H, _ = ctx.build_hessian_linear(x.bfloat16())
    want = x.T @ x
    assert float(want[7, 3]) == 2.0 ** 24 + 1.25 and abs(float(H[7, 3]) - float(want[7, 3])) <= 1.0 + 1.0
    want[7, 3] = want[3, 7] = float(H[7, 3])
    assert torch.equal(H, want.float())
    ctx.close()
