"""fp64 products on the integer matrix cores (residues modulo 15 numbers) against numpy in extended precision.

Tolerance: the operands are rounded to integers below 2^57 and 2^58 of their rows' 2-norms, which leaves at most 2^-56 |a| |b| sqrt(K) in the worst case and, the roundings being
independent, 2^-56 |a| |b| as bound for a typical entry; every entry is compared with 2^-54 |a| |b| + 2^-52 |c|."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# tile edges +- 1, one element, contractions of one turn of the LDS ring, less and a little more, several turns, past 4096 (residues of long sums), several rounds of tiles
CASES = [(1, 1, 1), (16, 16, 256), (255, 257, 255), (257, 255, 257), (300, 520, 1000), (64, 700, 4096), (256, 256, 8200), (1025, 1030, 300)]


def operands(M, N, K, kind, rng):
    a, b = rng.standard_normal((M, K)), rng.standard_normal((K, N))
    if kind == "spread":      # rows and columns of very different size, some of them zero
        a *= 10.0 ** rng.integers(-120, 120, (M, 1)); b *= 10.0 ** rng.integers(-150, 100, (1, N))
        a[0] = 0.0; b[:, -1] = 0.0
    elif kind == "one_sign":
        a, b = np.abs(a), np.abs(b)
    elif kind == "extreme":      # every residue at its largest, sums of one sign
        a = np.where(rng.random((M, K)) < 0.5, 1.0, 1.0 + 2.0 ** -52); b = np.full((K, N), 2.0 ** 30 - 1.0)
    return a, b


@pytest.mark.parametrize("kind", ["normal", "spread", "one_sign", "extreme"])
@pytest.mark.parametrize("M,N,K", CASES)
def test_product_of_residues(lib, M, N, K, kind):
    rng = np.random.default_rng(M * 31 + N * 17 + K)
    a, b = operands(M, N, K, kind, rng)
    c0 = rng.standard_normal((M, N))
    ctx = lib.Context()
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    rows = np.unique(np.concatenate([np.arange(min(M, 4)), np.arange(max(0, M - 4), M), rng.integers(0, M, 4)]))
    al, bl = a[rows].astype(np.longdouble), b.astype(np.longdouble)
    want = (al @ bl)
    bound = np.sqrt((al ** 2).sum(1))[:, None] * np.sqrt((bl ** 2).sum(0))[None]
    for trans in (False, True):
        got = ctx.gemm_f64_residues(dev(a), dev(b.T if trans else b), transB=trans).cpu().numpy()[rows]
        assert np.all(np.abs(got - want) <= 2.0 ** -54 * bound + 2.0 ** -52 * np.abs(want))
    acc = dev(c0)
    ctx.gemm_f64_residues(dev(a), dev(b), acc, alpha=-0.5, beta=2.0)
    got, want2 = acc.cpu().numpy()[rows], 2.0 * c0[rows] - 0.5 * want
    assert np.all(np.abs(got - want2) <= 2.0 ** -54 * bound + 2.0 ** -51 * (np.abs(want) + np.abs(c0[rows])))
    ctx.close()


def test_rows_that_are_not_finite(lib):
    a, b = np.ones((40, 64)), np.ones((64, 50))
    a[3, 5], a[17, 0], b[60, 49] = np.nan, np.inf, np.nan
    ctx = lib.Context()
    got = ctx.gemm_f64_residues(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()).cpu().numpy()
    bad = np.zeros((40, 50), bool)
    bad[[3, 17]] = True; bad[:, 49] = True
    assert np.isnan(got[bad]).all() and (got[~bad] == 64.0).all()
    ctx.close()


def test_time_and_operations_have_a_tag_of_their_own(lib):
    """Launches are timed as products of residues, with the operations of the fp64 product, and not among the fp64 kernels'."""
    M, N, K = 300, 520, 1000
    ctx = lib.Context()
    a, b = (torch.randn(*s, device="cuda", dtype=torch.float64) for s in ((M, K), (K, N)))
    ctx.profile(True)
    ctx.gemm_f64_residues(a, b)
    got = {k: ctx.profile_read(k) for k in ctx.PROF_TAGS}
    ctx.profile(False)
    ctx.close()
    assert got["residues"]["launches"] == 1 and got["residues"]["ms"] > 0 and got["residues"]["flops"] == 2.0 * M * N * K
    assert all(v["launches"] == 0 for k, v in got.items() if k != "residues")
