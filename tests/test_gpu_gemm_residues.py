"""fp64 products on the integer matrix cores (residues modulo 15 numbers) against numpy in extended precision, and exactly where nothing is rounded.

Tolerance: the operands are rounded to integers below 2^57 and 2^58 of their rows' 2-norms (2^56 and 2^57 at least), half a unit an entry: 0.75 sqrt(K) 2^-56 |a| |b| at most, and, the roundings
being independent, 0.65 x 2^-57 |a| |b| as root mean square; every entry is compared with 2^-54 |a| |b| (12 times that) + 2^-52 |c|."""
import os
import re

import numpy as np
import pytest
import torch

SOURCE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_04929_amd", "csrc", "gemm_rns.hip")
MODULI = [int(m) for m in re.search(r"MODULI\[NMAX\] = \{([^}]*)\}", open(SOURCE).read()).group(1).split(",")]

# tile edges +- 1, one element, contractions of one turn of the LDS ring, less and a little more, several turns, past 4096 (residues of long sums), several rounds of tiles
CASES = [(1, 1, 1), (16, 16, 256), (255, 257, 255), (257, 255, 257), (300, 520, 1000), (64, 700, 4096), (256, 256, 8200), (1025, 1030, 300)]


def operands(M, N, K, kind, rng):
    a, b = rng.standard_normal((M, K)), rng.standard_normal((K, N))
    if kind == "spread":      # rows and columns of very different size, some of them zero
        a *= 10.0 ** rng.integers(-120, 120, (M, 1)); b *= 10.0 ** rng.integers(-150, 100, (1, N))
        a[0] = 0.0; b[:, -1] = 0.0
    elif kind == "one_sign":
        a, b = np.abs(a), np.abs(b)
    elif kind == "equal":      # every product of the sum alike
        a = np.where(rng.random((M, K)) < 0.5, 1.0, 1.0 + 2.0 ** -52); b = np.full((K, N), 2.0 ** 30 - 1.0)
    return a, b


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["normal", "spread", "one_sign", "equal"])
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


def extreme_row(K, bits, sign, rng):
    """K integers (as floats, exact) of a row with 2-norm in [2^(bits - 1), 2^bits), which is taken as it is, whose residues modulo 256, 239, 237, 235 and 233 are the largest there are: -128 and
    (m - 1) / 2, or its negative; sign: +1, -1, or 0 for either at random."""
    big = MODULI[:5]
    assert big == [256, 239, 237, 235, 233]
    P = int(np.prod([int(m) for m in big], dtype=object))
    low = {}
    for s in (1, -1):
        x = 0
        for m in big:
            r = 128 if m == 256 else s * (m - 1) // 2 if s > 0 else -((m - 1) // 2)
            q = P // m
            x += r * q * pow(q, -1, m)
        low[s] = x % P
    top = int(2.0 ** bits / np.sqrt(K))
    out = []
    for _ in range(K):
        s = sign or int(rng.choice([1, -1]))
        j = int(rng.integers(int(0.72 * top) // P + 1, int(0.98 * top) // P))
        out.append(j * P + low[s] if rng.random() < 0.5 else -(j * P) + low[s])
    norm2 = sum(v * v for v in out)
    assert 4 ** (bits - 1) <= norm2 < 4 ** bits and all(abs(v) < 2 ** 53 for v in out)
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("K", [4096, 4097, 8192, 32768])
def test_largest_residues(lib, K):
    """Operands that are not rounded, with residues at their largest in the largest moduli and sums of one sign, of the other and mixed: 4096 terms are the most without the correction
    step, 4097 the fewest with it, 32768 the longest contraction.  The product is exact but for the result's rounding; one residue off by one would show as 2^-8 of 2^115."""
    rng = np.random.default_rng(K)
    a, b = ([extreme_row(K, bits, s, rng) for s in (1, -1, 0)] for bits in (57, 58))
    ctx = lib.Context()
    to = lambda x: torch.tensor(np.array(x, dtype=np.float64)).cuda()  # noqa: E731
    got = ctx.gemm_f64_residues(to(a), to(b), transB=True).cpu().numpy()
    ctx.close()
    for i in range(3):
        for j in range(3):
            want = sum(x * y for x, y in zip(a[i], b[j]))
            assert abs(int(got[i, j]) - want) <= 2.0 ** -52 * abs(want) + 2.0 ** 40, (i, j)


@pytest.mark.parametrize("terms", [4096, 65536])
def test_quotients_of_the_longest_sums(terms):
    """The epilogue's steps in float32 on the host, at and near the largest sums that `terms` products of residues can have and at random ones: a byte that is the sum's residue, with the correction
    step for sums of more than 4096 terms (two operands of 32768: 65536)."""
    rng = np.random.default_rng(terms)
    magic = np.float32(12582912.0)
    for m in MODULI[1:]:
        top = terms * (m // 2) ** 2
        acc = np.unique(np.concatenate([np.arange(top - 3 * m, top + 1), -np.arange(top - 3 * m, top + 1), np.arange(-2 * m, 2 * m + 1), rng.integers(-top, top + 1, 200000)])).astype(np.int64)
        inv = np.float32(1.0) / np.float32(m)
        # a fused multiply-add of 24-bit factors is exact in float64 before it is rounded
        q = (acc.astype(np.float32).astype(np.float64) * np.float64(inv) + np.float64(magic)).astype(np.float32)
        n = q.view(np.int32).astype(np.int64)
        n24 = ((n & 0xffffff) ^ 0x800000) - 0x800000      # the 24 bits that __mul24 takes, signed
        v = acc - n24 * m
        assert (np.abs(v + m * (1 << 22)) < 2 * m).all()
        if terms > 4096:
            v = v + m * (1 << 22)
            v = np.where(v < -128, v + m, v)
            v = np.where(v > 127, v - m, v)
        else:
            assert (v + m * (1 << 22) >= -128).all() and (v + m * (1 << 22) <= 127).all()
        byte = ((v & 0xff) ^ 0x80) - 0x80
        assert ((byte - acc) % m == 0).all()


@pytest.mark.gpu
def test_rows_that_are_not_finite(lib):
    a, b = np.ones((40, 64)), np.ones((64, 50))
    a[3, 5], a[17, 0], b[60, 49] = np.nan, np.inf, np.nan
    ctx = lib.Context()
    got = ctx.gemm_f64_residues(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()).cpu().numpy()
    bad = np.zeros((40, 50), bool)
    bad[[3, 17]] = True; bad[:, 49] = True
    assert np.isnan(got[bad]).all() and (got[~bad] == 64.0).all()
    ctx.close()


@pytest.mark.gpu
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
