"""fp64 GEMM over the tile shapes and contraction splits its dispatch chooses from, against numpy in fp64.

Tolerance: a dot product of K terms of N(0, 1) factors accumulated in any order stays within K * 2^-53 * sum |a b| <= K^2 2^-53 of the
exact value; 1e-13 relative to the result's norm covers K <= 4100 with a wide margin (observed 3e-15)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# (batch, M, N, K): one tile and long contractions (split), tile edges +- 1, a row count of the skinny shape, many tiles, an odd
# pitch (no 16-byte loads), a contraction that is no whole step, an empty one
CASES = [(1, 128, 128, 4096), (8, 128, 128, 1024), (1, 129, 127, 515), (2, 64, 64, 32), (1, 65, 63, 33), (3, 32, 256, 96), (2, 31, 130, 1000),
         (1, 33, 33, 2050), (1, 1, 1, 1), (1, 7, 300, 64), (1, 1000, 1000, 250), (1, 500, 501, 77), (40, 128, 128, 128), (1, 600, 1300, 256), (1, 20, 20, 0)]


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_gemm_f64_shapes(lib, case, ta, tb):
    b, M, N, K = case
    rng = np.random.default_rng(b * 7919 + M * 31 + N * 17 + K)
    A = rng.standard_normal((b, K, M) if ta else (b, M, K)); B = rng.standard_normal((b, N, K) if tb else (b, K, N))
    C0 = rng.standard_normal((b, M, N))
    ctx = lib.Context()
    dev = lambda x: torch.from_numpy(x).cuda()
    if K == 0:      # the binding derives the strides from the shapes: an empty operand still needs an address
        A = np.zeros((b, 1, M) if ta else (b, M, 1)); B = np.zeros((b, N, 1) if tb else (b, 1, N))
    ref = (np.swapaxes(A, 1, 2) if ta else A) @ (np.swapaxes(B, 1, 2) if tb else B)
    got = ctx.gemm_f64(dev(A), dev(B), transA=bool(ta), transB=bool(tb)).cpu().numpy()
    tol = 1e-13 * max(np.linalg.norm(ref), 1.0)
    assert np.linalg.norm(got - ref) <= tol
    acc = dev(C0)
    ctx.gemm_f64(dev(A), dev(B), acc, alpha=-0.5, beta=2.0, transA=bool(ta), transB=bool(tb))
    want = 2.0 * C0 - 0.5 * ref
    assert np.linalg.norm(acc.cpu().numpy() - want) <= 1e-13 * np.linalg.norm(want) + tol
    ctx.close()


@pytest.mark.parametrize("rep,dh,d", [(8, 128, 1024), (3, 100, 520), (1, 64, 4096), (5, 33, 65)])
def test_hout_sums_the_heads_of_a_group(lib, rep, dh, d):
    """build_hout adds the d_h x d_h products of a group's heads in one launch."""
    rng = np.random.default_rng(rep * 100 + dh)
    X = rng.standard_normal((2 * d, d)); H = (X.T @ X).astype(np.float32)
    nh = 3
    W = (0.02 * rng.standard_normal((nh * rep * dh, d))).astype(np.float32)
    ctx = lib.Context()
    got = ctx.build_hout(torch.from_numpy(H).cuda(), torch.from_numpy(W).cuda(), nh, rep, dh).cpu().numpy().astype(np.float64)
    W64 = W.astype(np.float64).reshape(nh, rep, dh, d)
    want = np.stack([sum(W64[g, r] @ H.astype(np.float64) @ W64[g, r].T for r in range(rep)) for g in range(nh)])
    assert np.abs(got - want).max() <= 2.0 ** -23 * np.abs(want).max()      # the rounding of the fp32 result
    ctx.close()


# (M, N, K): one 128 x 128 tile that smaller shapes would cut into several rows or columns, and several such tiles
@pytest.mark.parametrize("M,N,K", [(64, 20, 64), (128, 64, 128), (128, 128, 128), (200, 200, 200), (300, 20, 300), (20, 300, 20), (1, 1, 1), (33, 65, 40)])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_result_over_an_operand(lib, M, N, K, ta, tb):
    """C in the place of A, of B, of both, and in a buffer that begins inside an operand: the product of the operands as they were."""
    rng = np.random.default_rng(M * 31 + N * 17 + K)
    a, b = rng.standard_normal((K, M) if ta else (M, K)), rng.standard_normal((N, K) if tb else (K, N))
    want = (a.T if ta else a) @ (b.T if tb else b)
    tol = 1e-13 * np.linalg.norm(want)
    ctx = lib.Context()
    buf = torch.empty(max(M * K, K * N) + M * N, dtype=torch.float64, device="cuda")

    def run(over, at):
        A, B = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
        op = A if over == "A" else B
        o = buf[:op.numel()].view(op.shape); o.copy_(op)
        C = buf[at:at + M * N].view(M, N)
        ctx.gemm_f64(o if over == "A" else A, o if over == "B" else B, C, transA=bool(ta), transB=bool(tb))
        assert np.linalg.norm(C.cpu().numpy() - want) <= tol, (over, at)
    for over, size in (("A", M * K), ("B", K * N)):
        run(over, 0)
        run(over, size // 3)
    ctx.close()


@pytest.mark.parametrize("bs,n", [(3, 40), (2, 150)])
def test_batched_result_over_an_operand(lib, bs, n):
    rng = np.random.default_rng(n)
    a, b = rng.standard_normal((bs, n, n)), rng.standard_normal((bs, n, n))
    ctx = lib.Context()
    for over in (0, 1):
        for beta in (0.0, 0.5):
            ops = [torch.from_numpy(x).cuda() for x in (a, b)]
            ctx.gemm_f64(ops[0], ops[1], ops[over], alpha=2.0, beta=beta)
            want = 2.0 * a @ b + beta * (a, b)[over]
            assert np.linalg.norm(ops[over].cpu().numpy() - want) <= 1e-13 * np.linalg.norm(want)
    sq = torch.from_numpy(a).cuda()
    ctx.gemm_f64(sq, sq, sq)
    assert np.linalg.norm(sq.cpu().numpy() - a @ a) <= 1e-13 * np.linalg.norm(a @ a)
    ctx.close()


def test_tall_result_in_the_place_of_A(lib):
    """More elements than the parts hold, row for row over A: the rows' own workgroups, bits as in a buffer of its own."""
    g = torch.Generator(device="cuda"); g.manual_seed(1)
    A = torch.randn(40000, 128, dtype=torch.float64, device="cuda", generator=g); B = torch.randn(128, 128, dtype=torch.float64, device="cuda", generator=g)
    ctx = lib.Context()
    want = ctx.gemm_f64(A, B)
    ctx.gemm_f64(A, B, A)
    assert torch.equal(A, want)
    ctx.close()


@pytest.mark.parametrize("M,N,K", [(65535 * 32 + 1, 3, 256), (65535 * 64 + 5, 40, 80)])
def test_more_rows_than_small_tiles_can_have(lib, M, N, K):
    """A launch has at most 65535 rows of tiles: from there on the tile must be the one of 128 rows."""
    g = torch.Generator(device="cuda"); g.manual_seed(N)
    A = torch.randn(M, K, dtype=torch.float64, device="cuda", generator=g); B = torch.randn(K, N, dtype=torch.float64, device="cuda", generator=g)
    ctx = lib.Context()
    got = ctx.gemm_f64(A, B)
    for rows in (slice(0, 1000), slice(M // 2, M // 2 + 1000), slice(M - 1000, M)):
        want = A[rows].cpu().numpy() @ B.cpu().numpy()
        assert np.linalg.norm(got[rows].cpu().numpy() - want) <= 1e-13 * np.linalg.norm(want)
    ctx.close()


def test_hout_sums_that_fit_no_launch_or_no_buffer(lib):
    """More terms than a launch has batch entries, and partial products that do not fit their buffer (15 of 530 x 530): the terms one after the other."""
    ctx = lib.Context()
    for nh, rep, dh, d in ((16384, 8, 1, 4), (3, 5, 530, 40)):
        g = torch.Generator(device="cuda"); g.manual_seed(rep)
        X = torch.randn(2 * d, d, dtype=torch.float64, device="cuda", generator=g); H = (X.T @ X).float()
        W = 0.02 * torch.randn(nh * rep * dh, d, device="cuda", generator=g)
        got = ctx.build_hout(H, W, nh, rep, dh).double()
        w = W.double().view(nh, rep * dh, d)
        y = (w @ H.double()).view(nh, rep, dh, d)
        want = torch.stack([y[:, r] @ w.view(nh, rep, dh, d)[:, r].transpose(1, 2).contiguous() for r in range(rep)]).sum(0)
        assert float((got - want).abs().max()) <= 2.0 ** -23 * float(want.abs().max())      # the rounding of the fp32 result
    ctx.close()
