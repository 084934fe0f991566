"""Factors of one diagonal block of 64 and its neighbours: every remainder of the 16 x 16 tiles, against an extended-precision factorisation, and the pivot
that is named where a matrix is not positive definite (GPU)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def reference(H):
    """U = V^-1 with H = V V^T, V upper, in long double."""
    n = H.shape[0]
    A, V, U = H.astype(np.longdouble), np.zeros((n, n), np.longdouble), np.zeros((n, n), np.longdouble)
    for c in range(n - 1, -1, -1):
        V[c, c] = np.sqrt(A[c, c]); V[:c, c] = A[:c, c] / V[c, c]
        A[:c, :c] -= np.outer(V[:c, c], V[:c, c])
    for r in range(n - 1, -1, -1):
        e = np.zeros(n, np.longdouble); e[r] = 1
        U[r] = (e - V[r, r + 1:] @ U[r + 1:]) / V[r, r]
    return U


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 33, 48, 63, 64, 65, 81, 128])
def test_against_extended_precision(lib, n):
    ctx = lib.Context()
    rng = np.random.default_rng(n)
    x = rng.standard_normal((3, 3 * n + 4, n)) * np.logspace(-2, 2, n)
    H = (x.transpose(0, 2, 1) @ x).astype(np.float32)
    U = ctx.chol_inv_upper(torch.tensor(H, device="cuda")).cpu().numpy()
    for b in range(3):
        want = reference(H[b].astype(np.float64))
        # backward stable: rows of U are off by a few n eps times the condition of the equilibrated matrix
        d = 1 / np.sqrt(np.diag(H[b].astype(np.float64)))
        bound = 8 * n * 2.0 ** -52 * np.linalg.cond(H[b].astype(np.float64) * d[:, None] * d[None, :])
        err = np.abs((U[b] - want).astype(np.float64)) / np.sqrt((want.astype(np.float64) ** 2).sum(1, keepdims=True)) / d[None, :] * d.min()
        assert err.max() <= bound and np.all(np.tril(U[b], -1) == 0)
    ctx.close()


@pytest.mark.parametrize("n,col", [(5, 0), (20, 3), (64, 40), (64, 63), (100, 70), (100, 10)])
def test_names_the_pivot(lib, n, col):
    """Columns are taken from the last to the first: the last one that is not positive is named."""
    ctx = lib.Context()
    H = torch.eye(n, device="cuda")[None].repeat(2, 1, 1)
    H[1, col, col] = -1.0
    H[1, 0, 0] = -2.0
    with pytest.raises(Exception, match=r"1 of the batch is not positive definite: pivot %d " % col):
        ctx.chol_inv_upper(H)
    ctx.close()
