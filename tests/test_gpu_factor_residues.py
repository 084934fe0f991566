"""chol_inv_upper where its updates run as products of residues: several outer blocks of 512 columns, the last one whole, ragged or a single column; channels of very different size,
whose columns of U outgrow their first power of two.

Tolerance: the factors of order n of a matrix with condition number c leave U H U^T - I within a few n 2^-53 c of zero (c ~ 1e3 .. 1e7 here after scaling of the channels; the
fp64 form leaves the same); compared with torch's factorisation in fp64 on the same matrices, which may be off by as much."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,batch", [(2049, 3), (2100, 3), (2304, 2), (3072, 1), (3100, 2)])
@pytest.mark.parametrize("kind", ["plain", "spread", "correlated"])
def test_factor_by_residues(lib, n, batch, kind):
    g = torch.Generator(device="cuda").manual_seed(n + batch)
    H = torch.empty(batch, n, n, device="cuda")
    for b in range(batch):
        x = torch.randn(2 * n, n, generator=g, device="cuda", dtype=torch.float64)
        if kind == "spread":
            x *= 10.0 ** torch.randint(-4, 5, (n,), generator=g, device="cuda")
        elif kind == "correlated":
            x += 20 * torch.randn(2 * n, 1, generator=g, device="cuda", dtype=torch.float64) * torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
        H[b] = (x.T @ x).float()
    ctx = lib.Context()
    U = ctx.chol_inv_upper(H)
    ctx.close()
    assert torch.isfinite(U).all() and (U.tril(-1) == 0).all()
    eye = torch.eye(n, dtype=torch.float64, device="cuda")
    for b in range(batch):
        h = H[b].double()
        h = h.triu() + h.triu(1).T
        s = h.diagonal().sqrt()
        hs = h / s[:, None] / s[None]                                     # unit diagonal: U diag(s) is its factor
        us = U[b] * s[None]
        v = torch.linalg.cholesky(hs.flip(0, 1)).flip(0, 1)
        want = torch.linalg.solve_triangular(v, eye, upper=True)
        cond = float(torch.linalg.norm(want)) ** 2 / n * float(torch.linalg.matrix_norm(hs, 2))
        assert (us @ hs @ us.T - eye).abs().max() <= 64 * 2.0 ** -53 * cond * n ** 0.5
        assert torch.linalg.norm(us - want) <= 64 * 2.0 ** -53 * cond * torch.linalg.norm(want)


def test_breakdown_is_reported(lib):
    n = 3100
    H = torch.eye(n, device="cuda")
    H[700, 700] = -1.0
    ctx = lib.Context()
    with pytest.raises(lib.TurboBoAError, match="pivot 700 is not positive"):
        ctx.chol_inv_upper(H)
    ctx.close()
