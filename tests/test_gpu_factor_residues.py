"""chol_inv_upper where its updates run as products of residues: several outer blocks of 512 columns, the last one whole, ragged or a single column; channels of very different size,
whose columns of U outgrow their first power of two.

Tolerance: the factors of order n of a matrix with condition number c leave U H U^T - I within a few n 2^-53 c of zero (c ~ 1e3 .. 1e7 here after scaling of the channels; the
fp64 form leaves the same); compared with torch's factorisation in fp64 on the same matrices, which may be off by as much."""
import math

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


@pytest.mark.parametrize("value", [1.5, 10.0, 12345.0, 3e6, 1e12, float("nan"), float("inf")])
@pytest.mark.parametrize("r,k", [(700, 2900), (3, 3099), (1500, 1530)])
def test_rows_longer_than_the_diagonal_says(lib, r, k, value):
    """A pivot that an entry beyond the diagonal's reach makes negative (or undefined), in a later block of 512 columns or the same one: refused, and named, whatever the residues hold."""
    n = 3100
    H = torch.eye(n, device="cuda")
    H[r, k] = H[k, r] = value
    H[r - 2, k - 1] = H[k - 1, r - 2] = 0.5
    ctx = lib.Context()
    with pytest.raises(lib.TurboBoAError, match="pivot %d is not positive" % r):
        ctx.chol_inv_upper(H)
    ctx.close()


@pytest.mark.parametrize("value", [0.0, -1e30])
def test_diagonal_entries_that_are_not_positive(lib, value):
    n = 3100
    H = torch.eye(n, device="cuda")
    H[40, 40] = value
    H[40, 2500] = H[2500, 40] = 1e12
    ctx = lib.Context()
    with pytest.raises(lib.TurboBoAError, match="pivot 40 is not positive"):
        ctx.chol_inv_upper(H)
    ctx.close()


@pytest.mark.parametrize("n,batch", [(1000, 1), (2048, 3), (3100, 2)])
def test_infinite_diagonal(lib, n, batch):
    """The damping, a share of the diagonal's mean, is infinite where an entry is: H + inf I is its diagonal alone and U is zero, in fp64 (orders below 2048) and with residues."""
    g = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randn(n + 100, n, generator=g, device="cuda")
    H = (x.T @ x)[None].repeat(batch, 1, 1)
    want = H.clone()
    H[-1, n // 2, n // 2] = math.inf
    ctx = lib.Context()
    U, rest = ctx.chol_inv_upper(H, damp=0.01), ctx.chol_inv_upper(want, damp=0.01)
    assert (U[-1] == 0.0).all() and torch.equal(U[:-1], rest[:-1])
    with pytest.raises(lib.TurboBoAError) as e:
        ctx.quantize_layer(0.02 * x[:64].contiguous(), H[-1].contiguous(), None, None, 1, bits=2, block=64)
    assert e.value.code == -5
    ctx.close()


def test_room_for_fp64_only(lib):
    """Residues take 30 bytes an element, more than the device has left: the factorisation and a layer run in fp64, as they would have without them."""
    n, batch = 2048, 96
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn(2 * n, n, generator=g, device="cuda")
    H = (x.T @ x)[None].repeat(batch, 1, 1)
    y = torch.randn(10000, 8192, generator=g, device="cuda")
    H1, W = y.T @ y, 0.02 * torch.randn(8192, 8192, generator=g, device="cuda")
    del y
    out = torch.empty(batch, n, n, dtype=torch.float64, device="cuda")
    for call in (lambda c: c.chol_inv_upper(H, out=out), lambda c: c.quantize_layer(W, H1, None, None, 1, bits=2, block=8192)["codes"]):
        ctx = lib.Context()
        want, need = call(ctx).clone(), ctx.workspace_bytes()
        ctx.close()
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        ballast = torch.empty(torch.cuda.mem_get_info()[0] - need + (4 << 30), dtype=torch.uint8, device="cuda")
        ctx = lib.Context()
        got = call(ctx)
        assert 0 < ctx.workspace_bytes() < need - (4 << 30)
        ctx.close()
        del ballast
        torch.cuda.empty_cache()
        if want.dtype == torch.float64:
            assert torch.linalg.norm(got - want) <= 1e-12 * torch.linalg.norm(want)
        else:
            assert torch.equal(got, want)


@pytest.mark.parametrize("n,batch", [(127, 33), (128, 32), (129, 31), (192, 22), (513, 9), (577, 8), (1000, 5), (1023, 4), (1100, 4), (1100, 3)])
def test_updates_inside_outer_blocks(lib, n, batch):
    """fp64 throughout: one update per diagonal block (rows x matrices from 4096 on) or one per finished block, in outer blocks of whole and ragged width."""
    g = torch.Generator(device="cuda").manual_seed(n * 7 + batch)
    x = torch.randn(batch, 2 * n, n, generator=g, device="cuda", dtype=torch.float64)
    H = torch.stack([(m.T @ m) for m in x]).float()
    ctx = lib.Context()
    U = ctx.chol_inv_upper(H)
    ctx.close()
    eye = torch.eye(n, dtype=torch.float64, device="cuda")
    for b in range(batch):
        h = H[b].double()
        h = h.triu() + h.triu(1).T
        assert (U[b].tril(-1) == 0).all()
        # condition numbers of 2n samples: below 40
        assert ((U[b] @ h) @ U[b].T - eye).abs().max() <= 64 * 2.0 ** -53 * 40 * n ** 0.5


def test_more_matrices_than_residues_hold(lib):
    """Residues of 64 matrices of order 2048 at a time: 65 go in two runs, and a breakdown names its matrix."""
    n = 2048
    g = torch.Generator(device="cuda").manual_seed(11)
    x = torch.randn(2 * n, n, generator=g, device="cuda")
    H = (x.T @ x)[None] * torch.arange(1, 66, device="cuda", dtype=torch.float32)[:, None, None].sqrt()
    ctx = lib.Context()
    U = ctx.chol_inv_upper(H)
    eye = torch.eye(n, dtype=torch.float64, device="cuda")
    for b in (0, 31, 32, 33, 64):
        assert ((U[b] @ H[b].double()) @ U[b].T - eye).abs().max() <= 64 * 2.0 ** -53 * 40 * n ** 0.5
    H[50, 900, 900] = -1.0
    with pytest.raises(lib.TurboBoAError, match="Hessian 50 .* pivot 900 is not positive"):
        ctx.chol_inv_upper(H)
    ctx.close()
