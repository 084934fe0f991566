"""Grids searched over 32, 64 and 128 columns (groups, narrow layers), in one kernel, against the definition in 64 bits: every width, numbers of candidates
around the tiles of 16 and beyond what the kernel takes, rows and matrices around what a workgroup takes (GPU)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def search(W, H, group, bits, points, shrink):
    """scales and zeros [rows, groups] of the lowest cost, the first among equals."""
    rows, n = W.shape
    maxq, ncand = 2.0 ** bits - 1, max(1, int(np.ceil(shrink * points)))
    S, Z = np.zeros((rows, n // group)), np.zeros((rows, n // group))
    for g in range(n // group):
        w, h = W[:, g * group:(g + 1) * group], H[g * group:(g + 1) * group, g * group:(g + 1) * group]
        lo, hi = np.minimum(w.min(1), 0)[:, None], np.maximum(w.max(1), 0)[:, None]
        zero = lo == hi
        lo, hi = np.where(zero, -1.0, lo), np.where(zero, 1.0, hi)
        p = 1.0 - np.arange(ncand)[None, :] / points
        s = (p * hi - p * lo) / maxq
        z = np.rint(-(p * lo) / s)
        d = s[..., None] * (np.clip(np.rint(w[:, None, :] / s[..., None]) + z[..., None], 0, maxq) - z[..., None]) - w[:, None, :]
        best = ((d @ h) * d).sum(-1).argmin(1)
        S[:, g], Z[:, g] = s[np.arange(rows), best], z[np.arange(rows), best]
    return S, Z


@pytest.mark.parametrize("n,group,rows,bits,points,shrink", [
    (128, 128, 1, 2, 100, 0.8), (256, 128, 513, 3, 100, 0.8), (256, 64, 40, 4, 17, 1.0), (192, 64, 600, 2, 16, 1.0), (96, 32, 5, 8, 20, 0.75), (64, 32, 1030, 3, 1, 1.0),
    (384, 128, 7, 4, 256, 1.0), (128, 64, 9, 2, 260, 1.0), (128, 0, 70, 3, 100, 0.8), (64, 0, 33, 4, 100, 0.8)])
def test_is_the_lowest_cost(lib, n, group, rows, bits, points, shrink):
    g = torch.Generator(device="cuda"); g.manual_seed(n + rows)
    x = torch.randn(3 * n, n, generator=g, device="cuda", dtype=torch.float64) @ (torch.eye(n, device="cuda") + 0.1 * torch.randn(n, n, generator=g, device="cuda")).double()
    H = (x.T @ x).float()
    W = 0.02 * torch.randn(rows, n, generator=g, device="cuda")
    W[0] = 0.0
    ctx = lib.Context()
    got = ctx.quantize_layer(W, H, None, None, 1, bits, rows, group=group, adaptive_grid=False, cd_iters=0, grid_points=points, max_shrink=shrink, damp=0.01)
    h = H.double().cpu().numpy()
    h = h + 0.01 * np.trace(h) / n * np.eye(n)
    S, Z = search(W.double().cpu().numpy(), h, group or n, bits, points, shrink)
    assert np.array_equal(got["scales"].cpu().numpy().reshape(S.shape), S.astype(np.float32)) and np.array_equal(got["zeros"].cpu().numpy().reshape(S.shape), Z.astype(np.float32))
    ctx.close()


@pytest.mark.parametrize("group", [32, 128])
def test_a_matrix_per_head(lib, group):
    g = torch.Generator(device="cuda"); g.manual_seed(group)
    x = torch.randn(3, 700, 256, generator=g, device="cuda", dtype=torch.float64)
    H = (x.transpose(1, 2) @ x).float().contiguous()
    W = 0.02 * torch.randn(3 * 20, 256, generator=g, device="cuda")
    Ho = torch.eye(20, device="cuda")[None].repeat(3, 1, 1).contiguous()
    ctx = lib.Context()
    got = ctx.quantize_layer(W, H, Ho, None, 3, 3, 20, group=group, adaptive_grid=False, cd_iters=0, damp=0.01)
    for k in range(3):
        h = H[k].double().cpu().numpy(); h = h + 0.01 * np.trace(h) / 256 * np.eye(256)
        S, _ = search(W[20 * k:20 * k + 20].double().cpu().numpy(), h, group, 3, 100, 0.8)
        assert np.array_equal(got["scales"][20 * k:20 * k + 20].cpu().numpy(), S.astype(np.float32))
    ctx.close()
