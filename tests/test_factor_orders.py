"""Orders that the products of residues do not take (contractions beyond 32768 terms): the factorisation of H_in stays in fp64 there, as the workspace plan shows on the CPU and a run on the GPU."""
import pytest
import torch


def layer_bytes(d_in):
    import paper_2602_04929_amd as tb
    return tb.Context.quantize_workspace_bytes(tb.LayerDesc(64, d_in, 1, 0, 2, 64, 0, tb.BF16, 1, 1, 100, 0.8, 0.01, 0.0), with_H_out=False, with_R=False)


def test_plan_of_the_largest_orders():
    """Residues of V and U take 30 bytes per element: with them up to 33280 (whose longest contraction has 32768 terms), without them from 33281 on."""
    n = 33280
    assert layer_bytes(n) - layer_bytes(n + 1) > 28 * n * n
    assert layer_bytes(53248) < 6 * 8 * 53248 ** 2


@pytest.mark.gpu
def test_factor_of_an_order_beyond_the_products(lib):
    """U^T U = H^-1 applied to a few vectors.  H = I + 0.5 q q^T (q of unit norm): condition number 1.5, an error of a few n 2^-53 at most."""
    n = 33281
    g = torch.Generator(device="cuda").manual_seed(1)
    q = torch.randn(n, generator=g, device="cuda")
    q /= q.norm()
    H = torch.outer(0.5 * q, q)
    H.diagonal().add_(1.0)
    ctx = lib.Context()
    U = ctx.chol_inv_upper(H)
    ctx.close()
    x = torch.randn(n, 3, generator=g, device="cuda", dtype=torch.float64)
    hx = torch.cat([H[i:i + 4096].double() @ x for i in range(0, n, 4096)])      # (H is symmetric to the bit: outer products round alike)
    assert (U.T @ (U @ hx) - x).abs().max() <= 8 * n ** 0.5 * 2.0 ** -52
