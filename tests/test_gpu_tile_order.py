"""fp64 products of a few rounds of workgroups whose contraction length depends on the tile column: per-head layers of many heads (more than 256 tiles, taken by length) against every head
quantized by itself (fewer).  The order of the tiles changes no sum, but tile shapes and splits differ with the
number of heads: whole numbers are compared for equality, scales with the spacing of fp32, losses with 1e-10."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,dh,n,with_R", [(9, 128, 1100, True), (12, 64, 1030, True), (33, 128, 520, False), (7, 96, 1537, True)])
def test_heads_together_and_alone(lib, heads, dh, n, with_R):
    g = torch.Generator(device="cuda").manual_seed(heads * 101 + n)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)  # noqa: E731
    H = torch.empty(heads, n, n, device="cuda")
    R = torch.empty_like(H) if with_R else None
    for h in range(heads):
        x = rnd(2 * n, n) + 0.5 * rnd(2 * n, 1)
        H[h] = x.T @ x
        if with_R:
            R[h] = 0.025 * (rnd(2 * n, n).T @ x)
    W = 0.02 * rnd(heads * dh, n)
    k = rnd(heads, 4 * dh, dh)
    Ho = torch.matmul(k.transpose(1, 2).contiguous(), k).contiguous()
    ctx = lib.Context()
    kw = dict(bits=2, block=32)
    whole = ctx.quantize_layer(W, H, Ho, R, heads, **kw)
    for h in {0, 1, heads // 2, heads - 1}:
        part = ctx.quantize_layer(W[h * dh:(h + 1) * dh].contiguous(), H[h:h + 1].contiguous(), Ho[h:h + 1].contiguous(), R[h:h + 1].contiguous() if with_R else None, 1, **kw)
        r = slice(h * dh, (h + 1) * dh)
        assert torch.equal(whole["codes"][r], part["codes"]) and torch.equal(whole["zeros"][r], part["zeros"])
        torch.testing.assert_close(whole["scales"][r], part["scales"], rtol=2.0 ** -22, atol=0.0)
        for a, b in zip(whole["loss_per_head_terms"][h], part["loss_per_head_terms"][0]):
            assert abs(a - b) <= 1e-10 * max(abs(a), abs(b), part["loss_quad"])
    ctx.close()
