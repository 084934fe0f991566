"""16-bit products with at most 128 result rows, which take tiles of 128 x 256: edges in every direction, short and long contractions, batches, both 16-bit
types and the causal limit, against torch in 64 bits (GPU)."""
import pytest
import torch

pytestmark = pytest.mark.gpu
CAUSAL, PERSISTENT, HALF = 2, 4, 64


@pytest.mark.parametrize("half", [0, 1])
@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("batch,M,N,K", [(1, 128, 256, 32), (1, 1, 256, 96), (9, 64, 300, 320), (3, 100, 777, 800), (8, 127, 1024, 1024), (2, 129, 512, 512), (1, 128, 255, 64), (33, 64, 2048, 64)])
def test_against_64_bits(lib, batch, M, N, K, causal, half):
    ctx = lib.Context()
    g = torch.Generator(device="cuda"); g.manual_seed(M + N + K)
    dt = torch.float16 if half else torch.bfloat16
    A = torch.randn(batch, M, K, generator=g, device="cuda").to(dt)
    B = torch.randn(batch, N, K, generator=g, device="cuda").to(dt)
    if causal:      # column n of the result takes k up to n, rounded up to the tile
        B = B * (torch.arange(K, device="cuda")[None, :] <= torch.arange(N, device="cuda")[:, None])
    B = B.contiguous()
    a, b = A.double(), B.double().transpose(1, 2).contiguous()
    want, size = a @ b, a.abs() @ b.abs()
    flags = PERSISTENT | (CAUSAL if causal else 0) | (HALF if half else 0)
    got = ctx.gemm_bf16_nt(A.view(torch.bfloat16), B.view(torch.bfloat16), flags=flags)
    assert bool(((got.double() - want).abs() <= (K + 2) * 2.0 ** -24 * size).all())      # one rounding a product in 32 bits at most
    got16 = ctx.gemm_bf16_nt(A.view(torch.bfloat16), B.view(torch.bfloat16), out_dtype=torch.bfloat16, flags=flags).view(dt)
    assert bool(((got16.double() - want).abs() <= (K + 2) * 2.0 ** -24 * size + (2.0 ** -11 if half else 2.0 ** -8) * want.abs() + 2.0 ** -24).all())
    ctx.close()
