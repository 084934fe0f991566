"""Workspaces on a device that has no room for residues: sizes with and without them (CPU), reservation and calls that keep to the smaller one (GPU)."""
import pytest
import torch

from paper_2602_04929_amd import synth


def test_least_sizes():
    """Residues are 15 bytes per element of an operand: layers and Hessians that use them need more with than without, others the same."""
    import paper_2602_04929_amd as tb
    C = tb.Context
    d = lambda rows, n, nh, per=0, block=32: tb.LayerDesc(rows, n, nh, per, 2, block, 0, tb.BF16, 1, 1, 100, 0.8, 0.01, 0.0)  # noqa: E731
    for desc, with_out in ((d(8192, 4096, 64), True), (d(8192, 8192, 1, block=8192), False), (d(1024, 8192, 8, 1, 64), True)):
        least, full = C.quantize_workspace_bytes(desc, with_out, least=True), C.quantize_workspace_bytes(desc, with_out)
        assert 0 < least < full - 15 * desc.d_in ** 2
    assert C.quantize_workspace_bytes(d(64, 512, 1), least=True) == C.quantize_workspace_bytes(d(64, 512, 1))
    # 8192 x 8192 and a few sequences: residues need more than the buffers whose room they share
    a = (8192, 64, 8, 128, 1, 256, torch.bfloat16)
    assert 0 < C.hessian_workspace_bytes(*a, least=True) < C.hessian_workspace_bytes(*a)
    a = (256, 4, 4, 64, 8, 128, torch.float32)
    assert 0 < C.hessian_workspace_bytes(*a, least=True) == C.hessian_workspace_bytes(*a)


def test_block_reservation_settles_for_less():
    """reserve_workspaces asks each context for the size with residues and, refused, for the one without; any other error is the caller's."""
    import paper_2602_04929_amd as tb
    from paper_2602_04929_amd import pipeline

    class Room(tb.Context):
        def __init__(self, room, code=-3):
            self.asked, self.room, self.code = [], room, code

        def reserve_workspace(self, nbytes):
            self.asked.append(nbytes)
            if nbytes > self.room:
                raise tb.TurboBoAError(self.code, "no room")

        close = __del__ = lambda self: None
    cfg = synth.CONFIGS["llama2-7b"]
    plenty = Room(1 << 60)
    full, = pipeline.reserve_workspaces(plenty, cfg)
    assert plenty.asked == [full]
    tight = Room(full - 1)
    least, = pipeline.reserve_workspaces(tight, cfg)
    assert tight.asked == [full, least] and least < full
    side = [Room(1 << 60), Room(1 << 20)]
    with pytest.raises(tb.TurboBoAError):
        pipeline.reserve_workspaces(Room(0, code=-4), cfg)
    with pytest.raises(tb.TurboBoAError):
        pipeline.reserve_workspaces(plenty, cfg, side_contexts=side[1:])
    assert len(pipeline.reserve_workspaces(plenty, cfg, side_contexts=side[:1])) == 2


@pytest.mark.gpu
def test_a_refused_size_is_not_asked_for_again(lib):
    n = 8192
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn(10000, n, generator=g, device="cuda")
    H, W = x.T @ x, 0.02 * torch.randn(n, n, generator=g, device="cuda")
    del x
    call = lambda c: c.quantize_layer(W, H, None, None, 1, bits=2, block=n)["codes"]  # noqa: E731
    desc = lib.Context.layer_desc(W, H, 1, 2, n)
    full, least = (lib.Context.quantize_workspace_bytes(desc, False, False, least=b) for b in (False, True))
    ctx = lib.Context()
    want = call(ctx).clone()
    assert ctx.workspace_bytes() == full
    ctx.close()
    # more than any device has: refused, and the workspace of before stays
    ctx = lib.Context()
    ctx.reserve_workspace(least)
    with pytest.raises(lib.TurboBoAError) as e:
        ctx.reserve_workspace(1 << 46)
    assert e.value.code == -3 and ctx.workspace_bytes() == least
    assert torch.equal(call(ctx), want) and ctx.workspace_bytes() == full      # (less than what was refused: tried)
    ctx.close()
    # the larger size refused, the smaller one reserved: calls keep to it, also once there is room again
    ctx = lib.Context()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    ballast = torch.empty(torch.cuda.mem_get_info()[0] - (least + full) // 2, dtype=torch.uint8, device="cuda")
    with pytest.raises(lib.TurboBoAError):
        ctx.reserve_workspace(full)
    ctx.reserve_workspace(least)
    assert torch.equal(call(ctx), want) and ctx.workspace_bytes() == least
    del ballast
    torch.cuda.empty_cache()
    assert torch.equal(call(ctx), want) and ctx.workspace_bytes() == least
    ctx.reserve_workspace(full)
    assert torch.equal(call(ctx), want) and ctx.workspace_bytes() == full
    ctx.close()
