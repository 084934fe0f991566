"""fp32-input Hessian builds in chunks of sequences and KV groups, and the compensation of a block of thousands of rows."""
import math

import numpy as np
import pytest
import torch

from oracle import turboboa_ref as O
from tests.parity import compare_layer

pytestmark = pytest.mark.gpu
F64 = torch.float64


def probs(x, wq, wk, causal):
    s = (x @ wq.T) @ (x @ wk.T).T / math.sqrt(wq.shape[0])
    if causal:
        s = s.masked_fill(torch.ones_like(s, dtype=torch.bool).triu(1), -math.inf)
    return torch.softmax(s, -1)


# one chunk of everything with grouped queries; more heads than 1 GiB of probabilities holds (15 of 20 KV groups, one sequence at a time);
# whole KV groups, several sequences (11 of 24) at a time
@pytest.mark.parametrize("S,L,d,hq,hkv,dh,causal", [(3, 20, 48, 6, 2, 16, 1), (2, 2048, 64, 40, 20, 8, 1), (24, 512, 32, 16, 8, 8, 0)])
def test_f64_build_in_chunks(lib, S, L, d, hq, hkv, dh, causal):
    g = torch.Generator(device="cuda"); g.manual_seed(L)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    Xf = rnd(S, L, d); X = Xf + 0.05 * rnd(S, L, d)
    Wq, Wk, Wv, Wo = 0.2 * rnd(hq * dh, d), 0.2 * rnd(hkv * dh, d), 0.2 * rnd(hkv * dh, d), 0.2 * rnd(d, hq * dh)
    ctx = lib.Context()
    got = ctx.build_hessians(X, Xf, Wq, Wk, Wv, Wo, hq, hkv, dh, alpha=0.25, causal=bool(causal))
    H, R = ctx.build_hessian_out_proj(X, Xf, Wq, Wk, Wv, Wq, Wk, Wv, hq, hkv, dh, alpha=0.25, causal=bool(causal))
    rep = hq // hkv
    x, xf, wq, wk, wv, wo = (t.to(F64) for t in (X, Xf, Wq, Wk, Wv, Wo))
    want = dict(Hin_v=torch.zeros(hkv, d, d, dtype=F64, device="cuda"), R_v=torch.zeros(hkv, d, d, dtype=F64, device="cuda"),
                Hout_q=torch.zeros(hq, dh, dh, dtype=F64, device="cuda"), Hout_k=torch.zeros(hkv, dh, dh, dtype=F64, device="cuda"),
                Hout_v=torch.zeros(hkv, dh, dh, dtype=F64, device="cuda"))
    o, of = torch.zeros(S, L, hq * dh, dtype=F64, device="cuda"), torch.zeros(S, L, hq * dh, dtype=F64, device="cuda")
    for h in range(hq):
        rows, kr = slice(h * dh, (h + 1) * dh), slice(h // rep * dh, (h // rep + 1) * dh)
        want["Hout_v"][h // rep] += wo[:, rows].T @ wo[:, rows]
        for s in range(S):
            A, Af = probs(x[s], wq[rows], wk[kr], causal), probs(xf[s], wq[rows], wk[kr], causal)
            Y, Yf = A @ x[s], Af @ xf[s]
            want["Hin_v"][h // rep] += Y.T @ Y
            want["R_v"][h // rep] += 0.25 * (Y - Yf).T @ Y
            k, q = x[s] @ wk[kr].T, x[s] @ wq[rows].T
            want["Hout_q"][h] += k.T @ k
            want["Hout_k"][h // rep] += q.T @ q
            o[s, :, rows], of[s, :, rows] = A @ (x[s] @ wv[kr].T), Af @ (xf[s] @ wv[kr].T)
    o, of = o.flatten(0, 1), of.flatten(0, 1)
    for name, a, b in [(k, got[k], v) for k, v in want.items()] + [("H_o", H, o.T @ o), ("R_o", R, 0.25 * (o - of).T @ o)]:
        assert float((a.to(F64) - b).abs().max() / b.abs().max()) <= 2.0 ** -23, name      # the rounding of the fp32 result
    ctx.close()


@pytest.mark.parametrize("dh,block", [(2112, 2080), (70, 65), (66, 1)])
def test_compensation_after_a_block(lib, dh, block):
    """Blocks of more rows than the right-hand sides fit LDS for, more than a wavefront is wide, and one."""
    n = 64
    rng = np.random.default_rng(dh)
    X = rng.standard_normal((4 * n, n)); H = (X.T @ X).astype(np.float32)
    K = rng.standard_normal((1, dh + 64, dh)); Ho = np.stack([k.T @ k for k in K]).astype(np.float32)
    W = (0.02 * rng.standard_normal((dh, n))).astype(np.float32)
    ctx = lib.Context()
    d = lambda a: torch.from_numpy(a).cuda()
    got = ctx.quantize_layer(d(W), d(H), d(Ho), None, 1, 3, block, cd_iters=0)
    ref = O.quantize_layer(W.astype(np.float64), H.astype(np.float64), Ho.astype(np.float64), None, 1, bits=3, block=block, cd_iters=0)
    compare_layer(got, ref, rtol=1e-6)
    ctx.close()


def test_more_heads_than_a_launch_has_batch_entries(lib):
    hq, hkv, L, d = 65600, 16400, 2, 4
    g = torch.Generator(device="cuda"); g.manual_seed(3)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    X, Wq, Wk, Wv, Wo = rnd(1, L, d), rnd(hq, d), rnd(hkv, d), rnd(hkv, d), rnd(d, hq)
    ctx = lib.Context()
    got = ctx.build_hessians(X, None, Wq, Wk, Wv, Wo, hq, hkv, 1, causal=False)
    x, wq, wk, wo = (t.to(F64) for t in (X[0], Wq, Wk, Wo))
    k, q = x @ wk.T, x @ wq.T
    A = torch.softmax(q.view(L, hkv, 4).permute(1, 2, 0)[..., None] * k.T[:, None, None, :], -1)      # [group, head, query, key]
    Y = (A @ x).reshape(hkv, 4 * L, d)
    want = dict(Hout_q=(k * k).sum(0).repeat_interleave(4), Hout_k=(q * q).sum(0).view(hkv, 4).sum(1), Hout_v=(wo * wo).sum(0).view(hkv, 4).sum(1),
                Hin_v=(Y[..., :, None] * Y[..., None, :]).sum(1))
    for name, w in want.items():
        assert float((got[name].to(F64).view(w.shape) - w).abs().max() / w.abs().max()) <= 2.0 ** -23, name
    ctx.close()


def test_f64_build_in_parts_of_a_group(lib):
    """A KV group that 1 GiB does not hold (30 of its 40 heads at a time), and a workspace that does not grow with the heads of a group."""
    test_f64_build_in_chunks(lib, 2, 2048, 64, 40, 1, 8, 1)
    need = lib.Context.hessian_workspace_bytes(64, 40, 1, 8, 2, 2048, torch.float32)
    assert need < 2 ** 30 + 2 ** 27
    # heads too long for 1 GiB: one at a time, however many there are in a group (only the projections grow)
    one, two = (lib.Context.hessian_workspace_bytes(64, hq, 1, 8, 1, 32768, torch.float32) for hq in (1, 2))
    assert two - one < 2 ** 27


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("S,L,d,hq,hkv,dh", [(1, 2048, 1032, 16, 2, 64), (3, 40, 64, 4, 2, 32), (2, 256, 256, 4, 2, 32)])
def test_reserved_workspace_is_enough_for_every_set_of_outputs(lib, S, L, d, hq, hkv, dh, dtype):
    g = torch.Generator(device="cuda"); g.manual_seed(L)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(dtype)
    X, Xf, Wq, Wk, Wv, Wo = rnd(S, L, d), rnd(S, L, d), rnd(hq * dh, d), rnd(hkv * dh, d), rnd(hkv * dh, d), rnd(d, hq * dh)
    ctx = lib.Context()
    need = lib.Context.hessian_workspace_bytes(d, hq, hkv, dh, S, L, dtype)
    ctx.reserve_workspace(need)
    f = [w.float() for w in (Wq, Wk, Wv)]
    for xf in (Xf, None):
        ctx.build_hessians(X, xf, Wq, Wk, Wv, Wo, hq, hkv, dh, alpha=0.25)
        ctx.build_hessian_out_proj(X, xf, *f, Wq, Wk, Wv, hq, hkv, dh, alpha=0.25)
        assert ctx.workspace_bytes() == need
    ctx.close()
