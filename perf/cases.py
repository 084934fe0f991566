"""The work that users of this library have it do, as cases whose time can be measured.

Every case goes through `paper_2602_04929_amd.Context` (or the block driver in `pipeline`), the way `bench.py`, the tests and
`quantize_blocks` do.  Kinds:

  block    one whole attention block through quantize_attention_block (fp32 inputs: the configuration of the smallest calls)
  layer    quantize_layer on one projection: [W_Q; W_K] stacked, W_V with a Hessian per head, W_O and the MLP projections without
           out-channel coupling, group-wise grids; ending, as a deployment does, with pack_codes (and dequant_gemv as its check)
  hess     build_hessians of one block over a batch of calibration sequences
  oproj    build_hessian_out_proj from dequantized weights
  linear   build_hessian_linear, the MLP's Hessians
  forward  the forward pass that carries activations to the next block (attention, W_O, gated MLP, down projection)
  act      the weight-activation setting's input transforms (Hadamard rotation, per-token fake quantization)

Inputs follow paper_2602_04929_amd/synth.py: Gaussian activations with 1 % heavy-tailed channels, weights N(0, 0.02^2), a second
activation stream 5 % away; Hessians handed to `layer` are made by torch in 64 bits so that every build of the library sees
the same ones.
"""
import math

import numpy as np
import torch

import paper_2602_04929_amd as tb
from paper_2602_04929_amd import pipeline, synth

ALPHA, DAMP, POINTS, SHRINK = 0.25, 0.01, 100, 0.8
NCAND = math.ceil(SHRINK * POINTS)
F64 = torch.float64
DEV = "cuda:0"


# ---------------------------------------------------------------------------------------------------- the cases
def _layer(name, d_in, heads, d_h, bits, block, group=0, per_head=0, coupled=1, corr=1, bf16=1, dev=1):
    """`coupled`: H_out given; `dev`: the deviation term R given; `corr`: rank-8 correlation between the input channels."""
    return dict(name=name, kind="layer", d_in=d_in, heads=heads, d_h=d_h, bits=bits, block=block, group=group, per_head=per_head,
                coupled=coupled, corr=corr, bf16=bf16, dev=dev)


def _attn(name, kind, d, hq, hkv, d_h, seqs, length, dev=1, group=0, d_ff=0):
    return dict(name=name, kind=kind, d=d, hq=hq, hkv=hkv, d_h=d_h, seqs=seqs, length=length, dev=dev, group=group, d_ff=d_ff)


def listed():
    return [
        # a whole small block in fp32 (the `tiny` configuration): launches and host latency are what a user waits for
        dict(_attn("block_tiny", "block", 256, 4, 4, 64, 8, 128), bits=2, block=4),
        # [W_Q; W_K] of the 7B-shaped block, INT2, 32 rows a step: the layer call of every multi-head block
        _layer("layer_qk_7b", 4096, 64, 128, 2, 32),
        # W_V of the 70B-shaped block: a Hessian per KV head, few rows against a large d_in
        _layer("layer_v_70b", 8192, 8, 128, 2, 64, per_head=1, corr=0),
        # W_O of the 70B-shaped block: the largest call, all rows in one step (gate, up and down projections run the same way)
        _layer("layer_o_70b", 8192, 1, 8192, 2, 8192, coupled=0, corr=0),
        # W_K of the 13B-shaped block: INT3, a grid per 128 input channels
        _layer("layer_k_13b", 5120, 40, 128, 3, 32, group=128, corr=0),
        # a small layer of odd sizes in fp32 weights, INT4: d_in no multiple of 32, a ragged last step; latency counts
        _layer("layer_ragged", 1000, 10, 100, 4, 48, bf16=0),
        # Hessians of the 70B-shaped grouped-query block over 8 calibration sequences (the benchmark runs 16 such chunks)
        _attn("hess_70b", "hess", 8192, 64, 8, 128, 8, 2048),
        # Hessians with a calibration length that is no multiple of 256 and an odd number of sequences, multi-head
        _attn("hess_ragged", "hess", 1536, 12, 12, 128, 5, 1000),
        # Hessian of W_O of the 7B-shaped block from its dequantized W_Q, W_K, W_V
        _attn("oproj_7b", "oproj", 4096, 32, 32, 128, 8, 2048),
        # forward pass of a quantized 7B-shaped block
        _attn("forward_7b", "forward", 4096, 32, 32, 128, 4, 2048, d_ff=11008),
        # Hessian and deviation of the 7B down projection
        dict(name="linear_7b_down", kind="linear", d_in=11008, tokens=8192, dev=1, bf16=1),
        # inputs of the weight-activation setting, an odd number of tokens
        dict(name="act_w4a4", kind="act", d=4096, tokens=16383, bits=4, bf16=1),
    ]


def _loguniform(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, int(round(v / step)) * step)


def draw(rng):
    """One more case of the same ranges: widths 128 .. 8192, 64 .. 4096 tokens a sequence, every option that the listed ones use."""
    kind = rng.choice(["layer", "layer", "layer", "hess", "hess", "oproj", "forward", "linear", "act", "block"])
    if kind == "layer":
        form = rng.choice(["qk", "v", "o", "group"])
        bits = rng.choice([2, 2, 3, 4, 8])
        opts = dict(corr=rng.randint(0, 1), bf16=rng.randint(0, 3) and 1, dev=rng.randint(0, 3) and 1)
        if form == "o":
            d_in = _loguniform(rng, 128, 8192, rng.choice([1, 8, 64, 64]))
            rows = _loguniform(rng, 64, 8192, rng.choice([1, 8, 64]))
            c = _layer("", d_in, 1, rows, bits, rows, coupled=0, **opts)
        else:
            d_h = rng.choice([32, 64, 80, 96, 100, 128, 128])
            heads = _loguniform(rng, 1, 8 if form == "v" else 64)
            block = rng.choice([8, 16, 32, 48, 64])
            if form == "group":
                group = rng.choice([32, 64, 128])
                c = _layer("", group * _loguniform(rng, 2, 5120 // group), min(heads, 40), d_h, min(bits, 4), block, group=group, **opts)
            else:
                d_in = _loguniform(rng, 128, 6144 if form == "v" else 5120, rng.choice([1, 8, 64, 64]))
                c = _layer("", d_in, heads, d_h, bits, block, per_head=int(form == "v"), **opts)
        c.pop("name")
        return c
    if kind == "linear":
        step = rng.choice([8, 64, 256])
        return dict(kind=kind, d_in=_loguniform(rng, 256, 11008, step), tokens=_loguniform(rng, 256, 8192, step), dev=rng.randint(0, 1), bf16=1)
    if kind == "act":
        return dict(kind=kind, d=1 << rng.randint(6, 13), tokens=_loguniform(rng, 1, 16383), bits=rng.choice([4, 4, 8]), bf16=rng.randint(0, 2) and 1)
    d_h = rng.choice([64, 128])
    if kind == "block":
        hq = rng.choice([2, 3, 4, 6])
        c = dict(_attn("", kind, 8 * rng.randint(16, 48), hq, rng.choice([1, hq]), rng.choice([32, 64]), rng.randint(2, 8), rng.randint(40, 160)),
                 bits=rng.choice([2, 3, 4]), block=rng.choice([4, 8, 16]))
    else:
        hkv = rng.choice([2, 4, 8])
        hq = hkv * rng.choice([1, 1, 2, 4])
        length = rng.choice([256, 512, 1024, 2048, _loguniform(rng, 64, 2048, 8), _loguniform(rng, 64, 1536, 8)])
        d = rng.choice([512, 1024, 2048, 3072, 4096, _loguniform(rng, 256, 2048, 8)])
        c = _attn("", kind, d, hq, hkv, d_h, rng.randint(1, 6), length, dev=rng.randint(0, 3) and 1 if kind != "forward" else 0,
                  group=rng.choice([0, 0, 1]) if kind in ("oproj", "forward") else 0, d_ff=_loguniform(rng, 256, 8192, 8) if kind == "forward" else 0)
    c.pop("name")
    return c


# ---------------------------------------------------------------------------------------------------- inputs
_CTX = []


def _ctx():
    """The one context that such a program keeps; its workspace is reserved ahead, as bench.py does, or grown by the first call."""
    if not _CTX:
        _CTX.append(tb.Context())
    return _CTX[0]


class _Rand:
    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed) * 1000003 + 29)

    def normal(self, *shape, std=1.0):
        return torch.randn(*shape, generator=self.g, device=DEV) * std

    def activations(self, tokens, d, corr=False):
        """(X, X~): Gaussian with 1 % of the channels Student-t (3 degrees) x 20; X = X~ + 5 % noise."""
        x = self.normal(tokens, d)
        n = max(1, round(0.01 * d))
        ch = torch.randperm(d, generator=self.g, device=DEV)[:n]
        den = (self.normal(tokens, n, 3) ** 2).sum(-1).div(3.0).sqrt()
        x[:, ch] = 20.0 * self.normal(tokens, n) / den
        if corr:
            x = x + 0.3 / math.sqrt(8) * ((x @ self.normal(d, 8)) @ self.normal(8, d))
        rms = x.pow(2).mean().sqrt()
        return x + 0.05 * rms * self.normal(tokens, d), x

    def weight(self, rows, cols, dtype):
        return self.normal(rows, cols, std=0.02).to(dtype)

    def dequantized(self, rows, cols, group=0):
        """A weight as quantize_layer leaves it: INT2 per row, or INT3 per 128 columns (fp32)."""
        w = self.normal(rows, cols, std=0.02)
        g = 128 if group and cols % 128 == 0 else cols
        v = w.view(rows, cols // g, g)
        q = 7.0 if group else 3.0
        lo, hi = 0.6 * v.amin(-1, keepdim=True), 0.6 * v.amax(-1, keepdim=True)
        s = (hi - lo) / q
        z = torch.round(-lo / s)
        return (s * (torch.clamp(torch.round(v / s) + z, 0, q) - z)).reshape(rows, cols).contiguous()


def _layer_inputs(c, seed):
    r = _Rand(seed)
    n, nh, dh = c["d_in"], c["heads"], c["d_h"]
    T = 2 * n

    def hessian(k):
        x, xf = r.activations(T, n, bool(c["corr"]))
        x, xf = x.bfloat16().to(F64), xf.bfloat16().to(F64)
        return (x.T @ x).float(), (ALPHA * ((x - xf).T @ x)).float() if c["dev"] else None
    if c["per_head"]:
        H = torch.empty(nh, n, n, device=DEV)
        R = torch.empty_like(H) if c["dev"] else None
        for h in range(nh):
            H[h], rh = hessian(h)
            if R is not None:
                R[h] = rh
    else:
        H, R = hessian(0)
    Ho = None
    if c["coupled"]:
        k = r.normal(nh, 4 * dh, dh).to(F64)
        k = k + 0.5 * r.normal(nh, 4 * dh, 1).to(F64)
        Ho = torch.stack([k[h].T @ k[h] for h in range(nh)]).float().contiguous()
    W = r.weight(nh * dh, n, torch.bfloat16 if c["bf16"] else torch.float32)
    return dict(W=W, H=H, Ho=Ho, R=R, x=r.normal(n))


def _attn_inputs(c, seed, dtype=torch.bfloat16):
    r = _Rand(seed)
    d, dq, dkv = c["d"], c["hq"] * c["d_h"], c["hkv"] * c["d_h"]
    X = torch.empty(c["seqs"], c["length"], d, device=DEV, dtype=dtype)
    Xf = torch.empty_like(X)
    x, xf = r.activations(c["seqs"] * c["length"], d)
    X.view(-1, d).copy_(x)
    Xf.view(-1, d).copy_(xf)
    s = dict(X=X, X_fp=Xf if c["dev"] else None, Wq=r.weight(dq, d, dtype), Wk=r.weight(dkv, d, dtype), Wv=r.weight(dkv, d, dtype), Wo=r.weight(d, dq, dtype))
    if c["kind"] in ("oproj", "forward"):
        s.update(Wq_deq=r.dequantized(dq, d, c["group"]), Wk_deq=r.dequantized(dkv, d, c["group"]), Wv_deq=r.dequantized(dkv, d, c["group"]))
    if c["kind"] == "forward":
        ff = c["d_ff"]
        s.update(Wo_deq=r.dequantized(d, dq, c["group"]), Wg_deq=r.dequantized(ff, d, c["group"]), Wu_deq=r.dequantized(ff, d, c["group"]),
                 Wd_deq=r.dequantized(d, ff, c["group"]))
    return s


def _block_config(c):
    return synth.BlockConfig("case", c["d"], c["hq"], c["hkv"], c["d_h"], c["seqs"], c["length"], dtype="fp32", outlier="scale",
                             n_outlier=4, bits=c["bits"], block=c["block"])


def _inputs(c, seed):
    k = c["kind"]
    if k == "layer":
        return _layer_inputs(c, seed)
    if k == "block":
        return synth.make_block(_block_config(c), seed=seed, device=DEV)
    if k == "linear":
        x, xf = _Rand(seed).activations(c["tokens"], c["d_in"])
        dt = torch.bfloat16 if c["bf16"] else torch.float32
        return dict(X=x.to(dt), X_fp=xf.to(dt) if c["dev"] else None)
    if k == "act":
        r = _Rand(seed)
        x, _ = r.activations(c["tokens"], c["d"])
        signs = torch.randint(0, 2, (c["d"],), generator=r.g, device=DEV).float() * 2 - 1
        return dict(X=x.to(torch.bfloat16 if c["bf16"] else torch.float32), signs=signs)
    return _attn_inputs(c, seed)


def prepare(case, seed):
    state = dict(_inputs(case, seed), case=case, ctx=_ctx())
    if case["kind"] == "layer":
        desc = tb.Context.layer_desc(state["W"], state["H"], case["heads"], case["bits"], case["block"], case["group"])
        state["ctx"].reserve_workspace(tb.Context.quantize_workspace_bytes(desc, bool(case["coupled"]), bool(case["dev"])))
    elif case["kind"] in ("hess", "oproj"):
        state["ctx"].reserve_workspace(tb.Context.hessian_workspace_bytes(case["d"], case["hq"], case["hkv"], case["d_h"], case["seqs"], case["length"],
                                                                          torch.bfloat16))
    elif case["kind"] == "block":
        pipeline.reserve_workspaces(state["ctx"], _block_config(case))
    return state


# ---------------------------------------------------------------------------------------------------- one pass
_LAYER_KEYS = ("codes", "scales", "zeros", "W_deq")


def run(state):
    c, ctx, s = state["case"], state["ctx"], state
    k = c["kind"]
    if k == "layer":
        r = ctx.quantize_layer(s["W"], s["H"], s["Ho"], s["R"], c["heads"], c["bits"], c["block"], group=c["group"], damp=DAMP)
        out = {key: r[key] for key in _LAYER_KEYS}
        out["loss"] = np.array(r["loss_per_head_terms"])
        out["packed"] = ctx.pack_codes(r["codes"], c["bits"])
        out["y"] = ctx.dequant_gemv(out["packed"], r["scales"], r["zeros"], s["x"], c["d_in"], c["bits"], c["group"])
        return out
    if k == "block":
        r = pipeline.quantize_attention_block(ctx, s, _block_config(c), alpha=ALPHA, damp=DAMP)
        out = {name: dict({key: r[name][key] for key in _LAYER_KEYS}, loss=np.array(r[name]["loss_per_head_terms"])) for name in ("q", "k", "v", "o")}
        out["hessians"] = {key: v for key, v in r["hessians"].items() if torch.is_tensor(v) and v.dtype == torch.float32}
        out["Hin_o"], out["R_o"] = r["Hin_o"], r["R_o"]
        return out
    if k == "hess":
        return ctx.build_hessians(s["X"], s["X_fp"], s["Wq"], s["Wk"], s["Wv"], s["Wo"], c["hq"], c["hkv"], c["d_h"], alpha=ALPHA)
    if k == "oproj":
        H, R = ctx.build_hessian_out_proj(s["X"], s["X_fp"], s["Wq_deq"], s["Wk_deq"], s["Wv_deq"], s["Wq"], s["Wk"], s["Wv"], c["hq"], c["hkv"],
                                          c["d_h"], alpha=ALPHA)
        return dict(H=H, R=R)
    if k == "linear":
        H, R = ctx.build_hessian_linear(s["X"], s["X_fp"], ALPHA)
        return dict(H=H, R=R)
    if k == "forward":
        O = ctx.attention_forward(s["X"], s["Wq_deq"], s["Wk_deq"], s["Wv_deq"], c["hq"], c["hkv"], c["d_h"])
        Xa = ctx.linear_forward(O, s["Wo_deq"], residual=s["X"])
        act = ctx.swiglu_forward(Xa, s["Wg_deq"], s["Wu_deq"])
        return dict(O=O, Xa=Xa, act=act, Y=ctx.linear_forward(act, s["Wd_deq"], residual=Xa))
    rot = ctx.hadamard_rotate(s["X"], s["signs"])
    return dict(rotated=rot, quantized=ctx.act_fakequant(rot, c["bits"]))


def work(case):
    """Inputs read once, outputs written once; the operations of the method (a symmetric result half, a causal factor its lower half)."""
    c, k = case, case["kind"]
    if k == "layer":
        n, rows, nhin, dh = c["d_in"], c["heads"] * c["d_h"], c["heads"] if c["per_head"] else 1, c["d_h"]
        esz = 2 if c["bf16"] else 4
        grid = NCAND * rows * n * (c["group"] or n)                        # delta H delta^T by symmetry: half of 2 n^2 a candidate
        factor = nhin * n ** 3 * (2 / 3 + (2 / 3 if c["dev"] else 0))
        sweep = rows * n * n * (2 if c["dev"] else 1)
        comp = rows * n * n * (4 if c["dev"] else 0) + rows * dh * n if c["coupled"] else 0
        refine = rows * n * n * (4 + (2 if c["dev"] else 0)) + (4 * rows * dh * n if c["coupled"] else 0)
        return dict(bytes=rows * n * (esz + 1 + 4 + c["bits"] / 8) + nhin * n * n * 4 * (2 if c["dev"] else 1), flops=grid + factor + sweep + comp + refine)
    if k == "linear":
        n, T = c["d_in"], c["tokens"]
        return dict(bytes=(1 + c["dev"]) * (T * n * 2 + n * n * 4), flops=T * n * n * (1 + 2 * c["dev"]))
    if k == "act":
        n = c["d"] * c["tokens"] * (2 if c["bf16"] else 4)
        return dict(bytes=4 * n, flops=c["d"] * c["tokens"] * (math.log2(c["d"]) + 6))
    d, hq, hkv, dh, S, L = c["d"], c["hq"], c["hkv"], c["d_h"], c["seqs"], c["length"]
    T, dq, dkv, paths = S * L, hq * dh, hkv * dh, 2 if c["dev"] else 1
    esz = 4 if k == "block" else 2
    proj, score = 2 * T * d * (dq + dkv), S * hq * L * L * dh
    if k == "forward":
        f = proj + 2 * T * d * dkv + 2 * score + 2 * T * dq * d + 6 * T * d * c["d_ff"]
        return dict(bytes=T * (3 * d + dq + c["d_ff"]) * 2 + 4 * d * (2 * dq + 2 * dkv + 3 * c["d_ff"]), flops=f)
    if k == "oproj":
        f = paths * (proj + 2 * T * d * dkv + 2 * score) + T * dq * dq + (2 * T * dq * dq if c["dev"] else 0)
        return dict(bytes=paths * (T * d * 2 + dq * dq * 4) + 4 * d * (dq + 2 * dkv), flops=f)
    value = S * (hq * L ** 3 / 3 + hkv * (2 * L * L * d + L * d * d))              # sum of A^T A over the group, times X, times X^T
    if c["dev"]:
        value += S * (hq * L ** 3 * 2 / 3 + hkv * (4 * L * L * d + 2 * L * d * d))
    f = paths * (proj + score) + T * d * d * (3 if c["dev"] else 1) + 2 * d * d * (dq + dkv) + value
    b = paths * T * d * esz + (2 * dq + 2 * dkv) * d * esz + paths * 4 * d * d * (1 + hkv)
    if k == "block":
        for rows, n, nhin in ((dq + dkv, d, 1), (dkv, d, hkv), (d, dq, 1)):
            f += NCAND * rows * n * n + nhin * n ** 3 * 4 / 3 + 12 * rows * n * n
            b += rows * n * 5
    return dict(bytes=b, flops=f)


def tolerance(case):
    k = case["kind"]
    if k in ("layer", "block"):
        # fp64 arithmetic, fp32 results: the values agree to fp32 rounding unless a code decision lies within 1e-12 of a tie, which
        # then moves the later codes of its row (share of codes, and its root for W_deq)
        return dict(rel=1e-2, max=0.9, differ=1e-4)
    if k in ("hess", "oproj"):
        # fp32 sums of exact products of (hi, lo) operands; the deviation terms are small sums of large terms (1.2e-5 against 64 bits
        # at the 70B shape, 7e-7 for W_O).  Lengths or widths without whole 256-tiles take single 16-bit operands for W_V (2.5e-4)
        if k == "hess":
            return dict(rel=3e-4 if case["length"] % 256 == 0 and case["d"] % 256 == 0 else 2e-3)
        return dict(rel=1e-5 if case["length"] % 256 == 0 else 1e-3)
    if k == "linear":
        return dict(rel=1e-6, max=1e-4)
    if k == "forward":
        return dict(rel=1e-2, max=0.1)
    # bf16 (fp32) results of fp32 butterflies, then levels: a value within rounding of a tie takes the next level
    return dict(rel=1e-2, max=0.9)


# ---------------------------------------------------------------------------------------------------- the same in 64 bits
def _damped(H):
    H = H.to(F64).clone()
    n = H.shape[-1]
    H += DAMP * H.diagonal(dim1=-2, dim2=-1).mean(-1)[..., None, None] * torch.eye(n, dtype=F64, device=H.device)
    return H


def _chol_inv_upper(H):
    """U upper with H^-1 = U^T U: the inverse of V, H = V V^T, V upper (a Cholesky factor taken from the last index)."""
    V = torch.linalg.cholesky(H.flip(-1, -2)).flip(-1, -2)
    return torch.linalg.solve_triangular(V, torch.eye(H.shape[-1], dtype=F64, device=H.device).expand_as(V), upper=True)


def _codes(w, s, z, maxq):
    return torch.clamp(torch.round(w / s) + z, 0.0, maxq)


def _grid(W, H, maxq):
    """Rows W [r, n] against H [n, n]: the candidate (s, z) of least delta H delta^T."""
    lo, hi = W.amin(1).clamp(max=0.0), W.amax(1).clamp(min=0.0)
    flat = lo == hi
    lo, hi = torch.where(flat, -torch.ones_like(lo), lo), torch.where(flat, torch.ones_like(hi), hi)
    one = torch.ones((), dtype=F64, device=W.device)  # (torch divides by a plain number as a product with its reciprocal)
    p = 1.0 - torch.arange(NCAND, dtype=F64, device=W.device) / (POINTS * one)
    s = (p * hi[:, None] - p * lo[:, None]) / (maxq * one)
    z = torch.round(-(p * lo[:, None]) / s)
    cost = torch.empty_like(s)
    step = max(1, int(1.5e8 / (NCAND * W.shape[1])))
    for i in range(0, W.shape[0], step):
        e = slice(i, i + step)
        d = s[e, :, None] * (_codes(W[e, None, :], s[e, :, None], z[e, :, None], maxq) - z[e, :, None]) - W[e, None, :]
        d2 = d.reshape(-1, W.shape[1])
        cost[e] = ((d2 @ H) * d2).sum(1).view(-1, NCAND)
    k = cost.argmin(1, keepdim=True)
    return s.gather(1, k)[:, 0], z.gather(1, k)[:, 0]


def _exact_layer(W, H_in, H_out, R, nh, bits, block, group):
    maxq = float(2 ** bits - 1)
    W = W.to(F64)
    rows, n = W.shape
    dh = rows // nh
    ng, gsz = (n // group, group) if group else (1, n)
    W = W.view(nh, dh, n)
    Hi = _damped(H_in if H_in.dim() == 3 else H_in[None])
    U = torch.stack([_chol_inv_upper(h) for h in Hi])
    Rd = None if R is None else (R if R.dim() == 3 else R[None]).to(F64)
    P = None if R is None else torch.stack([torch.triu(Rd[i] @ U[i].T, 1) @ U[i] for i in range(len(U))])
    Ho = None if H_out is None else _damped(H_out)
    Uo = None if Ho is None else torch.stack([_chol_inv_upper(h) for h in Ho])
    per = len(U) > 1 or nh == 1                       # one Hessian a head (or one head): products go head by head

    def mul(A, B):                                    # A [nh, r, k] times B [1 or nh, k, m], head by head
        if per:
            return torch.stack([A[h] @ B[h] for h in range(nh)])
        return (A.reshape(-1, A.shape[-1]) @ B[0]).view(nh, A.shape[1], B.shape[-1])
    codes, scales, zeros = torch.zeros_like(W), torch.zeros(nh, dh, ng, dtype=F64, device=DEV), torch.zeros(nh, dh, ng, dtype=F64, device=DEV)
    Wt = W.clone()

    def search(X, g0, g1, gi, i0, i1):
        if per:
            got = [_grid(X[h][:, g0:g1].contiguous(), Hi[h, g0:g1, g0:g1], maxq) for h in range(nh)]
            scales[:, i0:i1, gi], zeros[:, i0:i1, gi] = torch.stack([s for s, _ in got]), torch.stack([z for _, z in got])
        else:
            s, z = _grid(X[:, :, g0:g1].reshape(-1, g1 - g0).contiguous(), Hi[0, g0:g1, g0:g1], maxq)
            scales[:, i0:i1, gi], zeros[:, i0:i1, gi] = s.view(nh, -1), z.view(nh, -1)
    for i0 in range(0, dh, block):
        i1 = min(dh, i0 + block)
        Wb = Wt[:, i0:i1].clone()
        Wk, Q = Wb.clone(), torch.zeros_like(Wb)
        if not group:
            search(Wk, 0, n, 0, i0, i1)
        pw = min(64, gsz)
        for c0 in range(0, n, pw):
            c1, gi = min(n, c0 + pw), c0 // gsz
            if group and c0 % gsz == 0:
                search(Wk, c0, c0 + gsz, gi, i0, i1)
            s, z = scales[:, i0:i1, gi], zeros[:, i0:i1, gi]
            panel = Wk[:, :, c0:c1].clone()
            E, S = torch.zeros_like(panel), torch.zeros_like(panel)
            Ub, Pb = U[:, c0:c1, c0:c1], None if P is None else P[:, c0:c1, c0:c1]
            for j in range(c1 - c0):
                w = panel[:, :, j].clone()
                q = _codes(w, s, z, maxq)
                dq = s * (q - z)
                e = (w - dq) / Ub[:, j, j][:, None]
                codes[:, i0:i1, c0 + j], Q[:, :, c0 + j], E[:, :, j], S[:, :, j] = q, dq, e, w
                panel -= e[:, :, None] * Ub[:, j][:, None, :]
                if P is not None:
                    panel -= w[:, :, None] * Pb[:, j][:, None, :]
            if c1 < n:
                Wk[:, :, c1:] -= mul(E, U[:, c0:c1, c1:])
                if P is not None:
                    Wk[:, :, c1:] -= mul(S, P[:, c0:c1, c1:])
        if Uo is not None and i1 < dh:
            E = Wb - Q
            if Rd is not None:
                E -= mul(mul(mul(Wb, Rd), U.transpose(1, 2)), U)
            for h in range(nh):
                Lo = Uo[h].T
                T = torch.linalg.solve_triangular(Lo[i0:i1, i0:i1], Lo[i1:, i0:i1], upper=False, left=False)
                Wt[h, i1:] -= T @ E[h]
    Wbar = codes - zeros.repeat_interleave(gsz, 2)
    WR = None if Rd is None else mul(W, Rd)
    if group:                                         # refinement of every (row, group) in turn
        Q = scales.repeat_interleave(gsz, 2) * Wbar
        HoT = None if Ho is None else Ho
        if Ho is None:                                # rows decouple: all rows of a group side by side
            for gi in range(ng):
                G = slice(gi * gsz, gi * gsz + gsz)
                a = mul(Wbar[:, :, G], Hi[:, G, :])
                num = ((W - Q) * a).sum(2) - (0 if WR is None else (WR[:, :, G] * Wbar[:, :, G]).sum(2))
                den = (a[:, :, G] * Wbar[:, :, G]).sum(2)
                scales[:, :, gi] += torch.where(den > 0, num / den, torch.zeros_like(num))
                Q[:, :, G] = scales[:, :, gi, None] * Wbar[:, :, G]
        else:
            for j in range(dh):
                for gi in range(ng):
                    G = slice(gi * gsz, gi * gsz + gsz)
                    wb = Wbar[:, j, G]
                    a = mul(wb[:, None], Hi[:, G, :])[:, 0]
                    v = (HoT[:, :, j, None] * (W - Q)).sum(1)
                    num = (v * a).sum(1)
                    if WR is not None:
                        num = num - ((HoT[:, :, j, None] * WR[:, :, G]).sum(1) * wb).sum(1)
                    den = (a[:, G] * wb).sum(1) * HoT[:, j, j]
                    scales[:, j, gi] += torch.where(den > 0, num / den, torch.zeros_like(num))
                    Q[:, j, G] = scales[:, j, gi, None] * wb
    else:
        A, Z = mul(Wbar, Hi), mul(W, Hi)
        if WR is not None:
            Z = Z - WR
        if Ho is None:
            C, F = (A * Wbar).sum(2), (Wbar * Z).sum(2)
            s = scales[:, :, 0]
            scales[:, :, 0] = torch.where(C > 0, s + (F - s * C) / C, s)
        else:
            C = torch.stack([A[h] @ Wbar[h].T for h in range(nh)])
            F = torch.stack([Wbar[h] @ Z[h].T for h in range(nh)])
            s = scales[:, :, 0]
            for j in range(dh):
                num = ((F[:, j] - s * C[:, j]) * Ho[:, :, j]).sum(1)
                den = C[:, j, j] * Ho[:, j, j]
                s[:, j] += torch.where(den > 0, num / den, torch.zeros_like(num))
    Q = scales.repeat_interleave(gsz, 2) * Wbar
    D = Q - W
    DH = mul(D, Hi)

    def trace(M):                                     # tr(H_out M D^T) per head
        if Ho is None:
            return (M * D).sum((1, 2))
        return torch.stack([(Ho[h] * (D[h] @ M[h].T)).sum() for h in range(nh)])
    cross = torch.zeros(nh, dtype=F64, device=DEV) if WR is None else 2.0 * trace(WR)
    return dict(codes=codes.view(rows, n).to(torch.uint8), scales=scales.view(rows, ng), zeros=zeros.view(rows, ng), W_deq=Q.view(rows, n),
                loss=torch.stack([trace(DH), cross], 1))


def _pack(codes, bits):
    rows, n = codes.shape
    words = -(-n * bits // 32)
    b = (codes.to(torch.int64)[:, :, None] >> torch.arange(bits, device=codes.device)) & 1
    b = torch.nn.functional.pad(b.reshape(rows, -1), (0, words * 32 - n * bits)).view(rows, words, 32)
    return (b << torch.arange(32, device=codes.device)).sum(2).to(torch.int32)


def _probs(x, wq, wk):
    q, k = x @ wq.T, x @ wk.T
    s = q @ k.T / math.sqrt(wq.shape[0])
    return torch.softmax(s.masked_fill(torch.ones_like(s, dtype=torch.bool).triu(1), -math.inf), -1)


def _exact_hessians(c, s):
    d, hq, hkv, dh = c["d"], c["hq"], c["hkv"], c["d_h"]
    rep, fp = hq // hkv, s["X_fp"] is not None
    X = s["X"].to(F64)
    Xf = s["X_fp"].to(F64) if fp else None
    Wq, Wk, Wo = (s[w].to(F64) for w in ("Wq", "Wk", "Wo"))
    z = lambda *sh: torch.zeros(*sh, dtype=F64, device=DEV)  # noqa: E731
    o = dict(Hin_qk=z(d, d), Hout_q=z(hq, dh, dh), Hout_k=z(hkv, dh, dh), Hin_v=z(hkv, d, d), Hout_v=z(hkv, dh, dh), R_qk=z(d, d) if fp else None,
             R_v=z(hkv, d, d) if fp else None)
    for i in range(X.shape[0]):
        x, xf = X[i], Xf[i] if fp else None
        o["Hin_qk"] += x.T @ x
        if fp:
            o["R_qk"] += ALPHA * ((x - xf).T @ x)
        for g in range(hkv):
            wk = Wk[g * dh:(g + 1) * dh]
            kk = x @ wk.T
            B, C = z(len(x), len(x)), z(len(x), len(x))
            for h in range(g * rep, (g + 1) * rep):
                wq = Wq[h * dh:(h + 1) * dh]
                q = x @ wq.T
                o["Hout_q"][h] += kk.T @ kk
                o["Hout_k"][g] += q.T @ q
                A = _probs(x, wq, wk)
                B += A.T @ A
                if fp:
                    C += _probs(xf, wq, wk).T @ A
            BX = B @ x
            o["Hin_v"][g] += x.T @ BX
            if fp:                                    # sum (A x - A~ x~)^T A x
                o["R_v"][g] += ALPHA * (x.T @ BX - xf.T @ (C @ x))
    for h in range(hq):
        w = Wo[:, h * dh:(h + 1) * dh]
        o["Hout_v"][h // rep] += w.T @ w
    return o


def _attention(c, X, wq, wk, wv):
    rep, dh = c["hq"] // c["hkv"], c["d_h"]
    X, wq, wk, wv = (t.to(F64) for t in (X, wq, wk, wv))
    out = torch.empty(X.shape[0], X.shape[1], c["hq"] * dh, dtype=F64, device=DEV)
    for i in range(X.shape[0]):
        for h in range(c["hq"]):
            g = slice(h // rep * dh, (h // rep + 1) * dh)
            out[i, :, h * dh:(h + 1) * dh] = _probs(X[i], wq[h * dh:(h + 1) * dh], wk[g]) @ (X[i] @ wv[g].T)
    return out


def _exact_oproj(c, s):
    O = _attention(c, s["X"], s["Wq_deq"], s["Wk_deq"], s["Wv_deq"]).flatten(0, 1)
    R = None
    if s["X_fp"] is not None:
        R = ALPHA * ((O - _attention(c, s["X_fp"], s["Wq"], s["Wk"], s["Wv"]).flatten(0, 1)).T @ O)
    return dict(H=O.T @ O, R=R)


def _exact_block(c, s):
    h = _exact_hessians(c, s)
    f = lambda t: None if t is None else t.float()  # noqa: E731  (the Hessians are handed on in 32 bits)
    out = {"hessians": h}
    q = _exact_layer(torch.cat([s["Wq"], s["Wk"]]), f(h["Hin_qk"]), f(torch.cat([h["Hout_q"], h["Hout_k"]])), f(h["R_qk"]), c["hq"] + c["hkv"], c["bits"],
                     c["block"], 0)
    rows = c["hq"] * c["d_h"]
    out["q"] = dict({k: q[k][:rows] for k in _LAYER_KEYS}, loss=q["loss"][:c["hq"]])
    out["k"] = dict({k: q[k][rows:] for k in _LAYER_KEYS}, loss=q["loss"][c["hq"]:])
    out["v"] = _exact_layer(s["Wv"], f(h["Hin_v"]), f(h["Hout_v"]), f(h["R_v"]), c["hkv"], c["bits"], c["block"], 0)
    o = _exact_oproj(c, dict(s, **{"W%s_deq" % n: out[n]["W_deq"].float() for n in "qkv"}))
    out["Hin_o"], out["R_o"] = o["H"], o["R"]
    out["o"] = _exact_layer(s["Wo"], f(o["H"]), None, f(o["R"]), 1, c["bits"], c["d"], 0)
    return out


def exact(case, seed):
    c, k, s = case, case["kind"], _inputs(case, seed)
    if k == "block":
        return _exact_block(c, s)
    if k == "layer":
        if c["group"] and c["coupled"] and c["heads"] * c["d_h"] ** 2 * c["d_in"] * (c["d_in"] // c["group"]) > 6e12:
            return None                               # the refinement visits every (row, group) in turn
        o = _exact_layer(s["W"], s["H"], s["Ho"], s["R"], c["heads"], c["bits"], c["block"], c["group"])
        o["packed"] = _pack(o["codes"], c["bits"])
        o["y"] = o["W_deq"] @ s["x"].to(F64)
        return o
    if k == "hess":
        return _exact_hessians(c, s)
    if k == "oproj":
        return _exact_oproj(c, s)
    if k == "linear":
        x = s["X"].to(F64)
        return dict(H=x.T @ x, R=None if s["X_fp"] is None else ALPHA * ((x - s["X_fp"].to(F64)).T @ x))
    if k == "forward":
        w = {n: s[n].to(F64) for n in ("Wo_deq", "Wg_deq", "Wu_deq", "Wd_deq")}
        O = _attention(c, s["X"], s["Wq_deq"], s["Wk_deq"], s["Wv_deq"])
        Xa = O @ w["Wo_deq"].T + s["X"].to(F64)
        act = torch.nn.functional.silu(Xa @ w["Wg_deq"].T) * (Xa @ w["Wu_deq"].T)
        return dict(O=O, Xa=Xa, act=act, Y=act @ w["Wd_deq"].T + Xa)
    x = s["X"].to(F64) * s["signs"].to(F64)
    d = x.shape[1]
    h = 1
    while h < d:
        x = x.view(-1, d // (2 * h), 2, h)
        x = torch.stack([x[:, :, 0] + x[:, :, 1], x[:, :, 0] - x[:, :, 1]], 2).reshape(-1, d)
        h *= 2
    rot = x / math.sqrt(d)
    maxq = float(2 ** c["bits"] - 1)
    r = rot.to(s["X"].dtype).to(F64)                  # the levels are decided on the stored values
    lo, hi = r.amin(1, keepdim=True).clamp(max=0.0), r.amax(1, keepdim=True).clamp(min=0.0)
    st = (hi - lo) / torch.full_like(hi, maxq)
    z = torch.round(-lo / st)
    return dict(rotated=rot, quantized=st * (_codes(r, st, z, maxq) - z))
