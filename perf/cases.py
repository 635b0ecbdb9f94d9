"""Performance cases of the dilated-attention library, through its public entry points.

A case is a dict of plain values.  `kind` names the call:

    fwd          dilated_attn on q, k, v
    bwd          dilated_attn_bwd on q, k, v, the forward's out and lse, and dout
    layer_fwd    LongNetAttention, forward without gradients
    layer_train  LongNetAttention, forward and the gradients of its input and parameters
    layer_norm   layer_norm and layer_norm_bwd
    wgrad        wgrad with the bias gradient

`patterns` is a text "w:r,w:r,...".  Inputs are seeded Gaussian values on the
GPU, the distribution the repository's workloads use; `exact` computes the same
outputs with plain float64 torch operations.
"""
import math

import torch

import paper_2307_02486_amd as da
from paper_2307_02486_amd.layer import LongNetAttention

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
PAPER = "2048:1,4096:2,8192:4,16384:6,32768:12"  # the paper's five patterns (Sec. 4.1)


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------
def _attn(kind, B, N, H, D, patterns, dtype="bf16", causal=True, sigma=1.0, name=None):
    c = {"kind": kind, "B": B, "N": N, "H": H, "D": D, "patterns": patterns, "dtype": dtype, "causal": causal,
         "sigma": sigma}
    return dict(c, name=name) if name else c


def _layer(kind, B, N, H, D, patterns, name=None):
    c = {"kind": kind, "B": B, "N": N, "H": H, "D": D, "patterns": patterns, "causal": True}
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest call: 256 tokens, two heads, float32 (a unit check, a
        # short prompt): launches and host latency are all there is.
        _attn("fwd", 1, 256, 2, 32, "64:1,128:2,256:4", "f32", name="fwd_tiny_f32"),
        # A float32 user (numerical studies, float32 models) at 4K tokens.
        _attn("fwd", 1, 4096, 12, 64, "2048:1,4096:2", "f32", name="fwd_4k_f32"),
        # Two 8K-token sequences of a 12-head model: an ordinary prefill batch.
        _attn("fwd", 2, 8192, 12, 64, "2048:1,4096:2,8192:4", name="fwd_8k_b2"),
        # The paper's model at 32K tokens with its five patterns.
        _attn("fwd", 1, 32768, 12, 64, PAPER, name="fwd_32k"),
        # One device's share of a long sequence: 1M tokens, heads of 128.
        _attn("fwd", 1, 1048576, 16, 128, "2048:1,8192:2,32768:4,131072:8,524288:16,1048576:32", name="fwd_1m_d128"),
        # An encoder: not causal, odd lengths, ragged segments, heads of 32.
        _attn("fwd", 2, 5003, 6, 32, "512:1,1777:3,5003:8", causal=False, name="fwd_ragged_d32"),
        # Training: the backward of the 32K-token call.
        _attn("bwd", 1, 32768, 12, 64, PAPER, name="bwd_32k"),
        # The backward with heads of 128, the first patterns of the 1M-token list.
        _attn("bwd", 1, 32768, 16, 128, "2048:1,8192:2,32768:4", name="bwd_32k_d128"),
        # Inference of one attention layer on a 2K-token prompt.
        _layer("layer_fwd", 1, 2048, 12, 64, PAPER, name="layer_fwd_2k"),
        # A training step of one attention layer: four sequences of 8K tokens.
        _layer("layer_train", 4, 8192, 12, 64, "2048:1,4096:2,8192:4", name="layer_train_8k_b4"),
        # The layer's LayerNorm, both directions, and the weight and bias
        # gradient of one projection, as single calls at the layer's shape.
        {"kind": "layer_norm", "rows": 32768, "E": 768, "name": "layer_norm_32k"},
        {"kind": "wgrad", "K": 32768, "M": 768, "N": 768, "name": "wgrad_32k"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _length(rng, lo, hi):
    n = _log_int(rng, lo, hi)
    if rng.random() < 0.5:  # a multiple of 64, otherwise as drawn
        n = max(lo, n // 64 * 64)
    return n


def _patterns(rng, N):
    """One to eight patterns of growing segment length and dilation."""
    w, r = rng.choice([128, 256, 512, 1024, 2048, 2048, 2048, 4096, rng.randint(100, 3000)]), 1
    a, b = rng.choice([2, 2, 4]), rng.choice([2, 2, 3, 4])
    out = []
    for _ in range(rng.randint(1, 8)):
        out.append((w, min(r, w)))
        if w >= N:
            break
        w, r = w * a, r * b
    return ",".join("%d:%d" % p for p in out)


def draw(rng):
    kind = rng.choice(["fwd", "fwd", "fwd", "fwd_f32", "bwd", "bwd", "layer_fwd", "layer_train", "layer_norm", "wgrad"])
    while True:
        if kind == "layer_norm":
            return {"kind": kind, "rows": _log_int(rng, 1, 65536), "E": 8 * rng.randint(4, 256)}
        if kind == "wgrad":
            return {"kind": kind, "K": _log_int(rng, 64, 65536), "M": 128 * rng.randint(1, 16), "N": 128 * rng.randint(1, 16)}
        B, D = rng.choice([1, 1, 2, 3]), rng.choice([32, 64, 64, 128])
        causal = rng.random() < 0.8
        if kind.startswith("layer"):
            H = rng.randint(1, 2048 // D)
            if rng.random() < 0.75:  # most models have widths of whole 128 columns
                H = max(1, H * D // 128) * 128 // D
            N = _length(rng, 256, 16384)  # xPos scales grow with N: beyond, the gradients lose accuracy
            c = _layer(kind, B, N, H, D, _patterns(rng, N))  # causal: xPos without a mask saturates the softmax
            most = 1e13
        elif kind == "fwd_f32":
            N = _length(rng, 256, 8192)
            c = _attn("fwd", B, N, rng.randint(1, 16), D, _patterns(rng, N), "f32", causal)
            most = 5e10
        else:
            N = _length(rng, 256, 1048576)
            c = _attn(kind, B, N, rng.randint(1, 16), D, _patterns(rng, N), "bf16", causal, rng.choice([0.5, 1.0, 1.0, 2.0]))
            most = 4e13 if kind == "fwd" else 5e12
        need = work(c)
        if need["flops"] <= most and need["bytes"] <= 1.6e10:
            return c


# ---------------------------------------------------------------------------
# Inputs and calls
# ---------------------------------------------------------------------------
def _pats(case):
    return [tuple(int(x) for x in p.split(":")) for p in case["patterns"].split(",")]


class _Draw:
    """Seeded Gaussian tensors on the GPU, drawn in chunks."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed * 1000003 + 17)

    def __call__(self, shape, dtype, sigma=1.0, mean=0.0):
        n = math.prod(shape)
        out = torch.empty(n, dtype=dtype, device="cuda")
        for lo in range(0, n, 1 << 27):
            hi = min(n, lo + (1 << 27))
            x = torch.randn(hi - lo, generator=self.gen, device="cuda")
            out[lo:hi] = x.mul_(sigma).add_(mean) if mean else x.mul_(sigma)
        return out.view(shape)


def _attn_inputs(case, seed):
    d, shape = _Draw(seed), (case["B"], case["N"], case["H"], case["D"])
    dt = DTYPES[case["dtype"]]
    names = ("q", "k", "v") if case["kind"] == "fwd" else ("q", "k", "v", "dout")
    return {n: d(shape, dt, 1.0 if n == "dout" else case["sigma"]) for n in names}


PARAMS = ("ln_in.weight", "ln_in.bias", "q_proj.weight", "q_proj.bias", "k_proj.weight", "k_proj.bias", "v_proj.weight",
          "v_proj.bias", "ln_sub.weight", "ln_sub.bias", "out_proj.weight", "out_proj.bias")


def _layer_inputs(case, seed):
    d, E = _Draw(seed), case["H"] * case["D"]
    bf = torch.bfloat16
    t = {"x": d((case["B"], case["N"], E), bf), "dy": d((case["B"], case["N"], E), bf)}
    for name in PARAMS:
        if name.startswith("ln_"):
            t[name] = d((E,), bf, 0.1, 1.0 if name.endswith("weight") else 0.0)
        elif name.endswith("weight"):
            t[name] = d((E, E), bf, E ** -0.5)
        else:
            t[name] = d((E,), bf, 0.1)
    return t


def _layer_norm_inputs(case, seed):
    d, bf, shape = _Draw(seed), torch.bfloat16, (case["rows"], case["E"])
    return {"x": d(shape, bf), "dy": d(shape, bf), "weight": d(shape[1:], bf, 0.1, 1.0), "bias": d(shape[1:], bf, 0.1)}


def _wgrad_inputs(case, seed):
    d, bf = _Draw(seed), torch.bfloat16
    return {"dy": d((case["K"], case["M"]), bf), "x": d((case["K"], case["N"]), bf)}


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("fwd", "bwd"):
        s = _attn_inputs(case, seed)
        if kind == "bwd":
            s["out"], s["lse"] = da.dilated_attn(s["q"], s["k"], s["v"], _pats(case), case["causal"])
        s["patterns"] = _pats(case)
    elif kind.startswith("layer_") and kind != "layer_norm":
        t = _layer_inputs(case, seed)
        layer = LongNetAttention(case["H"] * case["D"], case["H"], _pats(case), case["causal"], device="cuda")
        params = dict(layer.named_parameters())
        with torch.no_grad():
            for name in PARAMS:
                params[name].copy_(t[name])
        s = {"layer": layer, "x": t["x"], "dy": t["dy"], "params": [params[n] for n in PARAMS]}
        if kind == "layer_train":
            s["x"].requires_grad_(True)
    elif kind == "layer_norm":
        s = _layer_norm_inputs(case, seed)
    else:
        s = _wgrad_inputs(case, seed)
    s["kind"], s["causal"] = kind, case.get("causal")
    return s


def run(s):
    kind = s["kind"]
    if kind == "fwd":
        out, lse = da.dilated_attn(s["q"], s["k"], s["v"], s["patterns"], s["causal"])
        return {"out": out, "lse": lse}
    if kind == "bwd":
        dq, dk, dv = da.dilated_attn_bwd(s["q"], s["k"], s["v"], s["out"], s["lse"], s["dout"], s["patterns"], s["causal"])
        return {"dq": dq, "dk": dk, "dv": dv}
    if kind == "layer_fwd":
        with torch.no_grad():
            return s["layer"](s["x"])
    if kind == "layer_train":
        y = s["layer"](s["x"])
        grads = torch.autograd.grad(y, [s["x"], *s["params"]], s["dy"])
        return {"y": y, "grads": list(grads)}
    if kind == "layer_norm":
        y, mean, rstd = da.layer_norm(s["x"], s["weight"], s["bias"])
        dx, dw, db = da.layer_norm_bwd(s["dy"], s["x"], s["weight"], mean, rstd)
        return {"y": y, "mean": mean, "rstd": rstd, "dx": dx, "dw": dw, "db": db}
    dw, db = da.wgrad(s["dy"], s["x"], bias_grad=True)
    return {"dw": dw, "db": db}


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
def _kept(length, s, r):
    return (length - s + r - 1) // r if length > s else 0


def _pairs(case):
    """(query, key) pairs of all patterns, heads and batches."""
    N, H, total = case["N"], case["H"], 0
    for w, r in _pats(case):
        w = min(w, N)
        for h in range(H):
            for count, length in ((N // w, w), (1, N % w)):
                L = _kept(length, h % r, r)
                total += count * (L * (L + 1) // 2 if case["causal"] else L * L)
    return case["B"] * total


def work(case):
    kind = case["kind"]
    if kind == "layer_norm":
        n = case["rows"] * case["E"]
        return {"bytes": 4 * n * 2 + 16 * case["rows"] + 8 * case["E"], "flops": 24 * n}
    if kind == "wgrad":
        K, M, N = case["K"], case["M"], case["N"]
        return {"bytes": 2 * (K * (M + N) + M * N + M), "flops": 2 * K * M * N + K * M}
    T, D = case["B"] * case["N"] * case["H"], case["D"]
    pairs = _pairs(case)
    if kind == "fwd":
        return {"bytes": T * (4 * D * (4 if case["dtype"] == "f32" else 2) + 4), "flops": 4 * D * pairs}
    if kind == "bwd":
        return {"bytes": T * (8 * D * 2 + 4), "flops": 10 * D * pairs}
    E = case["H"] * D
    rows = case["B"] * case["N"]
    if kind == "layer_fwd":
        return {"bytes": 2 * (2 * rows * E + 4 * E * E), "flops": 8 * rows * E * E + 4 * D * pairs}
    return {"bytes": 2 * (4 * rows * E + 8 * E * E), "flops": 24 * rows * E * E + 14 * D * pairs}


def tolerance(case):
    """About four times the error against float64 that the paths show: bf16
    inputs, probabilities and outputs with float32 sums (2e-3 to 2.5e-3, 4e-3
    for sharp scores), or float32 throughout (up to 7e-7 against the 1e-5 of
    sums in any order).  A layer rounds every intermediate tensor to bf16
    (gradients 7e-3 off, the key bias's, whose terms nearly cancel, 9e-3)."""
    kind = case["kind"]
    if kind == "fwd":
        return {"rel": 1e-5, "max": 1e-3} if case["dtype"] == "f32" else {"rel": 1e-2, "max": 0.2}
    if kind == "bwd":
        return {"rel": 1e-2, "max": 0.4}
    if kind == "layer_norm" or kind == "wgrad":
        return {"rel": 7e-3, "max": 0.1}
    return {"rel": 2.5e-2, "max": 0.5}


# ---------------------------------------------------------------------------
# The same outputs in float64, with plain torch operations
# ---------------------------------------------------------------------------
def _segments(N, w, s, r):
    """Index tensors [segments, L] of the kept rows: full segments, then the tail."""
    w = min(w, N)
    for first, count, length in ((0, N // w, w), (N // w, 1, N % w)):
        L = _kept(length, s, r)
        if L:
            g = torch.arange(first, first + count, device="cuda")[:, None] * w
            yield g + s + r * torch.arange(L, device="cuda")[None, :]


def _blocks(case):
    """(head, row indices [segments, L]) of every pattern, a bounded number of scores each."""
    for w, r in _pats(case):
        for h in range(case["H"]):
            for idx in _segments(case["N"], w, h % r, r):
                step = max(1, (1 << 27) // (case["B"] * idx.shape[1] ** 2))
                for lo in range(0, idx.shape[0], step):
                    yield h, idx[lo:lo + step]


def _scores(case, q, k):
    S = (q @ k.transpose(-1, -2).contiguous()) * case["D"] ** -0.5
    if case["causal"]:
        L = S.shape[-1]
        S.masked_fill_(torch.ones(L, L, dtype=torch.bool, device="cuda").triu(1), -math.inf)
    return S


def _mix64(case, q, k, v):
    """out [B, N, H, D] and lse [B, N, H] in float64."""
    out, lse = torch.zeros_like(q), torch.full(q.shape[:3], -math.inf, dtype=q.dtype, device="cuda")
    for h, idx in _blocks(case):
        S = _scores(case, q[:, idx, h], k[:, idx, h])
        li = torch.logsumexp(S, -1)
        oi = S.sub_(li[..., None]).exp_() @ v[:, idx, h]
        old = lse[:, idx, h]
        new = torch.logaddexp(old, li)
        out[:, idx, h] = out[:, idx, h] * (old - new).exp()[..., None] + oi * (li - new).exp()[..., None]
        lse[:, idx, h] = new
    return out, lse


class _Attention64(torch.autograd.Function):
    @staticmethod
    def forward(ctx, q, k, v, case):
        out, lse = _mix64(case, q, k, v)
        ctx.save_for_backward(q, k, v, out, lse)
        ctx.case = case
        return out

    @staticmethod
    def backward(ctx, dout):
        q, k, v, out, lse = ctx.saved_tensors
        case, sc = ctx.case, ctx.case["D"] ** -0.5
        dq, dk, dv = torch.zeros_like(q), torch.zeros_like(q), torch.zeros_like(q)
        delta = (dout * out).sum(-1)
        for h, idx in _blocks(case):
            qs, ks, vs, gs = (t[:, idx, h] for t in (q, k, v, dout))
            P = _scores(case, qs, ks).sub_(lse[:, idx, h][..., None]).exp_()
            dv[:, idx, h] += P.transpose(-1, -2).contiguous() @ gs
            dS = P.mul_(gs @ vs.transpose(-1, -2).contiguous() - delta[:, idx, h][..., None])
            dq[:, idx, h] += (dS @ ks) * sc
            dk[:, idx, h] += (dS.transpose(-1, -2).contiguous() @ qs) * sc
        return dq, dk, dv, None


def _xpos64(x, sign):
    B, N, H, D = x.shape
    i = torch.arange(D // 2, dtype=torch.float64, device="cuda")
    n = torch.arange(N, dtype=torch.float64, device="cuda")[:, None]
    ang = n * 10000.0 ** (-2.0 * i / D)
    scl = ((2.0 * i / D + 0.4) / 1.4) ** (sign * (n - N // 2) / 512.0)
    cs, sn = (ang.cos() * scl)[None, :, None], (ang.sin() * scl)[None, :, None]
    x0, x1 = x[..., 0::2], x[..., 1::2]
    return torch.stack((x0 * cs - x1 * sn, x0 * sn + x1 * cs), -1).reshape(x.shape)


def _layer64(case, x, p):
    B, N, E = x.shape
    lin = torch.nn.functional.linear
    norm = torch.nn.functional.layer_norm
    u = norm(x, (E,), p["ln_in.weight"], p["ln_in.bias"], 1e-5)
    q, k, v = (lin(u, p[n + ".weight"], p[n + ".bias"]).view(B, N, case["H"], case["D"]) for n in ("q_proj", "k_proj", "v_proj"))
    a = _Attention64.apply(_xpos64(q, 1), _xpos64(k, -1), v, case).reshape(B, N, E)
    return lin(norm(a, (E,), p["ln_sub.weight"], p["ln_sub.bias"], 1e-5), p["out_proj.weight"], p["out_proj.bias"])


def exact(case, seed):
    kind = case["kind"]
    if kind == "layer_norm":
        t = {n: x.double() for n, x in _layer_norm_inputs(case, seed).items()}
        mean, var = t["x"].mean(1), t["x"].var(1, unbiased=False)
        rstd = (var + 1e-5).rsqrt()
        xh = (t["x"] - mean[:, None]) * rstd[:, None]
        g = t["dy"] * t["weight"]
        dx = rstd[:, None] * (g - g.mean(1, keepdim=True) - xh * (g * xh).mean(1, keepdim=True))
        return {"y": xh * t["weight"] + t["bias"], "mean": mean, "rstd": rstd, "dx": dx, "dw": (t["dy"] * xh).sum(0),
                "db": t["dy"].sum(0)}
    if kind == "wgrad":
        t = _wgrad_inputs(case, seed)
        dy, x = t["dy"].double(), t["x"].double()
        return {"dw": dy.t().contiguous() @ x, "db": dy.sum(0)}
    tensor = case["B"] * case["N"] * case["H"] * case["D"]
    if _pairs(dict(case, causal=False)) > 4e10 or tensor > 4e8:
        return None  # minutes in float64
    if kind in ("fwd", "bwd"):
        t = {n: x.double() for n, x in _attn_inputs(case, seed).items()}
        if kind == "fwd":
            out, lse = _mix64(case, t["q"], t["k"], t["v"])
            return {"out": out, "lse": lse.permute(0, 2, 1).contiguous()}
        q, k, v = (t[n].requires_grad_(True) for n in ("q", "k", "v"))
        dq, dk, dv = torch.autograd.grad(_Attention64.apply(q, k, v, case), [q, k, v], t["dout"])
        return {"dq": dq, "dk": dk, "dv": dv}
    t = {n: x.double() for n, x in _layer_inputs(case, seed).items()}
    if kind == "layer_fwd":
        return _layer64(case, t["x"], t)
    leaves = [t[n].requires_grad_(True) for n in ("x", *PARAMS)]
    y = _layer64(case, t["x"], t)
    return {"y": y.detach(), "grads": list(torch.autograd.grad(y, leaves, t["dy"]))}
