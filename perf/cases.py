"""The work a user has this framework do, as a list of timed cases.

Every case is one adapted linear layer (or one pass over it) through a public entry point: the autograd modules for
training, the C ABI binding where a serving loop or a quantised layer calls it.  Sizes are those of the workload
table in paper_2312_03415_amd/synth.py and of the tests, and generic ones between them.

    kind    entry point                                              a pass returns
    serve   binding.runlora_forward into buffers kept by the caller  y
    train   RunLoRALinear forward + backward (RunLoRAFunction with   y, dx, dA, dB
            an explicit seed when LoRA dropout is on)
    int4    binding.runlora_forward + runlora_backward on an         y, dx, dA, dB
            Int4Weight, buffers kept by the caller
    dora    RunDoRALinear forward + backward                         y, dx, dA, dB, dm
    vera    RunVeRALinear forward + backward                         y, dx, dd, db

Values are those the layers meet in training: X, dY ~ N(0, 1), W, A ~ N(0, 1/i), B ~ N(0, 0.1/r), drawn on the GPU
from the seed.
"""
import math

import torch

from paper_2312_03415_amd import binding as rl
from paper_2312_03415_amd.module import RunDoRALinear, RunLoRAFunction, RunLoRALinear, RunVeRALinear

DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}


def _case(kind, n, i, o, r, dtype="bf16", bias=False, alpha=None, dropout=0.0, name=None):
    c = dict(kind=kind, n=n, i=i, o=o, r=r, dtype=dtype, bias=bias, alpha=float(alpha if alpha is not None else r), dropout=dropout)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one token through an attention projection while generating: latency of a single small call
        _case("serve", 1, 4096, 4096, 16, alpha=32, name="serve_1x4096x4096"),
        # a batch of 48 sequences generating one token each, through the wide projection of a gated MLP
        _case("serve", 48, 4096, 11008, 32, name="serve_48x4096x11008"),
        # the smallest training layer of the workload table, the fp32 path
        _case("train", 256, 768, 768, 8, "f32", name="train_f32_256x768x768"),
        # a short fp16 batch (one row of the selector sweep)
        _case("train", 1024, 4096, 4096, 64, "f16", alpha=128, name="train_f16_1024x4096x4096"),
        # a batch of unpadded sequences and widths that are no multiple of a tile
        _case("train", 1237, 2056, 5464, 24, bias=True, alpha=48, name="train_1237x2056x5464"),
        # the MLP pair of the middle-sized workload: up projection, and down projection with LoRA dropout
        _case("train", 4096, 2048, 8192, 16, bias=True, alpha=32, name="train_4096x2048x8192"),
        _case("train", 4096, 8192, 2048, 16, bias=True, alpha=32, dropout=0.1, name="train_drop_4096x8192x2048"),
        # the large workload: an attention projection, and the wide MLP projection at a high rank
        _case("train", 8192, 4096, 4096, 32, name="train_8192x4096x4096"),
        _case("train", 8192, 4096, 11008, 128, name="train_8192x4096x11008"),
        # training adapters over a 4-bit frozen weight
        _case("int4", 4096, 5120, 13824, 64, name="int4_4096x5120x13824"),
        # the two other adapter families on the middle-sized workload
        _case("dora", 4096, 2048, 8192, 16, alpha=32, name="dora_4096x2048x8192"),
        _case("vera", 4096, 2048, 8192, 256, name="vera_4096x2048x8192"),
    ]


def _log(rng, lo, hi, step=1):
    """A multiple of `step` in [lo, hi], spread over its logarithm."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)) * step
    return max(lo, min(hi, v))


def _width(rng, step, lo=512, hi=11008):
    """A layer width: half of them as models have them (multiples of 256), half any width the library takes."""
    return _log(rng, lo, hi, 256) if rng.random() < 0.5 else _log(rng, lo, hi, step)


def draw(rng):
    kind = rng.choices(["serve", "train", "int4", "dora", "vera"], [5, 10, 2, 2, 2])[0]
    dtype = rng.choices(["bf16", "f16", "f32"], [6, 2, 1])[0] if kind == "train" else rng.choice(["bf16", "bf16", "f16"])
    step = 4 if dtype == "f32" else 8
    i, o = _width(rng, step), _width(rng, step)
    n = _log(rng, 1, 256) if kind == "serve" else _log(rng, 200, 8192)
    if rng.random() < 0.4 and n >= 64:
        n = (n + 63) // 64 * 64  # padded batches
    r = rng.choice([8, 16, 24, 32, 48, 64, 128, 8, 16, 32, 64, 256])
    dropout = 0.0
    if kind == "vera":
        r = rng.choice([64, 128, 256])
    if kind == "dora" or (kind == "train" and rng.random() < 0.25):
        r = min(r, 128)
        dropout = 0.1 if kind == "train" else 0.0
    if kind == "int4":
        i, o = max(i, 1024), max(o, 1024)
    # fp32 products take about ten times as long as 16-bit ones; DoRA and int4 layers read more than the others
    cap = {"f32": 1.0e10}.get(dtype, {"dora": 2.0e11, "int4": 2.9e11}.get(kind, 3.6e11))
    while n * i * o > cap:
        n = max(1, n // 2)
    return _case(kind, n, i, o, r, dtype, bias=rng.random() < 0.4, alpha=r * rng.choice([1, 2]), dropout=dropout)


# ---- inputs ------------------------------------------------------------------------------------------

def _inputs(case, seed):
    """Everything a pass reads, from the seed alone (same values wherever it is called)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    n, i, o, r = case["n"], case["i"], case["o"], case["r"]
    dt = DTYPES[case["dtype"]]

    def normal(shape, var):
        return (torch.randn(shape, generator=g, device="cuda") * math.sqrt(var)).to(dt)

    t = dict(X=normal((n, i), 1.0), A=normal((i, r), 1.0 / i), B=normal((r, o), 0.1 / r))
    if case["kind"] == "int4":
        t["q"] = torch.randint(-7, 8, (i, o), generator=g, device="cuda", dtype=torch.int8)
        u = torch.rand(((i + 63) // 64, o), generator=g, device="cuda")
        t["scales"] = ((0.5 + u) / (4.32 * math.sqrt(i))).half()
    else:
        t["W"] = normal((i, o), 1.0 / i)
    if case["kind"] != "serve":
        t["dY"] = normal((n, o), 1.0)
    t["bias"] = normal((o,), 0.01) if case["bias"] else None
    if case["kind"] == "vera":
        # A and B random and shared, d and b some way from where they start (0.1 and 0)
        t["B"] = normal((r, o), 1.0 / r)
        t["d"] = (0.1 + 0.02 * torch.randn(r, generator=g, device="cuda")).to(dt)
        t["b"] = normal((o,), 0.25)
    if case["kind"] == "dora":
        m = t["W"].float().norm(dim=0)
        t["m"] = (m * (1.0 + 0.05 * torch.randn(o, generator=g, device="cuda"))).to(dt)
    t["drop_seed"] = int(seed) & 0x7FFFFFFF
    return t


def _scale(case):
    return 1.0 if case["kind"] == "vera" else case["alpha"] / case["r"]


def prepare(case, seed):
    t = _inputs(case, seed)
    kind, n, i, o, r = case["kind"], case["n"], case["i"], case["o"], case["r"]
    code = rl.dtype_code(DTYPES[case["dtype"]])
    s = dict(case=case, t=t)
    if kind in ("serve", "int4"):
        like = t["X"]
        s["y"] = like.new_empty((n, o))
        if kind == "serve":
            s["pair"] = pair = rl.runlora_select(n, i, o, r, code)
            s["ws"] = rl.new_workspace(pair[0], -1, n, i, o, r, code)
        else:
            q = t.pop("q").to(torch.int16) + 8
            t["W"] = rl.Int4Weight((q[:, 0::2] | (q[:, 1::2] << 4)).to(torch.uint8), t.pop("scales"), i, o)
            s["pair"] = pair = rl.runlora_select(n, i, o, r, rl.RL_INT4_G64)
            s["ws"] = rl.new_workspace(pair[0], pair[1], n, i, o, r, code, w_dtype=rl.RL_INT4_G64)
            s.update(dx=like.new_empty((n, i)), dA=like.new_empty((i, r)), dB=like.new_empty((r, o)))
        s["T"] = like.new_empty((n, r)) if pair[0] == rl.FWD_DEFAULT else None
        return s
    t["X"].requires_grad_(True)
    if kind == "train":
        layer = RunLoRALinear(t["W"], r, case["alpha"], t["bias"], dropout=case["dropout"])
    elif kind == "dora":
        layer = RunDoRALinear(t["W"], r, case["alpha"], t["bias"])
    else:
        layer = RunVeRALinear(t["W"], t["A"], t["B"], t["bias"])
    with torch.no_grad():
        if kind == "vera":
            layer.vera_d.copy_(t["d"])
            layer.vera_b.copy_(t["b"])
        else:
            layer.lora_A.copy_(t["A"])
            layer.lora_B.copy_(t["B"])
        if kind == "dora":
            layer.dora_m.copy_(t["m"])
    s["layer"] = layer
    return s


def run(state):
    case, t = state["case"], state["t"]
    kind = case["kind"]
    if kind == "serve":
        rl.runlora_forward(state["pair"][0], t["X"], t["W"], t["A"], t["B"], state["y"], rl.new_saved(state["T"]), workspace=state["ws"],
                           scale=_scale(case), bias=t["bias"])
        return state["y"]
    if kind == "int4":
        saved = rl.new_saved(state["T"])
        rl.runlora_forward(state["pair"][0], t["X"], t["W"], t["A"], t["B"], state["y"], saved, workspace=state["ws"], scale=_scale(case),
                           bias=t["bias"])
        rl.runlora_backward(state["pair"][1], t["dY"], saved, t["W"], t["A"], t["B"], state["dx"], state["dA"], state["dB"],
                            workspace=state["ws"])
        return state["y"], state["dx"], state["dA"], state["dB"]
    layer, x = state["layer"], t["X"]
    if kind == "train" and case["dropout"] > 0.0:
        # the layer's own function with the mask's seed given, so that a pass can be repeated
        y = RunLoRAFunction.apply(x, layer.weight, layer.lora_A, layer.lora_B, layer.bias, layer.scale, (1, 1), False,
                                  (case["dropout"], t["drop_seed"]))
    else:
        y = layer(x)
    if kind == "vera":
        params = (layer.vera_d, layer.vera_b)
    elif kind == "dora":
        params = (layer.lora_A, layer.lora_B, layer.dora_m)
    else:
        params = (layer.lora_A, layer.lora_B)
    grads = torch.autograd.grad(y, (x,) + params, t["dY"])
    return (y.detach(),) + grads


# ---- what a pass needs, and what it should give ---------------------------------------------------------

def work(case):
    kind, n, i, o, r = case["kind"], case["n"], case["i"], case["o"], case["r"]
    e = 4 if case["dtype"] == "f32" else 2
    w = (i * o / 2 + (i + 63) // 64 * o * 2) if kind == "int4" else i * o * e
    factors = r * (i + o) * e
    fwd = 2.0 * n * (i * o + r * (i + o))
    if kind == "serve":
        return {"bytes": float(e * n * (i + o) + w + factors), "flops": fwd}
    # with X A kept: dY B^T, (.) A^T, dA and dB
    flops = fwd + 2.0 * n * (i * o + 2 * r * (i + o))
    if kind == "vera":
        flops -= 2.0 * n * i * r  # no gradient for A
        return {"bytes": float(2 * e * n * (i + o) + w + factors + 2 * e * (r + o)), "flops": flops}
    if kind == "dora":
        # the merged weight is formed for its column norms: Y = X M, dX = dY M^T, and the rank-r gradients
        flops = 4.0 * n * i * o + 2.0 * r * i * o + 4.0 * n * r * (i + o)
    return {"bytes": float(2 * e * n * (i + o) + w + 2 * factors), "flops": flops}


def tolerance(case):
    # about four times the largest errors measured against exact() over the listed and 24 drawn cases (2-norm /
    # per element): bf16 3.0e-3 / 1.3e-2, f16 4.1e-4 / 1.3e-3, f32 7.0e-7 / 3.0e-6
    rel, most = {"bf16": (1e-2, 5e-2), "f16": (1.6e-3, 6e-3), "f32": (3e-6, 1.2e-5)}[case["dtype"]]
    return {"rel": rel, "max": most}


def _keep_mask(n, i, p, seed):
    """The documented LoRA dropout mask (runlora.h): float64 [n, i] of 0 / 1, and the kept share's inverse."""
    def mix(x):
        x = x ^ (x >> 16)
        x = (x * 0x7FEB352D) & 0xFFFFFFFF
        x = x ^ (x >> 15)
        x = (x * 0x846CA68B) & 0xFFFFFFFF
        return x ^ (x >> 16)

    thr = min(255, max(1, int(p * 256.0 + 0.5)))
    key = mix(torch.tensor((seed & 0xFFFFFFFF) ^ 0x9E3779B9, dtype=torch.int64, device="cuda"))
    h = mix(torch.arange(n * (i // 4), dtype=torch.int64, device="cuda") ^ key)
    keep = torch.stack([((h >> (8 * k)) & 255) >= thr for k in range(4)], dim=1).reshape(n, i)
    return keep.double(), 256.0 / (256 - thr)


def exact(case, seed):
    t = _inputs(case, seed)
    kind, n, i, o, s = case["kind"], case["n"], case["i"], case["o"], _scale(case)
    X, A, B = t["X"].double(), t["A"].double(), t["B"].double()
    if kind == "int4":
        W = t["q"].double() * t["scales"].double().repeat_interleave(64, dim=0)[:i]
    else:
        W = t["W"].double()
    bias = t["bias"].double() if t["bias"] is not None else torch.zeros(o, dtype=torch.float64, device="cuda")
    if kind == "serve":
        return X @ W + s * ((X @ A) @ B) + bias
    dY = t["dY"].double()
    if kind == "dora":
        V = W + s * (A @ B)
        c = V.norm(dim=0)
        g = t["m"].double() / c
        XV, G = X @ V, dY * g
        GB = G @ B.t()
        return (XV * g + bias, G @ V.t(), s * (X.t() @ GB), s * ((X @ A).t() @ G), (dY * XV).sum(0) / c)
    if kind == "vera":
        d, b = t["d"].double(), t["b"].double()
        T, H = X @ A, (dY * b) @ B.t()
        return (X @ W + s * (((T * d) @ B) * b) + bias, dY @ W.t() + s * ((H * d) @ A.t()), s * (T * H).sum(0),
                s * (dY * ((T * d) @ B)).sum(0))
    if case["dropout"] > 0.0:
        keep, q = _keep_mask(n, i, case["dropout"], t["drop_seed"])
        s = s * q
        Xm = X * keep
    else:
        keep, Xm = 1.0, X
    T, Z = Xm @ A, dY @ B.t()
    return (X @ W + s * (T @ B) + bias, dY @ W.t() + keep * (s * (Z @ A.t())), s * (Xm.t() @ Z), s * (T.t() @ dY))
