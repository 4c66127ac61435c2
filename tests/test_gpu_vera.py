"""GPU parity of the VeRA entry points (frozen A, B; trainable vectors d, b; the paper's conclusion names VeRA
among the adapters its method carries over to): Y, dX, dd, db of every computation graph against the fp64
oracle of the layer's definition (oracle.vera_forward / vera_backward), the reduction to the LoRA calls
for d = 1, b = 1, skipped outputs, and one full-size layer."""
import numpy as np
import pytest

import oracle
from helpers import TOL, layer_on_device, relerr, to_device, to_f64, torch_dtype
from paper_2312_03415_amd import binding as rl
from paper_2312_03415_amd import synth
from test_gpu_parity import legal_pairs

pytestmark = pytest.mark.gpu


def vectors(L, ones=False):
    out = {}
    for name, count, stream in (("d", L.r, 10), ("b", L.o, 11), ("bias", L.o, 9)):
        v = np.ones(count) if (ones and name != "bias") else synth.normal(synth.BASE_SEED + L.index, stream, (count,))
        st = synth.store(v, L.dtype)
        out[name] = (to_device(st, L.dtype), synth.widen(st, L.dtype))
    return out


def run_vera(L, dev, vec, fwd, bwd, scale, bias, want=("dX", "dd", "db")):
    import torch
    td = torch_dtype(L.dtype)
    code = rl.dtype_from_name(L.dtype)
    nan = float("nan")
    Y = torch.full((L.n, L.o), nan, dtype=td, device="cuda")
    T = torch.full((L.n, L.r), nan, dtype=td, device="cuda") if fwd == rl.FWD_DEFAULT else None
    saved = rl.new_saved(T)
    ws = torch.empty(max(rl.runlora_vera_workspace_bytes(fwd, bwd, L.n, L.i, L.o, L.r, code), 256), dtype=torch.uint8, device="cuda")
    d, b = vec["d"][0], vec["b"][0]
    rl.runlora_vera_forward(fwd, dev["X"], dev["W"], dev["A"], dev["B"], d, b, Y, saved, ws, scale=scale, bias=bias)
    ws.fill_(0xFF)  # nothing the forward left in the workspace may matter to the backward
    dX = torch.full((L.n, L.i), nan, dtype=td, device="cuda") if "dX" in want else None
    dd = torch.full((L.r,), nan, dtype=td, device="cuda") if "dd" in want else None
    db = torch.full((L.o,), nan, dtype=td, device="cuda") if "db" in want else None
    rl.runlora_vera_backward(bwd, dev["dY"], saved, dev["W"], dev["A"], dev["B"], d, b, dX, dd, db, ws)
    torch.cuda.synchronize()
    out = {"Y": to_f64(Y)}
    for k, t in (("dX", dX), ("dd", dd), ("db", db)):
        if t is not None:
            out[k] = to_f64(t)
    return out


def vera_reference(host, vec, scale, with_bias=True):
    d, b, bias = vec["d"][1], vec["b"][1], vec["bias"][1]
    Y = oracle.vera_forward(host["X"], host["W"], host["A"], host["B"], d, b, scale, bias if with_bias else None)
    dX, dd, db = oracle.vera_backward(host["X"], host["W"], host["A"], host["B"], d, b, host["dY"], scale)
    return {"Y": Y, "dX": dX, "dd": dd, "db": db}


@pytest.mark.parametrize("dtype,r", [("bf16", 24), ("f16", 64), ("f32", 12), ("bf16", 264)])
def test_vera_all_pairs(dtype, r):
    """Ragged shape, every legal forward x backward pair, s = 0.5, a bias, random d and b.  r = 264 (VeRA runs
    at ranks of a few hundred) sends the rank-r products to the tile GEMM."""
    L = synth.Layer("vera", 301, 264, 328, r, dtype, 41)
    dev, host = layer_on_device(L)
    vec = vectors(L)
    want = vera_reference(host, vec, 0.5)
    for f, b in legal_pairs():
        print(f"case vera layer={L} fwd={f} bwd={b}", flush=True)
        got = run_vera(L, dev, vec, f, b, 0.5, vec["bias"][0])
        for k in ("Y", "dX", "dd", "db"):
            err = relerr(got[k], want[k])
            assert err < TOL[dtype], (f, b, k, err)


def test_vera_with_unit_vectors_is_the_lora_layer():
    """d = 1 and b = 1 make B~ = B exactly: Y and dX must be bit for bit what the LoRA calls give, and
    dd, db are then the row and column sums of dB o B."""
    import torch
    L = synth.Layer("vera1", 200, 136, 264, 16, "bf16", 42)
    dev, host = layer_on_device(L)
    vec = vectors(L, ones=True)
    code = rl.dtype_from_name(L.dtype)
    for f, b in [(1, 1), (2, 5), (0, 0), (1, 3)]:
        got = run_vera(L, dev, vec, f, b, None, None)
        Y = torch.empty((L.n, L.o), dtype=torch.bfloat16, device="cuda")
        T = torch.empty((L.n, L.r), dtype=torch.bfloat16, device="cuda") if f == rl.FWD_DEFAULT else None
        saved = rl.new_saved(T)
        ws = rl.new_workspace(f, b, L.n, L.i, L.o, L.r, code)
        rl.runlora_forward(f, dev["X"], dev["W"], dev["A"], dev["B"], Y, saved, workspace=ws)
        dX = torch.empty((L.n, L.i), dtype=torch.bfloat16, device="cuda")
        dB = torch.empty((L.r, L.o), dtype=torch.bfloat16, device="cuda")
        rl.runlora_backward(b, dev["dY"], saved, dev["W"], dev["A"], dev["B"], dX, None, dB, workspace=ws)
        torch.cuda.synchronize()
        assert np.array_equal(got["Y"], to_f64(Y)) and np.array_equal(got["dX"], to_f64(dX)), (f, b)
        G = to_f64(dB) * host["B"]
        assert relerr(got["dd"], G.sum(axis=1)) < 4e-3 and relerr(got["db"], G.sum(axis=0)) < 4e-3, (f, b)


def test_vera_skipped_outputs_and_zero_vectors():
    """Any of dX / dd / db may be skipped; the others do not change.  d = 0 switches the adapter off but
    leaves a gradient for d (and none for b)."""
    import torch
    L = synth.Layer("vera2", 130, 72, 96, 8, "f16", 43)
    dev, host = layer_on_device(L)
    vec = vectors(L)
    full = run_vera(L, dev, vec, 1, 1, 1.0, None)
    for want in (("dd",), ("db",), ("dX",), ("dX", "db"), ()):
        part = run_vera(L, dev, vec, 1, 1, 1.0, None, want=want)
        assert set(part) == {"Y", *want}
        for k in part:
            assert np.array_equal(part[k], full[k]), (want, k)
    zero = dict(vec)
    zero["d"] = (torch.zeros_like(vec["d"][0]), np.zeros(L.r))
    got = run_vera(L, dev, zero, 1, 1, 1.0, None)
    ref = vera_reference(host, zero, 1.0, with_bias=False)
    assert relerr(got["Y"], ref["Y"]) < TOL["f16"] and relerr(got["dX"], ref["dX"]) < TOL["f16"]
    assert np.all(got["db"] == 0.0) and np.linalg.norm(ref["dd"]) > 0 and relerr(got["dd"], ref["dd"]) < TOL["f16"]


def test_vera_full_size_opt_fc1_rank256():
    """OPT-1.3B fc1 shape (n 4096, 2048 -> 8192, bf16) at a VeRA-sized rank, pair (1, 1): dd and db in
    full, Y and dX on sampled token rows (rows are independent; the oracle evaluates the layer on them)."""
    import torch
    L = synth.Layer("vera_fc1", 4096, 2048, 8192, 256, "bf16", 44)
    dev, host = layer_on_device(L)
    vec = vectors(L)
    d, b, bias = vec["d"][1], vec["b"][1], vec["bias"][1]
    got = run_vera(L, dev, vec, 1, 1, 0.25, vec["bias"][0])
    # dd and db do not involve W: evaluate the definition with the n x r and n x o factors only
    T = oracle.matmul(host["X"], host["A"])
    V = oracle.matmul(T * d[None, :], host["B"])
    db = 0.25 * np.sum(host["dY"] * V, axis=0)
    dU = oracle.matmul(0.25 * host["dY"] * b[None, :], host["B"], tb=True)
    dd = np.sum(T * dU, axis=0)
    assert relerr(got["dd"], dd) < TOL["bf16"] and relerr(got["db"], db) < TOL["bf16"]
    rng = np.random.default_rng(5)
    rows = np.unique(np.concatenate([np.arange(0, L.n, 512), np.arange(255, L.n, 512), rng.integers(0, L.n, 24)]))
    Yr = oracle.vera_forward(host["X"][rows], host["W"], host["A"], host["B"], d, b, 0.25, bias)
    dXr = oracle.matmul(host["dY"][rows], host["W"], tb=True) + oracle.matmul(dU[rows] * d[None, :], host["A"], tb=True)
    assert relerr(got["Y"][rows], Yr) < TOL["bf16"] and relerr(got["dX"][rows], dXr) < TOL["bf16"]


@pytest.mark.parametrize("r", [192, 256])
def test_vera_module_beyond_rank_128(r):
    """RunVeRALinear at 4096 x 4096 -> 4096, bf16: its backward forms no dA, so that Z1 and X A share a launch and dB runs alone, in the workspace
    that the module asks for.  All of dd and db, sampled rows of dX, in fp32 from the same operands."""
    import torch
    from paper_2312_03415_amd.module import RunVeRALinear
    n, i, o = 4096, 4096, 4096
    L = synth.Layer("vera_module", n, i, o, r, "bf16", 45)
    dev, _ = layer_on_device(L)
    vec = vectors(L)
    layer = RunVeRALinear(dev["W"], dev["A"], dev["B"], scale=0.25, pair=(1, 1))
    with torch.no_grad():
        layer.vera_d.copy_(vec["d"][0])
        layer.vera_b.copy_(vec["b"][0])
    x = dev["X"].clone().requires_grad_()
    layer(x).backward(dev["dY"])
    torch.cuda.synchronize()
    X, A, B, dY, d, b = (t.detach().float() for t in (dev["X"], dev["A"], dev["B"], dev["dY"], layer.vera_d, layer.vera_b))
    T, U = X @ A, 0.25 * (dY * b) @ B.t().contiguous()
    rows = torch.arange(0, n, 61, device="cuda")
    dX = dY[rows] @ dev["W"].float().t().contiguous() + (U[rows] * d) @ A.t().contiguous()
    for got, want in ((layer.vera_d.grad, (T * U).sum(0)), (layer.vera_b.grad, 0.25 * (dY * ((T * d) @ B)).sum(0)), (x.grad[rows], dX)):
        assert relerr(to_f64(got), to_f64(want)) < TOL["bf16"]
