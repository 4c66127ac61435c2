"""GPU parity for a frozen W stored as symmetric int4 with group-of-64 fp16 scales (the quantised
configuration of the task; the paper mentions quantised weights in one sentence of Section 1):
every graph that does not need W + AB as a matrix, through the C ABI, against the fp64 oracle
evaluated on the dequantised W = q * scale."""
import numpy as np
import pytest

import oracle
from helpers import TOL, relerr, to_device, to_f64, torch_dtype
from paper_2312_03415_amd import binding as rl
from paper_2312_03415_amd import synth

pytestmark = pytest.mark.gpu

PAIRS = [(0, 0), (1, 1), (1, 2), (1, 3), (0, 0), (1, 1)]


def make_layer(L, q=None, scale=None):
    st = synth.layer_inputs(L)
    if q is None:
        q, scale = synth.int4_weight(L)
    dev = {k: to_device(v, L.dtype) for k, v in st.items() if k != "W"}
    host = {k: synth.widen(v, L.dtype) for k, v in st.items() if k != "W"}
    dev["W"] = rl.Int4Weight.from_host(q, scale)
    host["W"] = oracle.dequant_int4(q, scale.astype(np.float64))
    return dev, host


def run_pair(L, dev, fwd, bwd):
    import torch
    td = torch_dtype(L.dtype)
    code = rl.dtype_from_name(L.dtype)
    nan = float("nan")
    Y = torch.full((L.n, L.o), nan, dtype=td, device="cuda")
    T = torch.full((L.n, L.r), nan, dtype=td, device="cuda") if fwd == 0 else None
    saved = rl.new_saved(T)
    ws = rl.new_workspace(fwd, bwd, L.n, L.i, L.o, L.r, code, w_dtype=rl.RL_INT4_G64)
    rl.runlora_forward(fwd, dev["X"], dev["W"], dev["A"], dev["B"], Y, saved, workspace=ws)
    dX = torch.full((L.n, L.i), nan, dtype=td, device="cuda")
    dA = torch.full((L.i, L.r), nan, dtype=td, device="cuda")
    dB = torch.full((L.r, L.o), nan, dtype=td, device="cuda")
    rl.runlora_backward(bwd, dev["dY"], saved, dev["W"], dev["A"], dev["B"], dX, dA, dB, workspace=ws)
    torch.cuda.synchronize()
    return {"Y": to_f64(Y), "dX": to_f64(dX), "dA": to_f64(dA), "dB": to_f64(dB)}


def direct_workspace(dev, L, fwd, bwd=None):
    """A workspace of what the call needs without dequantised panels of W: the figure in its refusal of a smaller one."""
    import re

    import torch
    td = torch_dtype(L.dtype)
    tiny = torch.empty(256, dtype=torch.uint8, device="cuda")
    Y = torch.empty((L.n, L.o), dtype=td, device="cuda")
    saved = rl.new_saved()
    with pytest.raises(rl.RunLoRAError) as e:
        if bwd is None:
            rl.runlora_forward(fwd, dev["X"], dev["W"], dev["A"], dev["B"], Y, saved, workspace=tiny)
        else:
            full = rl.new_workspace(fwd, bwd, L.n, L.i, L.o, L.r, rl.dtype_from_name(L.dtype), w_dtype=rl.RL_INT4_G64)
            rl.runlora_forward(fwd, dev["X"], dev["W"], dev["A"], dev["B"], Y, saved, workspace=full)
            rl.runlora_backward(bwd, dev["dY"], saved, dev["W"], dev["A"], dev["B"], torch.empty_like(dev["X"]), torch.empty_like(dev["A"]),
                                torch.empty_like(dev["B"]), workspace=tiny)
    assert e.value.code == rl.RL_ERR_WORKSPACE
    return torch.empty(int(re.search(r"(\d+) bytes", str(e.value)).group(1)), dtype=torch.uint8, device="cuda")


def reference(host):
    Y = oracle.reference_forward(host["X"], host["W"], host["A"], host["B"])
    dX, dA, dB = oracle.reference_backward(host["X"], host["W"], host["A"], host["B"], host["dY"])
    return {"Y": Y, "dX": dX, "dA": dA, "dB": dB}


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("shape", [(333, 264, 392, 24), (70, 72, 136, 8), (600, 520, 328, 16)])
def test_int4_weight_all_supported_pairs(shape, dtype):
    """Ragged shapes: d_in not a multiple of the group (a partial last group), several tiles."""
    n, i, o, r = shape
    L = synth.Layer("int4", n, i, o, r, dtype, 9)
    dev, host = make_layer(L)
    want = reference(host)
    for f, b in [(0, 0), (1, 1), (1, 2), (1, 3)]:
        print(f"case int4 shape={shape} dtype={dtype} fwd={f} bwd={b}", flush=True)
        got = run_pair(L, dev, f, b)
        for k in ("Y", "dX", "dA", "dB"):
            assert relerr(got[k], want[k]) < TOL[dtype], (f, b, k, relerr(got[k], want[k]))


def test_int4_merged_graphs_are_refused():
    L = synth.Layer("int4", 64, 64, 64, 8, "bf16", 9)
    dev, _ = make_layer(L)
    import torch
    Y = torch.empty((L.n, L.o), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    with pytest.raises(rl.RunLoRAError) as e:
        rl.runlora_forward(2, dev["X"], dev["W"], dev["A"], dev["B"], Y, rl.new_saved(), workspace=ws)
    assert e.value.code == rl.RL_ERR_UNSUPPORTED
    saved = rl.new_saved()
    rl.runlora_forward(1, dev["X"], dev["W"], dev["A"], dev["B"], Y, saved, workspace=ws)
    dX = torch.empty((L.n, L.i), dtype=torch.bfloat16, device="cuda")
    for bwd in (4, 5):
        with pytest.raises(rl.RunLoRAError) as e:
            rl.runlora_backward(bwd, dev["dY"], saved, dev["W"], dev["A"], dev["B"], dX, None, None, workspace=ws)
        assert e.value.code == rl.RL_ERR_UNSUPPORTED


def test_int4_exact_with_unit_scales():
    """scales = 1 and small integer inputs: every product is an exact integer, so the GPU must
    return the oracle's values bit for bit (the integer GEMM check of the quantised path)."""
    rng = np.random.default_rng(4)
    n, i, o, r = 96, 136, 72, 8
    L = synth.Layer("int4ints", n, i, o, r, "bf16", 0)
    q = rng.integers(-7, 8, size=(i, o)).astype(np.int8)
    scale = np.ones(((i + 63) // 64, o), dtype=np.float16)
    host = {"X": (rng.random((n, i)) < 0.1) * rng.integers(-1, 2, size=(n, i)),
            "A": (rng.random((i, r)) < 0.1).astype(np.int64), "B": rng.integers(-1, 2, size=(r, o)),
            "dY": (rng.random((n, o)) < 0.08) * rng.integers(-1, 2, size=(n, o))}
    host = {k: v.astype(np.float64) for k, v in host.items()}
    dev = {k: to_device(synth.store(v, "bf16"), "bf16") for k, v in host.items()}
    dev["W"] = rl.Int4Weight.from_host(q, scale)
    host["W"] = oracle.dequant_int4(q, scale.astype(np.float64))
    want = reference(host)
    for v in want.values():
        assert np.abs(v).max() <= 256
    for f, b in [(0, 0), (1, 1), (1, 3)]:
        got = run_pair(L, dev, f, b)
        for k in ("Y", "dX", "dA", "dB"):
            assert np.array_equal(got[k], want[k]), (f, b, k)


def test_int4_config_shape_sampled_rows():
    """The quantised configuration at its full size (n 4096, 5120 -> 13824, r 64, bf16): Y and dX on
    sampled token rows (rows are independent), dA and dB in full."""
    L = synth.config_qlora()[0]
    dev, host = make_layer(L)
    rows = np.unique(np.concatenate([np.arange(0, L.n, 256), np.arange(255, L.n, 256),
                                     np.random.default_rng(5).integers(0, L.n, 32)]))
    got = run_pair(L, dev, 1, 1)
    Yr, dXr = oracle.reference_rows(host["X"][rows], host["dY"][rows], host["W"], host["A"], host["B"])
    assert relerr(got["Y"][rows], Yr) < TOL["bf16"]
    assert relerr(got["dX"][rows], dXr) < TOL["bf16"]
    Z1 = oracle.matmul(host["dY"], host["B"], tb=True)
    assert relerr(got["dA"], oracle.matmul(host["X"], Z1, ta=True)) < TOL["bf16"]
    Tm = oracle.matmul(host["X"], host["A"])
    assert relerr(got["dB"], oracle.matmul(Tm, host["dY"], ta=True)) < TOL["bf16"]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_int4_matrix_core_route_ragged(dtype):
    """Panels of W on the dense kernels (the workspace is the one runlora_workspace_bytes_w names; the same layer on the
    matrix-core kernel's int4 route: test_int4_direct_route_with_real_scales), ragged in every direction: n not a multiple of the tile, d_in = 32*64 + 8 (a partial last K tile and a
    partial last scale group for X W), d_out = 32*112 + 8 (the same for dY W^T), r = 24 (a partial K
    tile in the dense second segment).  Y and dX on sampled rows (first and last row of every tile
    row, plus random ones), dA and dB in full; also the default chain, whose dX GEMM has no second
    segment."""
    L = synth.Layer("int4mc", 3001, 2056, 3592, 24, dtype, 12)
    dev, host = make_layer(L)
    rows = np.unique(np.concatenate([np.arange(0, L.n, 256), np.arange(255, L.n, 256), [L.n - 1],
                                     np.random.default_rng(6).integers(0, L.n, 24)]))
    Yr, dXr = oracle.reference_rows(host["X"][rows], host["dY"][rows], host["W"], host["A"], host["B"])
    dA = oracle.matmul(host["X"], oracle.matmul(host["dY"], host["B"], tb=True), ta=True)
    dB = oracle.matmul(oracle.matmul(host["X"], host["A"]), host["dY"], ta=True)
    for f, b in [(1, 1), (0, 0)]:
        print(f"case int4 matrix-core dtype={dtype} fwd={f} bwd={b}", flush=True)
        got = run_pair(L, dev, f, b)
        assert not np.isnan(got["Y"]).any() and not np.isnan(got["dX"]).any()
        assert relerr(got["Y"][rows], Yr) < TOL[dtype], (f, b)
        assert relerr(got["dX"][rows], dXr) < TOL[dtype], (f, b)
        assert relerr(got["dA"], dA) < TOL[dtype] and relerr(got["dB"], dB) < TOL[dtype]


def test_int4_matrix_core_route_with_scale_and_bias():
    """The panels' epilogue and the dense second segment with a LoRA scale and a bias."""
    import torch
    L = synth.Layer("int4mcs", 3001, 2056, 3592, 24, "bf16", 13)
    dev, host = make_layer(L)
    bst = synth.store(synth.normal(synth.BASE_SEED, 98, (L.o,)), L.dtype)
    bias_dev, bias64 = to_device(bst, L.dtype), synth.widen(bst, L.dtype)
    scale = 0.5
    rows = np.unique(np.concatenate([np.arange(0, L.n, 256), [L.n - 1], np.random.default_rng(7).integers(0, L.n, 24)]))
    Yr, dXr = oracle.scaled_rows(host["X"][rows], host["dY"][rows], host["W"], host["A"], host["B"], scale, bias64)
    code = rl.dtype_from_name(L.dtype)
    Y = torch.full((L.n, L.o), float("nan"), dtype=torch.bfloat16, device="cuda")
    gX = torch.full((L.n, L.i), float("nan"), dtype=torch.bfloat16, device="cuda")
    gA = torch.full((L.i, L.r), float("nan"), dtype=torch.bfloat16, device="cuda")
    gB = torch.full((L.r, L.o), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = rl.new_workspace(1, 1, L.n, L.i, L.o, L.r, code, w_dtype=rl.RL_INT4_G64)
    saved = rl.new_saved()
    rl.runlora_forward(1, dev["X"], dev["W"], dev["A"], dev["B"], Y, saved, workspace=ws, scale=scale, bias=bias_dev)
    rl.runlora_backward(1, dev["dY"], saved, dev["W"], dev["A"], dev["B"], gX, gA, gB, workspace=ws)
    torch.cuda.synchronize()
    assert relerr(to_f64(Y)[rows], Yr) < TOL["bf16"] and relerr(to_f64(gX)[rows], dXr) < TOL["bf16"]
    Z1 = scale * oracle.matmul(host["dY"], host["B"], tb=True)
    assert relerr(to_f64(gA), oracle.matmul(host["X"], Z1, ta=True)) < TOL["bf16"]
    Tm = scale * oracle.matmul(host["X"], host["A"])
    assert relerr(to_f64(gB), oracle.matmul(Tm, host["dY"], ta=True)) < TOL["bf16"]


# the tile ids (rl_step_time_t.tile_cfg) of X W and dY W^T: 6 = matrix-core kernel and 1 = generic engine, each dequantising W on
# its way to LDS; panels run on the dense kernels (7, 12-16)
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("n,i,o,r,cfg_y,cfg_dx", [(3001, 3592, 3592, 24, 6, 6),   # ragged in every direction, partial last scale group
                                                  (333, 264, 328, 24, 1, 1),      # generic engine
                                                  (65, 200, 40, 8, 1, 1)])        # one tile, most of it outside
def test_int4_direct_route_with_real_scales(n, i, o, r, cfg_y, cfg_dx, dtype):
    """The kernels that dequantise on their way to LDS, forced by a workspace of only their need (with the one
    runlora_workspace_bytes_w names, all of these shapes multiply dequantised panels): scales that differ per group and column,
    LoRA scale and bias, Y and dX on sampled rows, dA and dB in full.  (Shapes whose direct plan splits its contraction or cuts
    columns off take more scratch that way than in panels: no workspace forces it.)"""
    import torch
    L = synth.Layer("int4direct", n, i, o, r, dtype, 14)
    dev, host = make_layer(L)
    td = torch_dtype(dtype)
    bst = synth.store(synth.normal(synth.BASE_SEED, 99, (o,)), dtype)
    rows = np.unique(np.concatenate([np.arange(0, n, 256), np.arange(255, n, 256), [n - 1], np.random.default_rng(8).integers(0, n, 24)]))
    Yr, dXr = oracle.scaled_rows(host["X"][rows], host["dY"][rows], host["W"], host["A"], host["B"], 0.5, synth.widen(bst, dtype))
    Z1, Tm = 0.5 * oracle.matmul(host["dY"], host["B"], tb=True), 0.5 * oracle.matmul(host["X"], host["A"])
    dAw, dBw = oracle.matmul(host["X"], Z1, ta=True), oracle.matmul(Tm, host["dY"], ta=True)
    full = rl.new_workspace(1, 1, n, i, o, r, rl.dtype_from_name(dtype), w_dtype=rl.RL_INT4_G64)
    for ws_f, ws_b, direct in ((direct_workspace(dev, L, 1), direct_workspace(dev, L, 1, 1), True), (full, full, False)):
        print(f"case int4 {n} {i}->{o} r={r} {dtype} {'direct' if direct else 'panels'}", flush=True)
        Y, gX = (torch.full(s, float("nan"), dtype=td, device="cuda") for s in ((n, o), (n, i)))
        gA, gB = (torch.full(s, float("nan"), dtype=td, device="cuda") for s in ((i, r), (r, o)))
        saved = rl.new_saved()
        rl.runlora_profile_enable(32)
        rl.runlora_forward(1, dev["X"], dev["W"], dev["A"], dev["B"], Y, saved, workspace=ws_f, scale=0.5, bias=to_device(bst, dtype))
        rl.runlora_backward(1, dev["dY"], saved, dev["W"], dev["A"], dev["B"], gX, gA, gB, workspace=ws_b)
        torch.cuda.synchronize()
        cfg = {s["what"].split(" ")[0]: s["tile_cfg"] for s in rl.runlora_profile_collect(32) if "W" in s["what"]}
        rl.runlora_profile_disable()
        if direct:
            assert cfg == {"Y": cfg_y, "dX": cfg_dx}
        else:
            assert all(c == 7 or 12 <= c <= 16 for c in cfg.values()), cfg
        assert relerr(to_f64(Y)[rows], Yr) < TOL[dtype] and relerr(to_f64(gX)[rows], dXr) < TOL[dtype]
        assert relerr(to_f64(gA), dAw) < TOL[dtype] and relerr(to_f64(gB), dBw) < TOL[dtype]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("n,i,o,r", [(300, 1096, 1000, 16),    # one panel, rows and columns that end inside a scale group / a tile
                                     (1237, 4104, 9000, 24),   # two panels of columns forward, ragged last one
                                     (1100, 9000, 4104, 72)])  # two panels of rows backward
def test_int4_panels_and_direct_route_agree(n, i, o, r, dtype):
    """A call with the workspace that runlora_workspace_bytes_w names multiplies dequantised panels of W; one with only what
    the direct route needs (the figure in the error text) still runs, on the kernels that dequantise on their way to LDS.
    Scales of 1 and 2 that differ per group and column, integer values: both give the same bits, every option included."""
    import re

    import torch
    rng = np.random.default_rng(n)
    td = torch_dtype(dtype)
    pick = lambda shape, p: to_device(synth.store((rng.random(shape) < p) * rng.choice([-1.0, 1.0], size=shape), dtype), dtype)
    q = (rng.integers(-4, 5, size=(i, o)) * (rng.random((i, o)) < 0.05)).astype(np.int8)
    scales = rng.integers(1, 3, size=((i + 63) // 64, o)).astype(np.float16)
    W = rl.Int4Weight.from_host(q, scales)
    X, A, B, dY = pick((n, i), 0.05), pick((i, r), 0.01), pick((r, o), 0.05), pick((n, o), 0.05)
    bias = pick((o,), 0.5)
    code = rl.dtype_from_name(dtype)
    print(f"case {n} {i}->{o} r={r} {dtype}", flush=True)

    def run(ws_f, ws_b):
        Y, dX = torch.empty((n, o), dtype=td, device="cuda"), torch.empty((n, i), dtype=td, device="cuda")
        saved = rl.new_saved()
        rl.runlora_profile_enable(32)
        rl.runlora_forward(1, X, W, A, B, Y, saved, workspace=ws_f, scale=2.0, bias=bias)
        rl.runlora_backward(1, dY, saved, W, A, B, dX, None, None, workspace=ws_b)
        torch.cuda.synchronize()
        steps = [(s["what"], s["tile_cfg"]) for s in rl.runlora_profile_collect(32)]
        rl.runlora_profile_disable()
        return Y, dX, steps

    def direct_need(fwd, bwd):
        tiny = torch.empty(256, dtype=torch.uint8, device="cuda")
        with pytest.raises(rl.RunLoRAError) as e:
            if bwd < 0:
                rl.runlora_forward(fwd, X, W, A, B, torch.empty((n, o), dtype=td, device="cuda"), rl.new_saved(), workspace=tiny)
            else:
                s = rl.new_saved()
                rl.runlora_forward(1, X, W, A, B, torch.empty((n, o), dtype=td, device="cuda"), s, workspace=full)
                rl.runlora_backward(bwd, dY, s, W, A, B, torch.empty((n, i), dtype=td, device="cuda"), None, None, workspace=tiny)
        assert e.value.code == rl.RL_ERR_WORKSPACE
        return torch.empty(int(re.search(r"(\d+) bytes", str(e.value)).group(1)), dtype=torch.uint8, device="cuda")

    full = rl.new_workspace(1, 1, n, i, o, r, code, w_dtype=rl.RL_INT4_G64)
    small_f, small_b = direct_need(1, -1), direct_need(1, 1)
    Y0, dX0, direct = run(small_f, small_b)
    Y1, dX1, panels = run(full, full)
    if n > 1000:  # (the short layers' direct route splits its contraction and takes more scratch than their panels)
        assert small_f.numel() < full.numel() and small_b.numel() < full.numel()
        assert direct != panels, "both calls took the same route"
    Wq = q.astype(np.float64) * np.repeat(scales.astype(np.float64), 64, axis=0)[:i]
    want = to_f64(X) @ Wq + 2.0 * (to_f64(X) @ to_f64(A)) @ to_f64(B) + to_f64(bias)
    want_dX = to_f64(dY) @ Wq.T + 2.0 * (to_f64(dY) @ to_f64(B).T) @ to_f64(A).T
    assert np.abs(want).max() <= 256 and np.abs(want_dX).max() <= 256   # integers bf16 holds
    for Y, dX in ((Y0, dX0), (Y1, dX1)):
        assert np.array_equal(to_f64(Y), want) and np.array_equal(to_f64(dX), want_dX)
