"""GPU parity of the DoRA entry points (magnitudes m, direction (W + sAB) / column norm; the paper's conclusion
names DoRA among the adapters its method carries over to): c, Y, dX, dA, dB, dm of every merged-weight graph
against the fp64 oracle of the layer's definition (oracle.dora_norm / dora_forward / dora_backward), the
reduction to the LoRA calls, the kept merged weight, skipped outputs, refusals, and one full-size layer."""
import numpy as np
import pytest

import oracle
from helpers import TOL, layer_on_device, relerr, to_device, to_f64, torch_dtype
from paper_2312_03415_amd import binding as rl
from paper_2312_03415_amd import synth

pytestmark = pytest.mark.gpu

BWDS = (4, 5, 7, 8)


def vectors(L):
    """m: positive magnitudes around the column norms' size (DoRA starts from m = ||W||); bias."""
    out = {}
    m = 0.5 + np.abs(synth.normal(synth.BASE_SEED + L.index, 10, (L.o,)))
    for name, v in (("m", m), ("bias", synth.normal(synth.BASE_SEED + L.index, 9, (L.o,)))):
        st = synth.store(v, L.dtype)
        out[name] = (to_device(st, L.dtype), synth.widen(st, L.dtype))
    return out


def run_dora(L, dev, vec, bwd, scale, bias, want=("dX", "dA", "dB", "dm"), keep=False, m=None):
    import torch
    td = torch_dtype(L.dtype)
    code = rl.dtype_from_name(L.dtype)
    nan = float("nan")
    Y = torch.full((L.n, L.o), nan, dtype=td, device="cuda")
    c = torch.full((L.o,), nan, dtype=torch.float32, device="cuda")
    M = torch.full((L.i, L.o), nan, dtype=td, device="cuda") if keep else None
    saved = rl.new_saved(None, M)
    ws = torch.empty(rl.runlora_dora_workspace_bytes(2, bwd, L.n, L.i, L.o, L.r, code), dtype=torch.uint8, device="cuda")
    m = vec["m"][0] if m is None else m
    rl.runlora_dora_forward(2, dev["X"], dev["W"], dev["A"], dev["B"], m, Y, saved, c, ws, scale=scale, bias=bias)
    ws.fill_(0xFF)  # nothing the forward left in the workspace may matter to the backward
    dX = torch.full((L.n, L.i), nan, dtype=td, device="cuda") if "dX" in want else None
    dA = torch.full((L.i, L.r), nan, dtype=td, device="cuda") if "dA" in want else None
    dB = torch.full((L.r, L.o), nan, dtype=td, device="cuda") if "dB" in want else None
    dm = torch.full((L.o,), nan, dtype=td, device="cuda") if "dm" in want else None
    rl.runlora_dora_backward(bwd, dev["dY"], saved, dev["W"], dev["A"], dev["B"], m, c, Y, dX, dA, dB, dm, ws, bias=bias)
    torch.cuda.synchronize()
    out = {"Y": to_f64(Y), "c": c.double().cpu().numpy()}
    for k, t in (("dX", dX), ("dA", dA), ("dB", dB), ("dm", dm)):
        if t is not None:
            out[k] = to_f64(t)
    if keep:
        out["M"] = to_f64(M)
    return out


def dora_reference(host, vec, scale, with_bias=True):
    m, bias = vec["m"][1], vec["bias"][1]
    args = (host["X"], host["W"], host["A"], host["B"], m)
    Y = oracle.dora_forward(*args, scale, bias if with_bias else None)
    dX, dA, dB, dm = oracle.dora_backward(*args, host["dY"], scale)
    return {"c": oracle.dora_norm(host["W"], host["A"], host["B"], scale), "Y": Y, "dX": dX, "dA": dA, "dB": dB, "dm": dm}


@pytest.mark.parametrize("dtype,r", [("bf16", 24), ("f16", 64), ("bf16", 128), ("f16", 8)])
def test_dora_all_graphs(dtype, r):
    """Ragged shape (several column strips and row slices of the norm pass, partial tiles everywhere), forward2
    with each of backward 4 / 5 / 7 / 8, s = 0.5, a bias.  c is an fp32 sum of unrounded terms: 1e-5."""
    L = synth.Layer("dora", 301, 264, 1096, r, dtype, 51)
    dev, host = layer_on_device(L)
    vec = vectors(L)
    want = dora_reference(host, vec, 0.5)
    for b in BWDS:
        print(f"case dora layer={L} bwd={b}", flush=True)
        got = run_dora(L, dev, vec, b, 0.5, vec["bias"][0])
        assert relerr(got["c"], want["c"]) < 1e-5, (b, relerr(got["c"], want["c"]))
        for k in ("Y", "dX", "dA", "dB", "dm"):
            err = relerr(got[k], want[k])
            assert err < TOL[dtype], (b, k, err)


def test_dora_kept_merged_weight_and_skipped_outputs():
    """Keeping (W + sAB) diag(g) between forward and backward changes no bit of any output; it is the oracle's
    adapted weight, whose columns have length m; skipped outputs leave the others unchanged."""
    L = synth.Layer("dora2", 200, 136, 264, 16, "bf16", 52)
    dev, host = layer_on_device(L)
    vec = vectors(L)
    full = run_dora(L, dev, vec, 5, 0.7, vec["bias"][0])
    kept = run_dora(L, dev, vec, 5, 0.7, vec["bias"][0], keep=True)
    for k in full:
        assert np.array_equal(full[k], kept[k]), k
    V = host["W"] + 0.7 * host["A"] @ host["B"]
    cn = np.sqrt((V * V).sum(axis=0))
    assert relerr(kept["M"], V * (vec["m"][1] / cn)[None, :]) < TOL["bf16"]
    assert relerr(np.sqrt((kept["M"] ** 2).sum(axis=0)), vec["m"][1]) < TOL["bf16"]
    for want in (("dm",), ("dB",), ("dX",), ("dA", "dm"), ()):
        part = run_dora(L, dev, vec, 5, 0.7, vec["bias"][0], want=want)
        assert set(part) == {"Y", "c", *want}
        for k in part:
            assert np.array_equal(part[k], full[k]), (want, k)


def test_dora_with_unit_gain_is_the_lora_layer():
    """m = c rounded to the storage type makes g = 1 up to that rounding (5e-4 in f16): Y, dX, dA and dB are
    then what the LoRA calls of the same graphs give, to tolerance."""
    import torch
    L = synth.Layer("dora3", 160, 136, 264, 16, "f16", 53)
    dev, host = layer_on_device(L)
    vec = vectors(L)
    c = oracle.dora_norm(host["W"], host["A"], host["B"], 1.0)
    st = synth.store(c, L.dtype)
    m_dev, m_host = to_device(st, L.dtype), synth.widen(st, L.dtype)
    got = run_dora(L, dev, vec, 4, None, None, m=m_dev)
    code = rl.dtype_from_name(L.dtype)
    Y = torch.empty((L.n, L.o), dtype=torch.float16, device="cuda")
    saved = rl.new_saved(None)
    ws = rl.new_workspace(2, 4, L.n, L.i, L.o, L.r, code)
    rl.runlora_forward(2, dev["X"], dev["W"], dev["A"], dev["B"], Y, saved, workspace=ws)
    dX = torch.empty((L.n, L.i), dtype=torch.float16, device="cuda")
    dA = torch.empty((L.i, L.r), dtype=torch.float16, device="cuda")
    dB = torch.empty((L.r, L.o), dtype=torch.float16, device="cuda")
    rl.runlora_backward(4, dev["dY"], saved, dev["W"], dev["A"], dev["B"], dX, dA, dB, workspace=ws)
    torch.cuda.synchronize()
    assert np.max(np.abs(m_host / c - 1.0)) < 1e-3
    for k, t in (("Y", Y), ("dX", dX), ("dA", dA), ("dB", dB)):
        assert relerr(got[k], to_f64(t)) < TOL["f16"], k


def test_dora_refusals():
    """Graphs that read W outside W + sAB, fp32, r > 128 and dropout are refused with the documented codes before
    anything is launched (outputs keep their fill)."""
    import torch
    L = synth.Layer("dora4", 64, 64, 128, 8, "bf16", 54)
    dev, host = layer_on_device(L)
    vec = vectors(L)
    code = rl.dtype_from_name(L.dtype)
    Y = torch.full((L.n, L.o), 7.0, dtype=torch.bfloat16, device="cuda")
    c = torch.zeros((L.o,), dtype=torch.float32, device="cuda")
    ws = torch.empty(rl.runlora_dora_workspace_bytes(2, 5, L.n, L.i, L.o, L.r, code) + 4096, dtype=torch.uint8, device="cuda")
    saved = rl.new_saved(torch.empty((L.n, L.r), dtype=torch.bfloat16, device="cuda"))
    for fwd in (0, 1, 3):
        with pytest.raises(rl.RunLoRAError) as e:
            rl.runlora_dora_forward(fwd, dev["X"], dev["W"], dev["A"], dev["B"], vec["m"][0], Y, saved, c, ws)
        assert e.value.code == rl.RL_ERR_UNSUPPORTED
    with pytest.raises(rl.RunLoRAError) as e:
        rl.runlora_dora_forward(4, dev["X"], dev["W"], dev["A"], dev["B"], vec["m"][0], Y, saved, c, ws)
    assert e.value.code == rl.RL_ERR_VARIANT
    saved = rl.new_saved(None)
    rl.runlora_dora_forward(2, dev["X"], dev["W"], dev["A"], dev["B"], vec["m"][0], Y, saved, c, ws)
    dX = torch.full((L.n, L.i), 7.0, dtype=torch.bfloat16, device="cuda")
    for bwd in (0, 1, 2, 3, 6):
        with pytest.raises(rl.RunLoRAError) as e:
            rl.runlora_dora_backward(bwd, dev["dY"], saved, dev["W"], dev["A"], dev["B"], vec["m"][0], c, Y, dX, None, None, None, ws)
        assert e.value.code == rl.RL_ERR_UNSUPPORTED
    torch.cuda.synchronize()
    assert bool((dX == 7.0).all())
    # dm without the forward's output
    dm = torch.zeros((L.o,), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(rl.RunLoRAError) as e:
        rl.runlora_dora_backward(5, dev["dY"], saved, dev["W"], dev["A"], dev["B"], vec["m"][0], c, None, dX, None, None, dm, ws)
    assert e.value.code == rl.RL_ERR_NULL
    assert rl.runlora_dora_workspace_bytes(2, 5, 64, 64, 128, 8, rl.dtype_from_name("f32")) == 0
    assert rl.runlora_dora_workspace_bytes(2, 5, 64, 64, 128, 136, code) == 0


def test_dora_full_size_opt_fc1():
    """OPT-1.3B fc1 shape (n 4096, 2048 -> 8192, bf16, r 16), forward2 + backward5: c, dm, dA, dB in full (they need
    every token), Y and dX on sampled token rows."""
    L = synth.Layer("dora_fc1", 4096, 2048, 8192, 16, "bf16", 55)
    dev, host = layer_on_device(L)
    vec = vectors(L)
    m, bias = vec["m"][1], vec["bias"][1]
    s = 2.0
    got = run_dora(L, dev, vec, 5, s, vec["bias"][0])
    V = host["W"] + s * oracle.matmul(host["A"], host["B"])
    c = np.sqrt((V * V).sum(axis=0))
    assert relerr(got["c"], c) < 1e-5
    g = m / c
    dU = host["dY"] * g[None, :]
    T = oracle.matmul(host["X"], host["A"])
    dB = s * oracle.matmul(T, dU, ta=True)
    dA = s * oracle.matmul(host["X"], oracle.matmul(dU, host["B"], tb=True), ta=True)
    # dm[j] = sum_t dY[t,j] (XV)[t,j] / c[j] = sum_i (X^T dY)[i,j] V[i,j] / c[j]
    dm = (oracle.matmul(host["X"], host["dY"], ta=True) * V).sum(axis=0) / c
    assert relerr(got["dB"], dB) < TOL["bf16"] and relerr(got["dA"], dA) < TOL["bf16"]
    assert relerr(got["dm"], dm) < TOL["bf16"], relerr(got["dm"], dm)
    rng = np.random.default_rng(6)
    rows = np.unique(np.concatenate([np.arange(0, L.n, 512), np.arange(255, L.n, 512), rng.integers(0, L.n, 24)]))
    Yr = oracle.dora_forward(host["X"][rows], host["W"], host["A"], host["B"], m, s, bias)
    dXr = oracle.matmul(dU[rows], V, tb=True)
    assert relerr(got["Y"][rows], Yr) < TOL["bf16"] and relerr(got["dX"][rows], dXr) < TOL["bf16"]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("n,i,o,r,scaled", [(4104, 520, 2568, 16, True),   # 256x256 tiles, ragged
                                            (8192, 264, 4360, 8, True),    # 256x256 with a column of tiles cut off
                                            (1240, 1096, 5464, 24, True), (520, 264, 1000, 128, True), (70, 136, 264, 8, True),
                                            (300, 4104, 264, 16, False),   # contraction split: M is formed as before
                                            (24, 264, 520, 8, False)])     # few rows: the generic engine
def test_dora_forward_with_scaled_columns(n, i, o, r, scaled, dtype):
    """Y = X V diag(g) on every kernel that scales its product's columns, and the route without one, against the oracle."""
    import torch
    L = synth.Layer("doracs", n, i, o, r, dtype, 55)
    dev, host = layer_on_device(L)
    vec = vectors(L)
    print(f"case {n} {i}->{o} r={r} {dtype}", flush=True)
    rows = np.unique(np.concatenate([np.arange(0, n, 253), [n - 1]]))
    V = host["W"] + 0.5 * host["A"] @ host["B"]
    c = np.sqrt((V * V).sum(axis=0))
    want = host["X"][rows] @ V * (vec["m"][1] / c)[None, :] + vec["bias"][1][None, :]
    buf = torch.full((n + 2, o + 16), 7.0, dtype=torch_dtype(dtype), device="cuda")
    Y = buf[1:n + 1, 8:o + 8]
    cd = torch.empty((o,), dtype=torch.float32, device="cuda")
    ws = torch.full((rl.runlora_dora_workspace_bytes(2, -1, n, i, o, r, rl.dtype_from_name(dtype)),), 0xFF, dtype=torch.uint8, device="cuda")
    rl.runlora_profile_enable(8)
    rl.runlora_dora_forward(2, dev["X"], dev["W"], dev["A"], dev["B"], vec["m"][0], Y, rl.new_saved(), cd, ws, scale=0.5, bias=vec["bias"][0])
    torch.cuda.synchronize()
    steps = [s["what"] for s in rl.runlora_profile_collect(8)]
    rl.runlora_profile_disable()
    assert ("Y = X V diag(g)" in steps) == (scaled and dtype == "bf16"), steps
    assert relerr(to_f64(cd), c) < 1e-5 and relerr(to_f64(Y)[rows], want) < TOL[dtype]
    edge = buf.float()
    edge[1:n + 1, 8:o + 8] = 7.0
    assert bool((edge == 7.0).all())


def test_dora_f16_weight_sum_beyond_the_type():
    """W + s A B may leave the range of f16 (70000 here) where its scaled columns do not: nothing is rounded in between."""
    import torch
    n, i, o, r = 520, 264, 1000, 8
    g = torch.Generator().manual_seed(3)
    X = torch.randn(n, i, generator=g).to(torch.float16)
    full = lambda a, b, v: torch.full((a, b), v, dtype=torch.float16, device="cuda")
    W, A, B, m = full(i, o, 60000.0), full(i, r, 50.0), full(r, o, 50.0), full(1, o, 30.0)[0]
    Y, cd = full(n, o, 0.0), torch.empty((o,), dtype=torch.float32, device="cuda")
    ws = torch.empty((rl.runlora_dora_workspace_bytes(2, -1, n, i, o, r, rl.RL_F16),), dtype=torch.uint8, device="cuda")
    rl.runlora_dora_forward(2, X.cuda(), W, A, B, m, Y, rl.new_saved(), cd, ws, scale=0.5)
    torch.cuda.synchronize()
    want = np.repeat(X.double().numpy().sum(axis=1, keepdims=True) * (30.0 / np.sqrt(i)), o, axis=1)  # c = 70000 sqrt(i) in every column
    assert relerr(to_f64(cd), np.full((o,), 70000.0 * np.sqrt(i))) < 1e-5
    assert relerr(to_f64(Y), want) < TOL["f16"]


@pytest.mark.parametrize("n,i,o,r,v", [(4104, 520, 2568, 16, False), (512, 256, 264, 16, False), (512, 256, 256, 24, False), (512, 256, 256, 16, True), (70, 136, 264, 8, True)])
def test_dora_forward_that_keeps_its_merged_weight(n, i, o, r, v):
    """A kept (W + s A B) diag(g) is what the product multiplies by; only where W is small and r low is V formed besides."""
    import torch
    L = synth.Layer("dorakeep", n, i, o, r, "bf16", 56)
    dev, host = layer_on_device(L)
    vec = vectors(L)
    print(f"case {n} {i}->{o} r={r}", flush=True)
    Y, M = (torch.full(s, float("nan"), dtype=torch.bfloat16, device="cuda") for s in ((n, o), (i, o)))
    cd = torch.empty((o,), dtype=torch.float32, device="cuda")
    ws = torch.full((rl.runlora_dora_workspace_bytes(2, -1, n, i, o, r, rl.RL_BF16),), 0xFF, dtype=torch.uint8, device="cuda")
    rl.runlora_profile_enable(8)
    rl.runlora_dora_forward(2, dev["X"], dev["W"], dev["A"], dev["B"], vec["m"][0], Y, rl.new_saved(None, M), cd, ws, scale=0.5, bias=vec["bias"][0])
    torch.cuda.synchronize()
    steps = [s["what"] for s in rl.runlora_profile_collect(8)]
    rl.runlora_profile_disable()
    assert steps == (["V = W + A B", "Y = X V diag(g)", "M = V diag(g)"] if v else ["M = W + A B", "Y = X M"])
    V = host["W"] + 0.5 * host["A"] @ host["B"]
    want = V * (vec["m"][1] / np.sqrt((V * V).sum(axis=0)))[None, :]
    assert relerr(to_f64(M), want) < TOL["bf16"]
    assert relerr(to_f64(Y), host["X"] @ want + vec["bias"][1][None, :]) < TOL["bf16"]
    if not v:
        Y2 = torch.empty_like(Y)
        rl.runlora_gemm(dev["X"], M, Y2, bias=vec["bias"][0])
        torch.cuda.synchronize()
        assert torch.equal(Y, Y2)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_dora_dB_does_not_depend_on_whether_dm_is_wanted(dtype):
    """dB = dB~ diag(g) is formed by the launch that finishes dm, or by one of its own: half a million elements, the same bits."""
    L = synth.Layer("doradb", 72, 64, 4096, 128, dtype, 57)
    dev, _ = layer_on_device(L)
    vec = vectors(L)
    both, alone = (run_dora(L, dev, vec, 5, 0.7, None, want=w) for w in (("dB", "dm"), ("dB",)))
    assert np.array_equal(both["dB"], alone["dB"])


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("i,o,r", [(2048, 8192, 16), (1000, 264, 32), (4096, 2056, 64), (4104, 1288, 48), (16456, 136, 8), (5000, 1544, 72), (2056, 4104, 128)])
def test_column_norms_add_their_squares_in_a_fixed_order(i, o, r, dtype):
    """c bit for bit: the rows of a column in slices (as many as make 512 workgroups of 512 columns, of 256 beyond r = 64), in a slice
    four chains of every fourth row (eight beyond r = 64), chains and slices one behind the other.  With A = 0 the squares are exact, so
    fp32 additions in that order are all there is; W's values span 2^12, so that another order gives other bits."""
    import torch
    td, code = torch_dtype(dtype), rl.dtype_from_name(dtype)
    print(f"case norms {i}x{o} r{r} {dtype}", flush=True)
    g = torch.Generator().manual_seed(i + o + r)
    W = (torch.randn(i, o, generator=g) * torch.exp2(8 * torch.rand(i, o, generator=g) - 6)).to(td)
    chains, strip = (4, 512) if r <= 64 else (8, 256)
    nb = -(-i // 32)
    blocks = -(-nb // max(1, min(nb, 512 // -(-o // strip))))
    slices = -(-nb // blocks)
    v = np.zeros((slices * blocks * 32, o), np.float32)
    v[:i] = W.float().numpy()
    v = (v * v).reshape(slices, blocks * 32 // chains, chains, o)

    def added(terms):
        t = np.zeros_like(terms[0])
        for k in range(len(terms)):
            t = t + terms[k]
        return t
    part = added(added(v.transpose(1, 0, 2, 3)).transpose(1, 0, 2))                    # [slices, o]
    want = np.sqrt(added([added(part[q::4]) if q < slices else np.zeros(o, np.float32) for q in range(4)]))
    dev = {k: t.to(td).cuda() for k, t in (("X", torch.ones(8, i)), ("A", torch.zeros(i, r)), ("B", torch.randn(r, o, generator=g)), ("m", torch.ones(o)))}
    ws = torch.empty(rl.runlora_dora_workspace_bytes(2, -1, 8, i, o, r, code), dtype=torch.uint8, device="cuda")
    for keep in (False, True):
        ws.fill_(0xFF)
        Y, c = torch.empty(8, o, dtype=td, device="cuda"), torch.full((o,), float("nan"), device="cuda")
        M = torch.empty(i, o, dtype=td, device="cuda") if keep else None
        rl.runlora_dora_forward(2, dev["X"], W.cuda(), dev["A"], dev["B"], dev["m"], Y, rl.new_saved(None, M), c, ws)
        assert np.array_equal(c.cpu().numpy(), want), (keep, int((c.cpu().numpy() != want).sum()))
