"""The torch.autograd front end (module.py) on the GPU: a RunLoRALinear's outputs and gradients against
the fp64 oracle of the scaled layer, gradient flow through a stack of layers, the memory kept between
forward and backward (Section 2: RunLoRA's forwards do not keep XA), and the nn.Linear replacement."""
import json

import numpy as np
import pytest

import oracle
from helpers import TOL, relerr, to_device, to_f64, torch_dtype
from paper_2312_03415_amd import binding as rl
from paper_2312_03415_amd import synth

pytestmark = pytest.mark.gpu


def make_layer(d_in, d_out, r, dtype, alpha, with_bias, pair=None, keep_merged=False, seed=41, keep_t=False):
    from paper_2312_03415_amd.module import RunLoRALinear
    import torch
    st = {"W": synth.store(synth.normal(seed, 2, (d_in, d_out), 1.0 / d_in), dtype),
          "A": synth.store(synth.normal(seed, 3, (d_in, r), 1.0 / d_in), dtype),
          "B": synth.store(synth.normal(seed, 4, (r, d_out), 0.1 / r), dtype),
          "bias": synth.store(synth.normal(seed, 9, (d_out,)), dtype)}
    host = {k: synth.widen(v, dtype) for k, v in st.items()}
    layer = RunLoRALinear(to_device(st["W"], dtype), r, alpha, to_device(st["bias"], dtype) if with_bias else None,
                          pair=pair, keep_merged=keep_merged, keep_t=keep_t)
    with torch.no_grad():
        layer.lora_A.copy_(to_device(st["A"], dtype))
        layer.lora_B.copy_(to_device(st["B"], dtype))
    if not with_bias:
        host["bias"] = None
    return layer, host


@pytest.mark.parametrize("dtype,pair", [("bf16", None), ("bf16", (0, 0)), ("f16", (2, 5)), ("f32", (1, 3)), ("bf16", (2, 4)), ("bf16", (1, 1)),
                                        ("f16", (3, 5))])
def test_layer_matches_oracle(dtype, pair):
    import torch
    b, s, d_in, d_out, r, alpha = 3, 50, 264, 136, 8, 20.0
    layer, host = make_layer(d_in, d_out, r, dtype, alpha, True, pair, keep_merged=pair in ((2, 5), (2, 4)), keep_t=pair in ((1, 1), (3, 5)))
    xs = synth.store(synth.normal(42, 1, (b * s, d_in)), dtype)
    gs = synth.store(synth.normal(42, 5, (b * s, d_out)), dtype)
    x = to_device(xs, dtype).view(b, s, d_in).requires_grad_(True)
    y = layer(x)
    assert y.shape == (b, s, d_out)
    y.backward(to_device(gs, dtype).view(b, s, d_out))
    torch.cuda.synchronize()
    X, G = synth.widen(xs, dtype), synth.widen(gs, dtype)
    scale = alpha / r
    Yw = oracle.scaled_forward(X, host["W"], host["A"], host["B"], scale, host["bias"])
    dXw, dAw, dBw = oracle.scaled_backward(X, host["W"], host["A"], host["B"], G, scale)
    tol = TOL[dtype]
    assert relerr(to_f64(y.reshape(-1, d_out)), Yw) < tol
    assert relerr(to_f64(x.grad.reshape(-1, d_in)), dXw) < tol
    assert relerr(to_f64(layer.lora_A.grad), dAw) < tol
    assert relerr(to_f64(layer.lora_B.grad), dBw) < tol
    assert layer.weight.grad is None and layer.bias.grad is None


def test_gradients_flow_through_a_stack():
    """Two layers with a nonlinearity between them: the chain rule through both (x.grad, and the first
    layer's adapter gradients, which need the second layer's dX) against the same stack in fp64 torch."""
    import torch
    n, d, h, r = 96, 72, 136, 8
    l1, h1 = make_layer(d, h, r, "f32", 16.0, True, seed=51)
    l2, h2 = make_layer(h, d, r, "f32", 16.0, False, seed=52)
    xs = synth.store(synth.normal(53, 1, (n, d)), "f32")
    x = to_device(xs, "f32").requires_grad_(True)
    out = l2(torch.tanh(l1(x)))
    out.square().sum().backward()
    torch.cuda.synchronize()

    t64 = lambda a: torch.tensor(a, dtype=torch.float64, requires_grad=True)
    X, A1, B1, A2, B2 = t64(synth.widen(xs, "f32")), t64(h1["A"]), t64(h1["B"]), t64(h2["A"]), t64(h2["B"])
    W1, W2, b1 = torch.tensor(h1["W"]), torch.tensor(h2["W"]), torch.tensor(h1["bias"])
    s = 16.0 / r
    hid = torch.tanh(X @ W1 + b1 + s * (X @ A1) @ B1)
    ref = hid @ W2 + s * (hid @ A2) @ B2
    ref.square().sum().backward()
    for got, want, name in ((x.grad, X.grad, "x"), (l1.lora_A.grad, A1.grad, "A1"), (l1.lora_B.grad, B1.grad, "B1"),
                            (l2.lora_A.grad, A2.grad, "A2"), (l2.lora_B.grad, B2.grad, "B2")):
        assert relerr(to_f64(got), want.numpy()) < 1e-4, name


def test_memory_kept_between_forward_and_backward():
    """What stays allocated after the forward, beyond the output: n*r elements for the default chain's
    XA, nothing for forward1/forward2, i*o elements when forward2 keeps W + AB."""
    import torch
    n, d_in, d_out, r = 4096, 1024, 2048, 64
    code = rl.RL_BF16
    xs = to_device(synth.store(synth.normal(61, 1, (n, d_in)), "bf16"), "bf16").requires_grad_(True)
    held = {}
    for name, pair, keep in (("default", (0, 0), False), ("fwd1", (1, 1), False), ("fwd2", (2, 5), False), ("fwd2+M", (2, 5), True),
                             ("fwd1+T", (1, 1), "t")):
        layer, _ = make_layer(d_in, d_out, r, "bf16", None, False, pair, keep is True, keep_t=keep == "t")
        layer(xs).sum().backward()      # warm: workspace and autograd buffers exist
        layer.zero_grad(); xs.grad = None
        torch.cuda.synchronize()
        before = torch.cuda.memory_allocated()
        y = layer(xs)
        torch.cuda.synchronize()
        held[name] = torch.cuda.memory_allocated() - before - y.numel() * 2
        y.sum().backward()
        del y
    assert held["fwd1"] == 0 and held["fwd2"] == 0
    assert held["default"] == rl.runlora_saved_bytes(0, n, d_in, d_out, r, code) == n * r * 2
    assert held["fwd2+M"] == rl.runlora_saved_bytes(2, n, d_in, d_out, r, code, keep_merged=True) == d_in * d_out * 2
    assert held["fwd1+T"] == rl.runlora_saved_bytes(1, n, d_in, d_out, r, code, keep_t=True) == n * r * 2


def test_wrap_linears_replaces_and_freezes():
    import torch
    from torch import nn
    from paper_2312_03415_amd.module import RunLoRALinear, wrap_linears

    class Block(nn.Module):
        def __init__(self):
            super().__init__()
            self.q_proj = nn.Linear(64, 64, bias=False)
            self.up = nn.Linear(64, 136)
            self.down = nn.Linear(136, 64)
            self.norm = nn.LayerNorm(64)

        def forward(self, x):
            return self.norm(x + self.down(torch.relu(self.up(self.q_proj(x)))))

    torch.manual_seed(0)
    model = Block().cuda()
    x = torch.randn(5, 40, 64, device="cuda")
    want = model(x)
    names = wrap_linears(model, r=8, alpha=16, targets=("q_proj", "down"))
    assert sorted(names) == ["down", "q_proj"]
    assert isinstance(model.q_proj, RunLoRALinear) and isinstance(model.down, RunLoRALinear) and isinstance(model.up, nn.Linear)
    trainable = sorted(n for n, p in model.named_parameters() if p.requires_grad)
    assert trainable == ["down.lora_A", "down.lora_B", "q_proj.lora_A", "q_proj.lora_B"]
    got = model(x)                      # B = 0 at the start: the wrapped model is the original one
    assert relerr(to_f64(got.reshape(-1, 64)), to_f64(want.reshape(-1, 64))) < 1e-5
    got.square().mean().backward()
    assert model.q_proj.lora_B.grad is not None and model.q_proj.lora_B.grad.abs().sum().item() > 0
    assert model.q_proj._pairs and list(model.q_proj._pairs) == [200]


def test_wrap_linears_with_dora_layers():
    """adapter="dora": bf16 linears become RunDoRALinear, the wrapped model starts as the original one (B = 0, m = the
    column norms of W), and A, B and m are what trains."""
    import torch
    from torch import nn
    from paper_2312_03415_amd.module import RunDoRALinear, wrap_linears

    class Mlp(nn.Module):
        def __init__(self):
            super().__init__()
            self.up = nn.Linear(64, 136)
            self.down = nn.Linear(136, 64, bias=False)

        def forward(self, x):
            return self.down(torch.relu(self.up(x)))

    torch.manual_seed(1)
    model = Mlp().cuda().to(torch.bfloat16)
    x = torch.randn(4, 50, 64, device="cuda").to(torch.bfloat16)
    want = model(x)
    names = wrap_linears(model, r=8, alpha=16, adapter="dora")
    assert sorted(names) == ["down", "up"] and isinstance(model.up, RunDoRALinear)
    trainable = sorted(n for n, p in model.named_parameters() if p.requires_grad)
    assert trainable == ["down.dora_m", "down.lora_A", "down.lora_B", "up.dora_m", "up.lora_A", "up.lora_B"]
    got = model(x)
    assert relerr(to_f64(got.reshape(-1, 64)), to_f64(want.reshape(-1, 64))) < 2 * TOL["bf16"]
    got.float().square().mean().backward()
    for layer in (model.up, model.down):
        assert layer.dora_m.grad is not None and layer.dora_m.grad.float().abs().sum().item() > 0
        assert layer.lora_B.grad.float().abs().sum().item() > 0
    with pytest.raises(ValueError):
        wrap_linears(Mlp(), r=8, adapter="dora", dropout=0.1)


def test_layer_dropout_in_training_mode():
    """Training mode with dropout: outputs and gradients match the oracle under the mask of the seed the
    layer drew; eval mode runs without dropout."""
    import torch
    b, s, d_in, d_out, r, alpha, p = 2, 60, 264, 136, 8, 16.0, 0.25
    layer, host = make_layer(d_in, d_out, r, "bf16", alpha, True)
    layer.dropout = p
    xs = synth.store(synth.normal(43, 1, (b * s, d_in)), "bf16")
    gs = synth.store(synth.normal(43, 5, (b * s, d_out)), "bf16")
    X, G = synth.widen(xs, "bf16"), synth.widen(gs, "bf16")
    scale = alpha / r
    layer.eval()
    y_eval = layer(to_device(xs, "bf16").view(b, s, d_in))
    assert relerr(to_f64(y_eval.reshape(-1, d_out)), oracle.scaled_forward(X, host["W"], host["A"], host["B"], scale, host["bias"])) < TOL["bf16"]
    layer.train()
    torch.manual_seed(5)
    x = to_device(xs, "bf16").view(b, s, d_in).requires_grad_(True)
    y = layer(x)
    y.backward(to_device(gs, "bf16").view(b, s, d_out))
    torch.cuda.synchronize()
    mask, pq = oracle.dropout_mask(b * s, d_in, p, layer.last_dropout_seed)
    Yw = oracle.dropout_forward(X, host["W"], host["A"], host["B"], mask, pq, scale, host["bias"])
    dXw, dAw, dBw = oracle.dropout_backward(X, host["W"], host["A"], host["B"], G, mask, pq, scale)
    assert relerr(to_f64(y.reshape(-1, d_out)), Yw) < TOL["bf16"]
    assert relerr(to_f64(x.grad.reshape(-1, d_in)), dXw) < TOL["bf16"]
    assert relerr(to_f64(layer.lora_A.grad), dAw) < TOL["bf16"] and relerr(to_f64(layer.lora_B.grad), dBw) < TOL["bf16"]
    torch.manual_seed(5)
    layer(x.detach())
    first = layer.last_dropout_seed
    layer(x.detach())
    assert layer.last_dropout_seed != first            # a fresh mask per call
    torch.manual_seed(5)
    layer(x.detach())
    assert layer.last_dropout_seed == first            # repeatable under torch.manual_seed


@pytest.mark.parametrize("model", ["opt1.3b", "llama7b"])
def test_block_timing_script_runs_the_same_block_both_ways(model, capsys):
    """The decoder-block timing script: RunLoRA layers and the default chain compute the same block
    output (bf16 rounding apart) and the script reports one time for each."""
    from paper_2312_03415_amd import block_timing
    out = block_timing.main(["--model", model, "--batch", "1", "--seq", "192", "--rank", "8", "--iters", "2", "--warmup", "1"])
    assert set(out["ms_fwd_bwd"]) == {"runlora", "default"} and all(v > 0 for v in out["ms_fwd_bwd"].values())
    assert out["rel_diff_vs_default"] < 2e-2
    assert len(out["pairs"]) == (7 if model == "llama7b" else 6)
    assert json.loads(capsys.readouterr().out.strip().splitlines()[-1])["model"] == model


def test_vera_module_matches_oracle_and_shares_frozen_factors():
    """RunVeRALinear through autograd: output and the gradients of x, d and b against the oracle's VeRA
    layer; A and B are buffers, not parameters, and two layers may hold the same tensors."""
    import torch
    from paper_2312_03415_amd.module import RunVeRALinear
    n, d_in, d_out, r = 150, 136, 264, 64
    L = synth.Layer("veramod", n, d_in, d_out, r, "bf16", 51)
    st = synth.layer_inputs(L)
    host = {k: synth.widen(v, "bf16") for k, v in st.items()}
    dvec = synth.store(synth.normal(51, 10, (r,)), "bf16")
    bvec = synth.store(synth.normal(51, 11, (d_out,)), "bf16")
    A, B = to_device(st["A"], "bf16"), to_device(st["B"], "bf16")
    layer = RunVeRALinear(to_device(st["W"], "bf16"), A, B, scale=0.5)
    other = RunVeRALinear(to_device(st["W"], "bf16"), A, B)
    assert other.vera_A.data_ptr() == layer.vera_A.data_ptr()
    assert sorted(k for k, p in layer.named_parameters() if p.requires_grad) == ["vera_b", "vera_d"]
    with torch.no_grad():
        layer.vera_d.copy_(to_device(dvec, "bf16"))
        layer.vera_b.copy_(to_device(bvec, "bf16"))
    x = to_device(st["X"], "bf16").view(3, 50, d_in).requires_grad_(True)
    y = layer(x)
    y.backward(to_device(st["dY"], "bf16").view(3, 50, d_out))
    torch.cuda.synchronize()
    d64, b64 = synth.widen(dvec, "bf16"), synth.widen(bvec, "bf16")
    Yw = oracle.vera_forward(host["X"], host["W"], host["A"], host["B"], d64, b64, 0.5)
    dXw, ddw, dbw = oracle.vera_backward(host["X"], host["W"], host["A"], host["B"], d64, b64, host["dY"], 0.5)
    assert relerr(to_f64(y.reshape(-1, d_out)), Yw) < TOL["bf16"]
    assert relerr(to_f64(x.grad.reshape(-1, d_in)), dXw) < TOL["bf16"]
    assert relerr(to_f64(layer.vera_d.grad), ddw) < TOL["bf16"] and relerr(to_f64(layer.vera_b.grad), dbw) < TOL["bf16"]
    # a fresh layer (b = 0) is the frozen linear layer
    y0 = other(x.detach())
    assert relerr(to_f64(y0.reshape(-1, d_out)), host["X"] @ host["W"]) < TOL["bf16"]


def test_dora_module_matches_oracle_and_starts_as_the_frozen_layer():
    """RunDoRALinear through autograd: output and the gradients of x, A, B and m against the oracle's DoRA layer
    (column norm held constant in the backward pass); a fresh layer (B = 0, m = ||W||) is the frozen linear layer."""
    import torch
    from paper_2312_03415_amd.module import RunDoRALinear
    n, d_in, d_out, r = 150, 136, 264, 16
    L = synth.Layer("doramod", n, d_in, d_out, r, "bf16", 57)
    st = synth.layer_inputs(L)
    host = {k: synth.widen(v, "bf16") for k, v in st.items()}
    mvec = synth.store(0.5 + np.abs(synth.normal(57, 10, (d_out,))), "bf16")
    bias = synth.store(synth.normal(57, 9, (d_out,)), "bf16")
    layer = RunDoRALinear(to_device(st["W"], "bf16"), r, alpha=8.0, bias=to_device(bias, "bf16"))
    assert sorted(k for k, p in layer.named_parameters() if p.requires_grad) == ["dora_m", "lora_A", "lora_B"]
    x = to_device(st["X"], "bf16").view(3, 50, d_in).requires_grad_(True)
    y0 = layer(x.detach())
    torch.cuda.synchronize()
    assert relerr(to_f64(y0.reshape(-1, d_out)), host["X"] @ host["W"] + synth.widen(bias, "bf16")[None, :]) < TOL["bf16"]
    with torch.no_grad():
        layer.lora_A.copy_(to_device(st["A"], "bf16"))
        layer.lora_B.copy_(to_device(st["B"], "bf16"))
        layer.dora_m.copy_(to_device(mvec, "bf16"))
    y = layer(x)
    y.backward(to_device(st["dY"], "bf16").view(3, 50, d_out))
    torch.cuda.synchronize()
    m64, b64 = synth.widen(mvec, "bf16"), synth.widen(bias, "bf16")
    args = (host["X"], host["W"], host["A"], host["B"], m64)
    Yw = oracle.dora_forward(*args, 0.5, b64)
    dXw, dAw, dBw, dmw = oracle.dora_backward(*args, host["dY"], 0.5)
    assert relerr(to_f64(y.reshape(-1, d_out)), Yw) < TOL["bf16"]
    assert relerr(to_f64(x.grad.reshape(-1, d_in)), dXw) < TOL["bf16"]
    assert relerr(to_f64(layer.lora_A.grad), dAw) < TOL["bf16"] and relerr(to_f64(layer.lora_B.grad), dBw) < TOL["bf16"]
    assert relerr(to_f64(layer.dora_m.grad), dmw) < TOL["bf16"]


@pytest.mark.parametrize("native", [True, False])
def test_forward_3_with_T_kept_gets_the_workspace_of_forward_1(native):
    """With T kept, forward 3 runs as forward 1, whose product is split here and needs scratch that forward 3 does not."""
    import torch
    from paper_2312_03415_amd.module import RunLoRAFunction
    layer, host = make_layer(2056, 2120, 16, "bf16", 32, False, (3, 1), keep_t=True)
    x = torch.randn(520, 2056, generator=torch.Generator().manual_seed(4)).to(torch.bfloat16).cuda().requires_grad_()
    assert rl.runlora_call_workspace_bytes(1, -1, 520, 2056, 2120, 16, rl.RL_BF16, keep_t=True) > 256
    if native:
        y = layer(x)
    else:
        y = super(RunLoRAFunction, RunLoRAFunction).apply(x, layer.weight, layer.lora_A, layer.lora_B, layer.bias, layer.scale, (3, 1), False, None, True)
    y.sum().backward()
    torch.cuda.synchronize()
    want = oracle.reference_forward(to_f64(x), to_f64(layer.weight), to_f64(layer.lora_A) * layer.scale, to_f64(layer.lora_B))
    assert relerr(to_f64(y), want) < TOL["bf16"]
    assert all(bool(t.grad.isfinite().all()) for t in (x, layer.lora_A, layer.lora_B))
