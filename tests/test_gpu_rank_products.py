"""GPU: rank-r products with r > 32 (paired launches of the middle-sized kernel where the rule takes them, the streaming
kernel elsewhere) at tile edges, with and without scratch to split into, padded operand rows, single gradients: against
Eq. 3 in fp64."""
import numpy as np
import pytest

import oracle
from helpers import TOL, relerr, to_device, to_f64, torch_dtype
from paper_2312_03415_amd import binding as rl
from paper_2312_03415_amd import synth

pytestmark = pytest.mark.gpu


def padded(t, extra):
    import torch
    buf = torch.full((t.shape[0], t.shape[1] + extra), float("nan"), dtype=t.dtype, device="cuda")
    v = buf[:, :t.shape[1]]
    v.copy_(t)
    return v


# (n, i, o, r): whole tiles of 128 x 64 and 64 x 128; one row / eight columns past them; r with a ragged last column tile;
# long token and feature contractions (split where the layer's dX product brings scratch)
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("n,i,o,r", [(2048, 1024, 1024, 128), (2049, 1032, 1160, 128), (1300, 2056, 520, 72), (4096, 264, 2048, 40),
                                     (129, 4104, 4096, 104), (3000, 520, 3080, 64)])
def test_rank_products_against_the_oracle(n, i, o, r, dtype):
    import torch
    print(f"case {n} {i}->{o} r={r} {dtype}", flush=True)
    L = synth.Layer("rank", n, i, o, r, dtype, 5)
    st = synth.layer_inputs(L)
    host = {k: synth.widen(v, dtype) for k, v in st.items()}
    dev = {k: to_device(v, dtype) for k, v in st.items()}
    X, dY = padded(dev["X"], 8), padded(dev["dY"], 16)
    td = torch_dtype(dtype)
    want = oracle.scaled_backward(host["X"], host["W"], host["A"], host["B"], host["dY"], 0.5)
    Yw = oracle.scaled_forward(host["X"], host["W"], host["A"], host["B"], 0.5)
    code = rl.dtype_from_name(dtype)
    for bwd, wants in ((1, "XAB"), (5, "XAB"), (1, "A"), (1, "B")):
        Y = torch.empty((n, o), dtype=td, device="cuda")
        ws = rl.new_workspace(1, bwd, n, i, o, r, code)
        saved = rl.new_saved()
        rl.runlora_forward(1, X, dev["W"], dev["A"], dev["B"], Y, saved, workspace=ws, scale=0.5)
        dX = torch.empty((n, i), dtype=td, device="cuda") if "X" in wants else None
        dA = torch.full((i, r), float("nan"), dtype=td, device="cuda") if "A" in wants else None
        dB = torch.full((r, o), float("nan"), dtype=td, device="cuda") if "B" in wants else None
        rl.runlora_backward(bwd, dY, saved, dev["W"], dev["A"], dev["B"], dX, dA, dB, workspace=ws)
        torch.cuda.synchronize()
        assert relerr(to_f64(Y), Yw) < TOL[dtype]
        for got, w, name in ((dX, want[0], "dX"), (dA, want[1], "dA"), (dB, want[2], "dB")):
            if got is not None:
                assert relerr(to_f64(got), w) < TOL[dtype], (bwd, wants, name)


def test_paired_rank_products_run_on_the_middle_sized_kernel():
    """The rule's two sides: 8192 tokens at r = 128 take the paired launch, r = 32 stays on the streaming kernel."""
    import torch
    for r, cfg in ((128, 15), (32, 8)):
        n, i, o = 8192, 4096, 11008
        g = torch.Generator(device="cuda").manual_seed(1)
        mk = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
        X, W, A, B, dY = mk(n, i), mk(i, o), mk(i, r), mk(r, o), mk(n, o)
        Y, dA, dB = torch.empty_like(dY), torch.empty_like(A), torch.empty_like(B)
        ws = rl.new_workspace(1, 1, n, i, o, r, rl.RL_BF16)
        saved = rl.new_saved()
        rl.runlora_forward(1, X, W, A, B, Y, saved, workspace=ws)
        rl.runlora_profile_enable(16)
        rl.runlora_backward(1, dY, saved, W, A, B, None, dA, dB, workspace=ws)
        torch.cuda.synchronize()
        steps = rl.runlora_profile_collect(16)
        rl.runlora_profile_disable()
        assert [s["tile_cfg"] for s in steps] == [cfg, cfg], steps
