"""GPU: dX = dY W^T + m o (Z1 A^T) of a layer with LoRA dropout, in one launch where the product's plan is built for it, in two
otherwise, on every kernel that serves it, against the oracle."""
import re

import numpy as np
import pytest

import oracle
from helpers import TOL, elem_excess, layer_on_device, relerr, to_f64, torch_dtype
from paper_2312_03415_amd import binding as rl
from paper_2312_03415_amd import synth

pytestmark = pytest.mark.gpu


# ids of rl_step_time_t: 7 = 256x256 tiles, 12-16 = the middle-sized kernel; launches of dX
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("n,i,o,r,fused", [(4104, 2568, 1096, 16, True),    # 256x256, ragged in both directions
                                           (8192, 4352, 1032, 32, True),    # 256x256 with a column of tiles cut off: the mask's column offset
                                           (4352, 2816, 264, 40, False),    # 256x256 and r > 32
                                           (1237, 2056, 5464, 24, True),    # 256x128, contraction split: segment 0 in the first slice only
                                           (300, 264, 4096, 32, True),      # 64x128, many slices
                                           (200, 264, 392, 128, True),      # segment 0 of two K tiles
                                           (2100, 4104, 72, 8, True), (257, 520, 136, 8, True), (1000, 4104, 200, 72, True),
                                           (24, 264, 136, 16, False)])      # few rows: the generic engine
def test_masked_update_of_dX(n, i, o, r, fused, dtype):
    import torch
    L = synth.Layer("maskdx", n, i, o, r, dtype, 61)
    dev, host = layer_on_device(L)
    td, code, p, seed, scale = torch_dtype(dtype), rl.dtype_from_name(dtype), 0.4, 99, 0.5
    print(f"case {n} {i}->{o} r={r} {dtype}", flush=True)
    mask, pq = oracle.dropout_mask(n, i, p, seed)
    rows = np.unique(np.concatenate([np.arange(0, n, 251), np.arange(15, n, 256), [n - 1]]))
    Z1 = scale / (1.0 - pq) * oracle.matmul(host["dY"][rows], host["B"], tb=True)
    want = oracle.matmul(host["dY"][rows], host["W"], tb=True) + mask[rows] * oracle.matmul(Z1, host["A"], tb=True)
    Y = torch.empty((n, o), dtype=td, device="cuda")
    buf = torch.full((n + 2, i + 16), 7.0, dtype=td, device="cuda")
    dX = buf[1:n + 1, 8:i + 8]
    ws = torch.full((rl.runlora_workspace_bytes(1, 1, n, i, o, r, code),), 0xFF, dtype=torch.uint8, device="cuda")
    saved = rl.new_saved()
    rl.runlora_forward(1, dev["X"], dev["W"], dev["A"], dev["B"], Y, saved, workspace=ws, scale=scale, dropout_p=p, dropout_seed=seed)
    rl.runlora_profile_enable(16)
    rl.runlora_backward(1, dev["dY"], saved, dev["W"], dev["A"], dev["B"], dX, None, None, workspace=ws)
    torch.cuda.synchronize()
    steps = [s["what"] for s in rl.runlora_profile_collect(16)]
    rl.runlora_profile_disable()
    assert ("dX = m o (Z1 A^T) + dY W^T" in steps) == fused and ("dX += Z1 A^T" in steps) != fused, steps
    got = to_f64(dX)[rows]
    assert relerr(got, want) < TOL[dtype]
    assert elem_excess(got, want, dtype, roundings=1 if fused else 2) < 1.0
    edge = buf.float()
    edge[1:n + 1, 8:i + 8] = 7.0
    assert bool((edge == 7.0).all())   # nothing beyond dX is written


@pytest.mark.parametrize("n,i,o,r", [(492, 104, 9568, 48), (706, 1384, 1112, 128)])
def test_masked_update_in_the_workspace_of_two_launches(n, i, o, r):
    """A call that brings what dX = dY W^T and its masked update take, less than their one launch does, runs those."""
    import torch
    L = synth.Layer("masktwo", n, i, o, r, "bf16", 62)
    dev, host = layer_on_device(L)
    p, seed, scale = 0.4, 99, 0.5
    print(f"case {n} {i}->{o} r={r}", flush=True)
    Y, dX = (torch.full(s, float("nan"), dtype=torch.bfloat16, device="cuda") for s in ((n, o), (n, i)))
    full = rl.runlora_workspace_bytes(1, 1, n, i, o, r, rl.RL_BF16)
    saved = rl.new_saved()
    rl.runlora_forward(1, dev["X"], dev["W"], dev["A"], dev["B"], Y, saved, workspace=torch.empty(full, dtype=torch.uint8, device="cuda"),
                       scale=scale, dropout_p=p, dropout_seed=seed)
    back = lambda ws: rl.runlora_backward(1, dev["dY"], saved, dev["W"], dev["A"], dev["B"], dX, None, None, workspace=ws)
    with pytest.raises(rl.RunLoRAError) as e:
        back(torch.empty(256, dtype=torch.uint8, device="cuda"))
    assert e.value.code == rl.RL_ERR_WORKSPACE
    least = int(re.search(r"(\d+) bytes", str(e.value)).group(1))
    rl.runlora_profile_enable(16)
    back(torch.full((least,), 0xFF, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    steps = [s["what"] for s in rl.runlora_profile_collect(16)]
    rl.runlora_profile_disable()
    assert steps[-2:] == ["dX = dY W^T", "dX += Z1 A^T"], steps
    mask, pq = oracle.dropout_mask(n, i, p, seed)
    Z1 = scale / (1.0 - pq) * oracle.matmul(host["dY"], host["B"], tb=True)
    want = oracle.matmul(host["dY"], host["W"], tb=True) + mask * oracle.matmul(Z1, host["A"], tb=True)
    assert relerr(to_f64(dX), want) < TOL["bf16"] and elem_excess(to_f64(dX), want, "bf16", roundings=2) < 1.0
