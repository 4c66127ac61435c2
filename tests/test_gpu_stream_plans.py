"""GPU: the builds that skinny_plan chooses between for the rank-r products of Algorithm 1: 64- or 32-row workgroups for dA, dB;
16 or 4 wavefronts for products with X under LoRA dropout.  Sizes on both sides of each rule, ragged, against the oracle."""
import numpy as np
import pytest

import oracle
from helpers import TOL, layer_on_device, relerr, to_f64, torch_dtype
from paper_2312_03415_amd import binding as rl
from paper_2312_03415_amd import synth

pytestmark = pytest.mark.gpu


def gradients(L, p, seed):
    """Y, dA and dB of forward 1 / Algorithm 1 on the GPU and from the oracle."""
    import torch
    dev, host = layer_on_device(L)
    td, code = torch_dtype(L.dtype), rl.dtype_from_name(L.dtype)
    Y, dA, dB = (torch.full(s, float("nan"), dtype=td, device="cuda") for s in ((L.n, L.o), (L.i, L.r), (L.r, L.o)))
    ws = torch.full((rl.runlora_workspace_bytes(1, 1, L.n, L.i, L.o, L.r, code) + (1 << 20),), 0xFF, dtype=torch.uint8, device="cuda")
    saved = rl.new_saved()
    drop = dict(dropout_p=p, dropout_seed=seed) if p else {}
    rl.runlora_forward(1, dev["X"], dev["W"], dev["A"], dev["B"], Y, saved, workspace=ws, **drop)
    rl.runlora_backward(1, dev["dY"], saved, dev["W"], dev["A"], dev["B"], None, dA, dB, workspace=ws)
    torch.cuda.synchronize()
    mask, pq = oracle.dropout_mask(L.n, L.i, p, seed) if p else (np.ones((L.n, L.i)), 0.0)
    s, Xm = 1.0 / (1.0 - pq), host["X"] * mask
    T, Z1 = oracle.matmul(Xm, host["A"]), oracle.matmul(host["dY"], host["B"], tb=True)
    want = (oracle.matmul(host["X"], host["W"]) + s * oracle.matmul(T, host["B"]), s * oracle.matmul(Xm, Z1, ta=True), s * oracle.matmul(T, host["dY"], ta=True))
    return [(name, relerr(to_f64(got), w)) for name, got, w in zip(("Y", "dA", "dB"), (Y, dA, dB), want)]


# (n, i, o, r): K tiles of the masked product below, at and past 24 (16 bits: 64 columns, fp32: 32), one row and a row more than a
# block, the masked part shorter than half of the other, r at both ends of a column block and beyond it
@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("n,i,o,r", [(1, 1536, 264, 8), (33, 1472, 72, 16), (97, 1544, 392, 32), (64, 2120, 4504, 24), (200, 4104, 136, 32), (130, 1608, 328, 40)])
def test_masked_products_on_many_waves(n, i, o, r, dtype):
    L = synth.Layer("masked", n, i, o, r, dtype, 51)
    print(f"case {n} {i}->{o} r={r} {dtype}", flush=True)
    for name, err in gradients(L, 0.3, 77):
        assert err < TOL[dtype], (name, err)


# 64-row blocks of X and dY: 64 and fewer with a short contraction and with a long one, between 65 and 128, more than 128
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n,i,o,r", [(200, 264, 392, 8), (4104, 136, 200, 24), (72, 4104, 136, 16), (72, 4104, 4104, 32), (136, 4104, 4168, 8)])
def test_gradients_in_32_and_64_row_blocks(n, i, o, r, dtype):
    L = synth.Layer("blocks", n, i, o, r, dtype, 52)
    print(f"case {n} {i}->{o} r={r} {dtype}", flush=True)
    for name, err in gradients(L, 0.0, 0):
        assert err < TOL[dtype], (name, err)
