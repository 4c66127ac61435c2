"""W + s A B (forward 2's kept M) and the rank-r updates of the default chain on the merge kernel, at the edges of its column strips
(256 a workgroup, 64 a wave), row blocks (32) and rank steps (16), against float64."""
import pytest

from helpers import TOL, relerr, to_f64, torch_dtype
from paper_2312_03415_amd import binding as rl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("i,o,r", [(8, 8, 8), (32, 64, 16), (33 * 8, 72, 24), (1032, 256, 32), (64, 264, 40), (2080, 520, 64), (1288, 1096, 72), (40, 4360, 128)])
def test_merged_weight_and_updates(i, o, r, dtype):
    import torch
    n, s, td, code = 40, 0.5, torch_dtype(dtype), rl.dtype_from_name(dtype)
    g = torch.Generator().manual_seed(i + o + r)
    t = {k: torch.randn(*sh, generator=g).to(td).cuda() for k, sh in (("X", (n, i)), ("W", (i, o)), ("A", (i, r)), ("B", (r, o)), ("dY", (n, o)))}
    d = {k: v.double().cpu() for k, v in t.items()}
    print(f"case merge {i}x{o} r{r} {dtype}", flush=True)
    nan = float("nan")
    Y, M = torch.full((n, o), nan, dtype=td, device="cuda"), torch.full((i, o), nan, dtype=td, device="cuda")
    saved = rl.new_saved(None, M)
    rl.runlora_forward(rl.FWD2, t["X"], t["W"], t["A"], t["B"], Y, saved, workspace=rl.new_workspace(rl.FWD2, -1, n, i, o, r, code), scale=s)
    AB = s * (d["A"] @ d["B"])
    want = d["W"] + AB
    # one rounding (half a unit of the last of 8 or 11 bits), and fp32 sums of r products
    bound = {"bf16": 2.0 ** -8, "f16": 2.0 ** -11}[dtype] * want.abs() + 2.0 ** -23 * (r + 2) * (s * (d["A"].abs() @ d["B"].abs()) + d["W"].abs())
    assert bool(((M.double().cpu() - want).abs() <= bound + 2.0 ** -25).all())
    assert relerr(to_f64(Y), (d["X"] @ want).numpy()) < TOL[dtype]
    # Y += T B and dX += Z1 A^T (A as stored: the contraction runs along its rows)
    T = torch.full((n, r), nan, dtype=td, device="cuda")
    saved = rl.new_saved(T)
    ws = rl.new_workspace(rl.FWD_DEFAULT, rl.BWD_DEFAULT, n, i, o, r, code)
    rl.runlora_forward(rl.FWD_DEFAULT, t["X"], t["W"], t["A"], t["B"], Y, saved, workspace=ws, scale=s)
    dX, dA, dB = (torch.full(sh, nan, dtype=td, device="cuda") for sh in ((n, i), (i, r), (r, o)))
    rl.runlora_backward(rl.BWD_DEFAULT, t["dY"], saved, t["W"], t["A"], t["B"], dX, dA, dB, workspace=ws)
    torch.cuda.synchronize()
    assert relerr(to_f64(Y), (d["X"] @ d["W"] + s * (d["X"] @ d["A"]) @ d["B"]).numpy()) < TOL[dtype]
    assert relerr(to_f64(dX), (d["dY"] @ d["W"].T + s * (d["dY"] @ d["B"].T) @ d["A"].T).numpy()) < TOL[dtype]
