"""GPU: rank-r products of X under LoRA dropout with r > 32 on the middle-sized kernel, T = (X o m) A and dA = (X o m)^T Z1, at edges of its
tiles (128 tokens or columns, 64 of the rank, 64 of the contraction), alone, in pairs, in slices, and on the streaming kernel next to it."""
import numpy as np
import pytest

import oracle
from helpers import TOL, elem_excess, layer_on_device, relerr, to_f64, torch_dtype
from paper_2312_03415_amd import binding as rl
from paper_2312_03415_amd import synth

pytestmark = pytest.mark.gpu


# (n, i, o, r), is T / the {Z1, T} pair / the {dA, dB} pair on tiles of the middle-sized kernel (ids 12-16)?
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("n,i,o,r,mt", [(1025, 4104, 1032, 64, (1, 1, 1)),   # a row, eight columns past the tiles; slices
                                        (1025, 2056, 4104, 64, (0, 1, 1)), (2048, 1024, 2048, 128, (0, 1, 1)), (700, 3000, 704, 96, (1, 1, 1)),
                                        (129, 4104, 4096, 40, (1, 1, 1)),    # long contraction over few tokens
                                        (4097, 2056, 2056, 72, (1, 1, 1)),   # 128x128 tiles for {Z1, T}
                                        (2049, 8200, 2568, 128, (1, 1, 1)),  # and for both pairs
                                        (300, 512, 512, 48, (0, 0, 1)), (40, 264, 136, 64, (0, 1, 1)), (1500, 1024, 1024, 64, (0, 0, 0))])
def test_masked_rank_products(n, i, o, r, mt, dtype):
    import torch
    L = synth.Layer("maskrank", n, i, o, r, dtype, 71)
    dev, host = layer_on_device(L)
    td, code, p, seed, scale = torch_dtype(dtype), rl.dtype_from_name(dtype), 0.3, 1234, 0.5
    print(f"case {n} {i}->{o} r={r} {dtype}", flush=True)
    mask, pq = oracle.dropout_mask(n, i, p, seed)
    Xm, s = host["X"] * mask, scale / (1.0 - pq)
    T, Z1 = s * (Xm @ host["A"]), s * (host["dY"] @ host["B"].T)
    want = {"T": T, "dA": Xm.T @ Z1, "dB": T.T @ host["dY"], "Y": host["X"] @ host["W"] + T @ host["B"]}
    nan = float("nan")
    for bring in ("all", "none to split into"):
        ws = rl.new_workspace(rl.FWD1, rl.BWD1, n, i, o, r, code)
        ws.fill_(0xFF)
        got = {k: torch.full(sh, nan, dtype=td, device="cuda") for k, sh in (("T", (n, r)), ("dA", (i, r)), ("dB", (r, o)), ("Y", (n, o)))}
        rl.runlora_profile_enable(16)
        # T alone, kept; then both pairs (T formed again), without dX
        saved = rl.new_saved(got["T"])
        rl.runlora_forward(rl.FWD1, dev["X"], dev["W"], dev["A"], dev["B"], got["Y"], saved, workspace=ws, scale=scale, dropout_p=p, dropout_seed=seed)
        saved.T, saved.ldt = None, 0
        if bring != "all":  # two rank-r factors and nothing else
            ws = ws[:2 * ((n * r * 2 + 255) // 256 * 256)]
        rl.runlora_backward(rl.BWD1, dev["dY"], saved, dev["W"], dev["A"], dev["B"], None, got["dA"], got["dB"], workspace=ws)
        torch.cuda.synchronize()
        steps = rl.runlora_profile_collect(16)
        rl.runlora_profile_disable()
        if bring == "all":
            cfgs = [st["tile_cfg"] for st in steps if "Y =" not in st["what"]]
            assert len(cfgs) == 3 and [int(c >= 12) for c in cfgs] == list(mt), steps
        for k, w in want.items():
            g = to_f64(got[k])
            assert relerr(g, w) < TOL[dtype], (k, bring)
            if k == "T":  # formed in one step from stored operands: a dropped or kept chunk too many moves every element of its row
                assert elem_excess(g, w, dtype) < 1.0


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("n,i,o,r", [(300, 8200, 72, 8), (65, 4104, 4200, 32),    # 64-row blocks of a pair, masked; rows and columns past the tiles
                                     (1019, 8480, 96, 40), (4160, 520, 264, 16),  # r > 32; few blocks and a long contraction
                                     (70, 2056, 136, 16), (33, 72, 40, 8)])       # 32-row blocks
def test_masked_streaming_pairs(n, i, o, r, dtype):
    """{dA, dB} on the streaming kernel (and {Z1, T} for r <= 32) with rows of X, dY and the outputs further apart than they are long."""
    import torch
    if dtype == "f32" and n * i * o > 2e9:
        pytest.skip("the reference takes long")
    td, code, p, seed, s = torch_dtype(dtype), rl.dtype_from_name(dtype), 0.3, 77, 0.5
    print(f"case stream {n} {i}->{o} r={r} {dtype}", flush=True)
    g = torch.Generator().manual_seed(n + i)
    mk = lambda rows, cols, var: (torch.randn(rows, cols + 8, generator=g) * var ** 0.5).to(td).cuda()[:, :cols]
    X, dY, W, A, B = mk(n, i, 1.0), mk(n, o, 1.0), mk(i, o, 1.0 / i), mk(i, r, 1.0 / i), mk(r, o, 1.0 / r)
    y = torch.empty(n, o, dtype=td, device="cuda")
    out = [torch.full((a + 1, b + 8), 7.0, dtype=td, device="cuda") for a, b in ((i, r), (r, o))]
    ws = rl.new_workspace(rl.FWD1, rl.BWD1, n, i, o, r, code)
    ws.fill_(0xFF)
    saved = rl.new_saved(None)
    rl.runlora_forward(rl.FWD1, X, W, A, B, y, saved, workspace=ws, scale=s, dropout_p=p, dropout_seed=seed)
    rl.runlora_profile_enable(8)
    rl.runlora_backward(rl.BWD1, dY, saved, W, A, B, None, out[0][:i, :r], out[1][:r, :o], workspace=ws)
    torch.cuda.synchronize()
    steps = rl.runlora_profile_collect(8)
    rl.runlora_profile_disable()
    streaming = [8 <= st["tile_cfg"] <= 10 for st in steps]
    assert len(steps) == 2 and streaming[1] and (r > 32 or streaming[0]), steps
    mask, pq = oracle.dropout_mask(n, i, p, seed)
    f = lambda t: t.double().cpu().numpy()
    Xm, sc = f(X) * mask, s / (1.0 - pq)
    T, Z1 = sc * (Xm @ f(A)), sc * (f(dY) @ f(B).T)
    for got, want in ((f(y), f(X) @ f(W) + T @ f(B)), (f(out[0][:i, :r]), Xm.T @ Z1), (f(out[1][:r, :o]), T.T @ f(dY))):
        assert relerr(got, want) < TOL[dtype]
    for t, (a, b) in zip(out, ((i, r), (r, o))):
        assert bool((t[a] == 7.0).all()) and bool((t[:, b:] == 7.0).all())
