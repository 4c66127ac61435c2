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


# (n, i, o, r): K tiles of the masked product (16 bits: 64 columns, fp32: 32) below, at and past 24 and 48, whole (16 waves from 48 on) and in
# slices, one row and a row more than a block, the masked part shorter than half of the other, r at both ends of a column block and beyond it
@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("n,i,o,r", [(1, 1536, 264, 8), (33, 1472, 72, 16), (97, 1544, 392, 32), (64, 2120, 4504, 24), (200, 4104, 136, 32), (130, 1608, 328, 40),
                                     (33, 3000, 72, 16), (1, 3016, 264, 8), (97, 3080, 392, 32), (65, 4088, 136, 24), (1030, 4104, 136, 16)])
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


# dA, dB from 44 MB of operands on: 128x128 tiles, a ragged last tile of each, tokens a row past a K tile; r at the edges of one column tile
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("n,i,o,r", [(8257, 1032, 2056, 72), (8193, 520, 3080, 128)])
def test_gradients_of_wide_pairs(n, i, o, r, dtype):
    L = synth.Layer("wide", n, i, o, r, dtype, 54)
    print(f"case {n} {i}->{o} r={r} {dtype}", flush=True)
    for name, err in gradients(L, 0.0, 0):
        assert err < TOL[dtype], (name, err)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("n,i,o,r", [(520, 2056, 2120, 64), (1032, 4104, 1096, 40), (300, 1000, 3000, 128), (2056, 264, 4104, 72),
                                     (4104, 520, 2056, 128), (1032, 4104, 1096, 256), (2056, 1096, 4104, 136), (200, 392, 264, 200),
                                     (520, 1032, 1096, 264)])
def test_rank_products_with_and_without_scratch_for_splits(n, i, o, r, dtype):
    """r > 32: with the workspace that the query names, a rank-r product may split its contraction into a few MB of it; a call whose
    workspace holds only what the other launches take (the figure in the error text) still runs, unsplit.  Integers: the same bits."""
    import re

    import torch
    rng = np.random.default_rng(n)
    td, code = torch_dtype(dtype), rl.dtype_from_name(dtype)
    pick = lambda shape, p: torch.from_numpy((rng.random(shape) < p) * rng.choice([-1.0, 1.0], size=shape)).to(td).cuda()
    X, W, A, B, dY = pick((n, i), 0.05), pick((i, o), 0.02), pick((i, r), 0.02), pick((r, o), 0.02), pick((n, o), 0.02)
    print(f"case {n} {i}->{o} r={r} {dtype}", flush=True)

    def run(wf, wb):
        outs = [torch.full(s, float("nan"), dtype=td, device="cuda") for s in ((n, o), (n, i), (i, r), (r, o))]
        saved = rl.new_saved()
        rl.runlora_forward(1, X, W, A, B, outs[0], saved, workspace=wf)
        rl.runlora_backward(1, dY, saved, W, A, B, *outs[1:], workspace=wb)
        torch.cuda.synchronize()
        return outs

    def least(call):
        with pytest.raises(rl.RunLoRAError) as e:
            call(torch.empty(256, dtype=torch.uint8, device="cuda"))
        assert e.value.code == rl.RL_ERR_WORKSPACE
        return torch.full((int(re.search(r"(\d+) bytes", str(e.value)).group(1)),), 0xFF, dtype=torch.uint8, device="cuda")

    full = torch.full((rl.runlora_workspace_bytes(1, 1, n, i, o, r, code),), 0xFF, dtype=torch.uint8, device="cuda")
    outs = run(full, full)
    saved = rl.new_saved()
    rl.runlora_forward(1, X, W, A, B, torch.empty_like(dY), saved, workspace=full)
    small_f = least(lambda w: rl.runlora_forward(1, X, W, A, B, torch.empty_like(dY), rl.new_saved(), workspace=w))
    small_b = least(lambda w: rl.runlora_backward(1, dY, saved, W, A, B, torch.empty_like(X), torch.empty_like(A), torch.empty_like(B), workspace=w))
    assert min(small_f.numel(), small_b.numel()) < full.numel()
    for a, b in zip(outs, run(small_f, small_b)):
        assert torch.equal(a, b)
    h = [to_f64(t) for t in (X, W, A, B, dY)]
    T, Z = h[0] @ h[2], h[4] @ h[3].T
    want = (h[0] @ h[1] + T @ h[3], h[4] @ h[1].T + Z @ h[2].T, h[0].T @ Z, T.T @ h[4])
    for got, w in zip(outs, want):
        assert np.abs(w).max() <= 256 and np.array_equal(to_f64(got), w)   # integers bf16 holds


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("n,i,o,r", [(4096, 4096, 4096, 256), (2056, 1096, 4104, 192), (520, 1032, 1096, 264), (4104, 520, 2056, 136), (6577, 2824, 8496, 72),
                                     (1032, 4104, 1096, 40)])
def test_rank_products_with_T_kept_and_with_fewer_gradients(n, i, o, r, dtype):
    """Algorithm 1 in exactly the bytes that the query names, with T = X A kept or not, for every choice of gradients (a VeRA layer never wants
    dA): Z1, X A, dA and dB then run alone or in pairs, each with splits of its own.  Integers: the same bits every time."""
    import torch
    rng = np.random.default_rng(n + r)
    td, code = torch_dtype(dtype), rl.dtype_from_name(dtype)
    pick = lambda shape, p: torch.from_numpy((rng.random(shape, dtype=np.float32) < p) * rng.choice(np.float32([-1.0, 1.0]), size=shape)).to(td).cuda()
    X, W, A, B, dY = pick((n, i), 0.02), pick((i, o), 0.01), pick((i, r), 0.01), pick((r, o), 0.01), pick((n, o), 0.01)
    print(f"case {n} {i}->{o} r={r} {dtype}", flush=True)
    f32 = lambda t: t.float().contiguous()
    Z, T = (f32(dY) @ f32(B.t())).to(td), (f32(X) @ f32(A)).to(td)   # (sums of integers below 2^24: exact in fp32; below 257 in bf16)
    want = {"dX": f32(dY) @ f32(W.t()) + f32(Z) @ f32(A.t()), "dA": f32(X.t()) @ f32(Z), "dB": f32(T.t()) @ f32(dY)}
    assert max(float(v.abs().max()) for v in (Z, T, *want.values())) <= 256
    wb = torch.empty((rl.runlora_workspace_bytes(-1, 1, n, i, o, r, code),), dtype=torch.uint8, device="cuda")
    wf = torch.empty((rl.runlora_workspace_bytes(1, -1, n, i, o, r, code),), dtype=torch.uint8, device="cuda")
    for keep in (False, True):
        wf.fill_(0xFF)
        kept = torch.full((n, r), float("nan"), dtype=td, device="cuda") if keep else None
        saved = rl.new_saved(kept)
        rl.runlora_forward(1, X, W, A, B, torch.empty_like(dY), saved, workspace=wf)
        for names in (("dX", "dA", "dB"), ("dX", "dA"), ("dX", "dB"), ("dA", "dB"), ("dX",), ("dA",), ("dB",)):
            out = {k: torch.full(s, float("nan"), dtype=td, device="cuda") if k in names else None for k, s in (("dX", (n, i)), ("dA", (i, r)), ("dB", (r, o)))}
            wb.fill_(0xFF)
            rl.runlora_backward(1, dY, saved, W, A, B, *out.values(), workspace=wb)
            torch.cuda.synchronize()
            for k in names:
                assert torch.equal(out[k].float(), want[k]), (keep, names, k)


@pytest.mark.parametrize("int4", [False, True])
def test_rank_products_split_into_the_workspace_that_is_there(int4):
    """1024 x 4096 -> 4096, r 64, in its least workspace, in 60 % of the way to what the rank-r products take, and (int4) in too little for panels of
    W: they split as far as it goes, and integers come out the same."""
    import torch
    n, i, o, r, td = 1024, 4096, 4096, 64, torch.bfloat16
    rng = np.random.default_rng(3)
    pick = lambda shape, p: torch.from_numpy((rng.random(shape, dtype=np.float32) < p) * rng.choice(np.float32([-1.0, 1.0]), size=shape)).to(td).cuda()
    X, A, B, dY = pick((n, i), 0.02), pick((i, r), 0.01), pick((r, o), 0.01), pick((n, o), 0.01)
    if int4:
        W = rl.Int4Weight(torch.randint(0, 256, (i, o // 2), dtype=torch.uint8, device="cuda"), torch.full((i // 64, o), 0.125, dtype=torch.float16, device="cuda"), i, o)
    else:
        W = pick((i, o), 0.01)
    outs, splits = [], []
    # (the whole of it is 2.75 MB: T of 128 KB, partials of up to ten slices of 256 KB; 2.88: Z1 and X A, five slices each)
    for wf, wb in ((655360, 1310720), (1900000, 2300000), (2752512, 2883584)):
        Y, dX, dA, dB = (torch.full(s, float("nan"), dtype=td, device="cuda") for s in ((n, o), (n, i), (i, r), (r, o)))
        wsf, wsb = (torch.full((b,), 0xFF, dtype=torch.uint8, device="cuda") for b in (wf, wb))
        saved = rl.new_saved()
        print(f"case int4={int4} {wf} {wb}", flush=True)
        rl.runlora_profile_enable(16)
        rl.runlora_forward(1, X, W, A, B, Y, saved, workspace=wsf)
        rl.runlora_backward(1, dY, saved, W, A, B, dX, dA, dB, workspace=wsb)
        torch.cuda.synchronize()
        steps = {s["what"]: s["splits"] for s in rl.runlora_profile_collect(16)}
        rl.runlora_profile_disable()
        splits.append((steps["T = X A"], steps["Z1 = dY B^T ; Z2 = X A"]))
        outs.append((Y, dX, dA, dB))
    assert splits[0][0] < splits[1][0] < splits[2][0] and splits[0][1] < splits[1][1] < splits[2][1], splits
    for k in (1, 2):
        for a, b in zip(outs[0], outs[k]):
            assert torch.equal(a, b)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_few_tokens_in_every_number_of_slices(dtype):
    """lora_finish_kernel takes the slices four at a time (eight up to r = 32 where there are more than four), zeros beyond the last: 1 to 16 slices,
    every remainder with and without a four before it, ranks on both sides of 8, 16, 24 and of its steps of 32, bit for bit on integers."""
    import torch
    rng = np.random.default_rng(8)
    td, seen = torch_dtype(dtype), set()
    for n, i, o, r in [(1, 200, 264, 8), (2, 576, 136, 16), (3, 1024, 520, 24), (5, 1096, 264, 48), (9, 2056, 136, 104), (33, 4096, 72, 56),
                       (1, 4096, 1024, 40), (2, 8192, 136, 8), (40, 11008, 72, 16), (70, 4104, 264, 72), (1, 11008, 264, 128),
                       (3, 1600, 1032, 24), (1, 2000, 264, 24), (1, 2400, 264, 24)]:
        h = {"X": rng.integers(0, 2, (n, i)) * 1.0, "W": (rng.random((i, o)) < 0.005) * rng.choice([-1.0, 1.0], (i, o)),
             "A": (rng.random((i, r)) < 0.002) * 1.0, "B": (rng.random((r, o)) < 0.3) * rng.choice([-1.0, 1.0], (r, o))}
        dev = {k: torch.from_numpy(v).to(td).cuda() for k, v in h.items()}
        Y = torch.full((n, o), float("nan"), dtype=td, device="cuda")
        T = torch.full((n, r), float("nan"), dtype=td, device="cuda")
        ws = torch.full((rl.runlora_workspace_bytes(1, -1, n, i, o, r, rl.dtype_from_name(dtype)),), 0xFF, dtype=torch.uint8, device="cuda")
        print(f"case {n} {i}->{o} r={r} {dtype}", flush=True)
        rl.runlora_profile_enable(8)
        rl.runlora_forward(1, dev["X"], dev["W"], dev["A"], dev["B"], Y, rl.new_saved(T), workspace=ws)
        torch.cuda.synchronize()
        steps = rl.runlora_profile_collect(8)
        rl.runlora_profile_disable()
        if len(steps) == 1:
            seen.add(steps[0]["splits"])
        want_T = h["X"] @ h["A"]
        want = h["X"] @ h["W"] + want_T @ h["B"]
        assert np.abs(want).max() <= 256 and np.abs(want_T).max() <= 256   # integers bf16 holds
        assert np.array_equal(to_f64(T), want_T) and np.array_equal(to_f64(Y), want), (n, i, o, r)
    assert {s % 4 for s in seen if s < 4} == {1, 2, 3} and {s % 4 for s in seen if s >= 4} == {0, 1, 2, 3} and max(seen) > 8, seen
