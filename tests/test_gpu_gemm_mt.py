"""GPU: the middle-sized matrix-core kernel (tile ids 12-16 of runlora_gemm) at the edges of its tiles, K tiles and ring of
stages, in every layout, whole and split, against the oracle's product of integer-valued operands: bit for bit."""
import numpy as np
import pytest

import oracle
from helpers import to_device, to_f64, torch_dtype
from paper_2312_03415_amd import binding as rl
from paper_2312_03415_amd import synth

pytestmark = pytest.mark.gpu

LAYOUTS = {"NN": (False, False), "NT": (False, True), "TN": (True, False)}
# (M, N, K, K2): one element; one tile of each id short of / at / past its edge; one K tile, fewer K tiles than stages,
# a partial K tile in the first segment, in the second, in both; a short second segment alone in its K tile
SHAPES = [(1, 8, 8, 0), (64, 64, 64, 0), (127, 120, 72, 0), (129, 136, 128, 8), (256, 128, 192, 64), (257, 264, 320, 24),
          (72, 392, 456, 40), (511, 72, 136, 128)]


def integers(rng, shape, hi, dtype):
    v = rng.integers(-hi, hi + 1, size=shape).astype(np.float64)
    return to_device(synth.store(v, dtype), dtype), v


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("layout", list(LAYOUTS))
@pytest.mark.parametrize("cfg", [12, 13, 14, 15, 16])
def test_middle_sized_kernel_is_exact_on_integers(cfg, layout, dtype):
    import torch
    a_str, b_kc = LAYOUTS[layout]
    rng = np.random.default_rng(cfg)
    td = torch_dtype(dtype)
    for M, N, K, K2 in SHAPES:
        if a_str:
            M = (M + 7) // 8 * 8
        print(f"case cfg={cfg} {layout} {dtype} {M}x{N}x{K}+{K2}", flush=True)
        A, Ah = integers(rng, (K, M) if a_str else (M, K), 1, dtype)
        B, Bh = integers(rng, (N, K) if b_kc else (K, N), 1, dtype)
        want = oracle.matmul(Ah, Bh, ta=a_str, tb=b_kc)
        A2 = B2 = None
        if K2:
            A2, A2h = integers(rng, (K2, M) if a_str else (M, K2), 1, dtype)
            B2, B2h = integers(rng, (N, K2) if b_kc else (K2, N), 1, dtype)
            want = want + oracle.matmul(A2h, B2h, ta=a_str, tb=b_kc)
        D, Dh = integers(rng, (M, N), 9, dtype)
        bias, bh = integers(rng, (N,), 9, dtype)
        full = 0.5 * want + Dh + bh
        assert np.abs(full).max() <= 128 and np.abs(want).max() <= 256   # halves up to 128: exact in bf16's 8-bit significand
        for splits in (1, 2, 5):
            buf = torch.full((M + 2, N + 16), 7.0, dtype=td, device="cuda")
            C = buf[1:M + 1, 8:N + 8]
            rl.runlora_gemm(A, B, C, a_strided=a_str, b_kcontig=b_kc, A2=A2, B2=B2, tile_cfg=cfg, splits=splits)
            torch.cuda.synchronize()
            assert np.array_equal(to_f64(C), want), (M, N, K, K2, splits)
            edge = to_f64(buf)
            edge[1:M + 1, 8:N + 8] = 7.0
            assert np.array_equal(edge, np.full_like(edge, 7.0)), (M, N, K, K2, splits)
            rl.runlora_gemm(A, B, C, a_strided=a_str, b_kcontig=b_kc, A2=A2, B2=B2, D=D, tile_cfg=cfg, splits=splits, alpha=0.5, bias=bias)
            torch.cuda.synchronize()
            assert np.array_equal(to_f64(C), full), (M, N, K, K2, splits, "options")


@pytest.mark.parametrize("layout", list(LAYOUTS))
def test_planned_products_match_the_generic_engine(layout):
    """The plan the library picks (any of the matrix-core kernels, tail launches and splits among them) and the generic
    engine sum the same integers: equal bits for shapes across the rule's range, operands with padded rows."""
    import torch
    a_str, b_kc = LAYOUTS[layout]
    g = torch.Generator(device="cuda").manual_seed(3)

    def operand(rows, cols):
        buf = torch.randint(-1, 2, (rows, cols + 24), generator=g, device="cuda").to(torch.bfloat16)
        return buf[:, 8:cols + 8]

    for M, N, K, K2 in [(40, 40, 4096, 16), (200, 768, 768, 8), (520, 4104, 2056, 0), (1000, 2056, 520, 24), (2048, 11008, 264, 32),
                        (4096, 2816, 1032, 8), (4104, 72, 1992, 0)]:
        print(f"case {layout} {M}x{N}x{K}+{K2}", flush=True)
        A = operand(K, M) if a_str else operand(M, K)
        B = operand(N, K) if b_kc else operand(K, N)
        A2 = (operand(K2, M) if a_str else operand(M, K2)) if K2 else None
        B2 = (operand(N, K2) if b_kc else operand(K2, N)) if K2 else None
        outs = []
        for cfg, splits in ((-1, 0), (1, 1)):
            C = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
            rl.runlora_gemm(A, B, C, a_strided=a_str, b_kcontig=b_kc, A2=A2, B2=B2, tile_cfg=cfg, splits=splits)
            torch.cuda.synchronize()
            outs.append(C)
        # sums of +-1 over a few thousand terms are exact in fp32 whatever the order; the one rounding to bf16 is the same
        assert torch.equal(outs[0], outs[1]), (M, N, K, K2)
