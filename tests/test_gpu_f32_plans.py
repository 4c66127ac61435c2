"""GPU: fp32 products on the tile shape and K split that the library's model picks, against the same product on 128x128 tiles with
the contraction whole: integer sums, equal bits."""
import pytest

from paper_2312_03415_amd import binding as rl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", ["NN", "NT", "TN"])
def test_planned_fp32_products_are_exact_on_integers(layout):
    import torch
    a_str, b_kc = {"NN": (False, False), "NT": (False, True), "TN": (True, False)}[layout]
    g = torch.Generator(device="cuda").manual_seed(4)
    operand = lambda rows, cols: torch.randint(-2, 3, (rows, cols + 12), generator=g, device="cuda").float()[:, 4:cols + 4]
    for M, N, K, K2 in [(36, 36, 40, 0), (256, 768, 768, 8), (260, 772, 4100, 12), (1000, 516, 260, 0), (4100, 136, 516, 36), (700, 3004, 132, 4), (132, 36, 3000, 8)]:
        print(f"case {layout} {M}x{N}x{K}+{K2}", flush=True)
        A, B = operand(*((K, M) if a_str else (M, K))), operand(*((N, K) if b_kc else (K, N)))
        A2 = operand(*((K2, M) if a_str else (M, K2))) if K2 else None
        B2 = operand(*((N, K2) if b_kc else (K2, N))) if K2 else None
        outs = []
        for cfg, splits in ((-1, 0), (1, 1)):
            buf = torch.full((M + 2, N + 8), 7.0, device="cuda")
            rl.runlora_gemm(A, B, buf[1:M + 1, 4:N + 4], a_strided=a_str, b_kcontig=b_kc, A2=A2, B2=B2, tile_cfg=cfg, splits=splits)
            torch.cuda.synchronize()
            outs.append(buf)
        assert torch.equal(outs[0], outs[1]), (M, N, K, K2)   # (sums of small integers are exact in fp32; the rim is untouched)
