"""Host-side checks of the plans the library makes for its launches (no GPU): what is taken is never modelled slower than what it
stands in for."""
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB_DIR = os.path.join(HERE, "..", "paper_2312_03415_amd")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plans") / "plan_probe")
    p = subprocess.run([HIPCC, "-std=c++17", "-O1", "--offload-arch=gfx950", os.path.join(HERE, "plan_probe.cpp"), "-o", exe,
                        "-L" + LIB_DIR, "-lrunlora", "-Wl,-rpath," + os.path.abspath(LIB_DIR)], capture_output=True, text=True)
    assert p.returncode == 0, p.stderr[-2000:]

    def ask(kind, rows):  # product: M, N, K, K of a second segment; few: tokens, d_in, d_out, r; padded: M, N, K, ld of A; int4: M, N, K, r
        text = "".join(kind + " " + " ".join(str(v) for v in r) + "\n" for r in rows)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.strip().split("\n")
        assert len(out) == len(rows)
        return [[float(v) for v in line.split()] for line in out]
    return ask


def products():
    rng = np.random.default_rng(5)
    dims = lambda hi: int(np.exp(rng.uniform(np.log(40), np.log(hi)))) // 8 * 8
    return [(int(np.exp(rng.uniform(np.log(33), np.log(8192)))), dims(12000), dims(12000), int(rng.choice([0, 8, 32, 128]))) for _ in range(400)]


def test_a_products_plan_is_not_modelled_slower_than_the_generic_engines(probe):
    rows = products()
    for r, (cfg, splits, tail, part, us, gcfg, gus) in zip(rows, probe("product", rows)):
        assert us <= gus * (1 + 1e-9), (r, cfg, splits, us, gcfg, gus)


def test_rows_that_split_lines_are_priced(probe):
    """4096 x 2056 x 5464: rows of 5464 and 2056 elements are no whole 128-byte lines, and narrow tiles pay most for them
    (64x128 tiles 182-201 us, 256x256 123-137); short contractions of many tiles stay on the middle-sized kernel."""
    wide, narrow = probe("product", [(4096, 2056, 5464, 0), (1024, 768, 768, 0)])
    assert wide[0] == 7 and narrow[0] >= 12


def test_operands_beyond_two_gib_stay_on_kernels_that_address_them(probe):
    """The middle-sized kernel addresses 2^30 elements of an operand, the 256x256 kernel twice that.  A product with a longer one
    (by its sizes or by its rows' distance) keeps the plan by tile counts, in the scratch reported for its sizes, instead of
    falling back from a middle-sized tile to the generic engine's 128x128."""
    rows = [(262144, 256, 4096, 4096), (262144, 2056, 4104, 4104), (200000, 1024, 2048, 8192), (524288, 264, 2056, 2056), (40000, 768, 768, 30000)]
    for r, (cfg, tail, part, reported) in zip(rows, probe("padded", rows)):
        assert cfg == 7 and tail == 7, (r, cfg, tail)
        assert part == reported, r
    short = probe("padded", [(r[0] // 8, r[1], r[2], r[2]) for r in rows])
    assert any(p[0] >= 12 or p[1] >= 12 for p in short)   # the same products with fewer rows do run on its tiles


def test_the_few_token_route_is_taken_where_it_is_modelled_faster(probe):
    """Two launches with the partials of [X W | X A] against T = X A and [X|T] [W;B]: a matter of rows and rank (256 x 4096 -> 11008,
    r 128: 66 us and 55; 48 rows, r 32: 23 and 33), and the workspace is the same either way."""
    rng = np.random.default_rng(6)
    rows = [(int(np.exp(rng.uniform(0, np.log(256)))), int(rng.integers(64, 1376)) * 8, int(rng.integers(64, 1376)) * 8, int(rng.choice([8, 32, 64, 128])))
            for _ in range(300)]
    taken = 0
    for r, (few, splits, us, other, ws) in zip(rows, probe("few", [(n, i, o, k) for n, i, o, k in rows])):
        assert bool(few) == (splits > 0 and us < other), (r, splits, us, other)
        taken += int(few)
    assert 150 < taken < 300
    wide, small, one = probe("few", [(256, 4096, 11008, 128), (48, 4096, 11008, 32), (1, 4096, 4096, 16)])
    assert not wide[0] and small[0] and one[0]


def test_int4_products_take_the_faster_route(probe):
    """Layers timed on both routes: panels of W on the dense kernels (512 x 2048 -> 2048 30.7 us against 38.8, 672 x 12960 -> 3208
    183 against 266, 4096 x 5120 -> 13824) and the kernels that dequantise on their way to LDS (913 x 6240 -> 6232 135 against 159,
    3748 x 12720 -> 7888 838 against 1156, 1062 x 8680 -> 7768 229 against 313)."""
    panels = [(512, 2048, 2048, 32), (672, 3208, 12960, 16), (4096, 13824, 5120, 64), (1024, 4096, 4096, 64)]
    direct = [(913, 6232, 6240, 16), (3748, 7888, 12720, 16), (1062, 7768, 8680, 16)]
    assert [p[0] for p in probe("int4", panels)] == [1] * 4
    assert [p[0] for p in probe("int4", direct)] == [0] * 3


def test_the_workspace_query_covers_lora_dropout(probe):
    """A masked product has a plan of its own (256 x 768 -> 768, fp32: dY W^T in six slices, [dY|Z1] [W^T;A^T] in five): the bytes that
    runlora_workspace_bytes names are enough with dropout too."""
    from paper_2312_03415_amd import binding as rl
    rng = np.random.default_rng(7)
    rows = [(256, 768, 768, 8), (512, 176, 5872, 24), (5653, 2216, 2720, 8)]
    rows += [(int(np.exp(rng.uniform(0, np.log(9000)))), int(rng.integers(8, 1000)) * 8, int(rng.integers(8, 1000)) * 8, int(rng.choice([8, 24, 64, 128]))) for _ in range(300)]
    for kind, code in (("drop32", rl.RL_F32), ("drop16", rl.RL_BF16)):
        for (n, i, o, r), need in zip(rows, probe(kind, rows)):
            assert rl.runlora_workspace_bytes(1, -1, n, i, o, r, code) >= need[0], (kind, n, i, o, r)
            assert rl.runlora_workspace_bytes(-1, 1, n, i, o, r, code) >= need[1], (kind, n, i, o, r)


def test_the_workspace_query_covers_every_call(probe):
    """Whatever a call keeps or leaves out, the bytes that runlora_workspace_bytes (runlora_vera_workspace_bytes) names for its variant are
    enough for the schedule it runs without a look at its workspace: Z1 alone of 4096 x 4096, r 256, takes more partials than Z1 and X A
    in one launch, and so does a product with r <= 128 whose pair is not split."""
    rng = np.random.default_rng(11)
    rows = [(4096, 4096, 4096, 256), (8192, 4096, 4096, 256), (8192, 2048, 2048, 256), (4096, 4096, 4096, 192), (6577, 2824, 8496, 72), (1032, 4104, 1096, 40)]
    dims = lambda: int(np.exp(rng.uniform(0, np.log(1200)))) * 8
    rows += [(int(np.exp(rng.uniform(0, np.log(9000)))), dims(), dims(), int(rng.choice([8, 24, 40, 64, 104, 128, 136, 192, 256, 264, 384]))) for _ in range(120)]
    for kind in ("calls16", "calls32", "calls4"):
        for row, (beyond, beyond_vera, inexact, first) in zip(rows, probe(kind, rows)):
            assert beyond == 0 and beyond_vera == 0, (kind, row, beyond, beyond_vera, first)
            assert inexact == 0, (kind, row, inexact)   # (runlora_call_workspace_bytes: the schedule of that call)


def test_a_call_runs_in_what_it_brings(probe):
    """Between the least workspace a layer runs in and the most it makes use of, its schedule takes no more than is there, and some of it:
    the rank-r products split their contraction as far as it goes, also next to an int4 W whose panels do not fit."""
    rng = np.random.default_rng(12)
    dims = lambda: int(np.exp(rng.uniform(np.log(8), np.log(1200)))) * 8
    rows = [(1024, 4096, 4096, 64), (1032, 4104, 1096, 40)]
    rows += [(int(np.exp(rng.uniform(0, np.log(9000)))), dims(), dims(), int(rng.choice([8, 40, 64, 128, 192, 256, 264]))) for _ in range(300)]
    for kind in ("fit16", "fit4"):
        got = probe(kind, rows)
        assert all(beyond == 0 for beyond, _ in got), [r for r, g in zip(rows, got) if g[0]]
        assert got[0][1] >= 12, got[0]   # (of nine amounts each way: T takes ten slices, Z1 and X A five each, and fewer than two are none)


def test_splits_of_T_fit_the_static_scratch(probe):
    """runlora_forward_static runs what runlora_forward runs: where its array holds T, it holds the partials that T is split into as well."""
    from paper_2312_03415_amd import binding as rl
    rng = np.random.default_rng(13)
    dims = lambda: int(np.exp(rng.uniform(0, np.log(1500)))) * 8
    rows = [(18292, 5640, 2520, 104), (21656, 9080, 8, 80), (24317, 3760, 3392, 80)]
    rows += [(int(np.exp(rng.uniform(0, np.log(40000)))), dims(), dims(), 8 * int(rng.integers(5, 64))) for _ in range(2000)]
    for row, (whole, least) in zip(rows, probe("static", rows)):
        assert whole <= rl.STATIC_SCRATCH_BYTES or least > rl.STATIC_SCRATCH_BYTES, (row, whole, least)


def test_masked_product_falls_back_where_the_workspace_is_that_of_two_launches(probe):
    """dX under LoRA dropout in one launch may split into more partials than dX = dY W^T and the masked update behind it: a call that brings
    what those take still runs."""
    rng = np.random.default_rng(14)
    dims = lambda: int(np.exp(rng.uniform(np.log(4), np.log(1200)))) * 8
    rows = [(492, 104, 9568, 48), (706, 1384, 1112, 128), (99, 168, 7856, 32)]
    rows += [(int(np.exp(rng.uniform(np.log(33), np.log(9000)))), dims(), dims(), int(rng.choice([8, 24, 48, 72, 128]))) for _ in range(600)]
    got = probe("masked", rows)
    for row, (one, two, need, steps) in zip(rows, got):
        assert need <= two, (row, one, two, need)
    assert all(one > two and steps == 4 for one, two, _, steps in got[:3]), got[:3]   # ({Z1, Z2}, {dA, dB}, dX, its update)


def test_slices_of_streaming_launches(probe):
    """T = X A, r <= 32: no more workgroups than compute units where it is split (16 bits), a masked product in no fewer slices than the same
    product without a mask, unless that one's slices leave compute units with two workgroups, and on 16 waves where it is whole and long:
    6795 x 10496 r 16 28.3 us, 33.1 on four; 3822 x 4928 r 32 in two slices 16.5 us on four, 18.5; 6262 x 2704 r 32 12.0 and 13.3."""
    rows = [(n, r, k) for n in (1, 5, 18, 64, 200, 700, 1240, 2048, 3232, 4096, 5000, 7000) for r in (8, 32) for k in (1536, 2048, 3744, 4096, 5464, 8192, 11008)]
    for kind in ("stream16", "stream32"):
        plain, masked = (probe(kind, [(*row, m) for row in rows]) for m in (0, 1))
        for (n, r, k), (s0, _, _), (s1, waves, _) in zip(rows, plain, masked):
            blocks = -(-n // 32)
            assert s1 == 1 or s1 * blocks <= 256, (n, r, k, s1)
            assert waves == (16 if s1 == 1 and -(-k // (64 if kind == "stream16" else 32)) >= 48 else 4), (kind, n, r, k, s1, waves)
            if kind == "stream16":
                assert s0 == 1 or s0 * blocks <= 256, (n, r, k, s0)
            assert s1 >= s0 or s0 * blocks > 256, (kind, n, r, k, s0, s1)
    assert [p[0] for p in probe("stream32", [(5, 16, 3744, 1)])] == [3]   # 20.9 us, 30.8 whole
    assert [p[0] for p in probe("stream16", [(5000, 16, 5464, 0), (3232, 16, 5840, 0), (2048, 16, 4096, 0)])] == [1, 2, 1]


def test_fp32_products_leave_the_plan_by_tile_counts_for_a_clear_gain(probe):
    """Modelled within 3 % of each other, 204 x 4008 x 4060 and 212 x 3284 x 1944 run 10-11 % faster on 128x128 tiles in a few slices;
    whole plans and those in many slices are left (52 x 344 x 5992 41 us, 46 on its plan by tile counts; 296 x 7496 x 32 17 and 20)."""
    kept = probe("f32", [(204, 4008, 4060, 0), (212, 3284, 1944, 0)])
    assert all(p[:2] == p[2:] for p in kept), kept
    assert all(p[:2] != p[2:] for p in probe("f32", [(256, 768, 768, 8), (300, 2000, 4000, 0), (52, 344, 5992, 192), (296, 7496, 32, 0), (2012, 240, 1044, 0), (233, 1304, 1552, 0)]))


def test_few_token_route_is_weighed_against_a_split_T(probe):
    """T = X A may split into more than the bytes that the few-token route takes, so the other route is priced with the splits it takes; a rank
    above the output's width decides nothing by itself.  us on the GPU, few-token / other: 67 x 2472 -> 72 r 96 11.2 / 19.8, 34 x 1200 -> 80 r 128
    12.4 / 17.8, 132 x 1272 -> 64 12.8 / 18.4, 77 x 1192 -> 64 12.5 / 19.0, 46 x 1328 -> 72 13.0 / 17.4; 35 x 5728 -> 8 30.5 / 21.6."""
    rows = [(67, 2472, 72, 96), (34, 1200, 80, 128), (132, 1272, 64, 128), (77, 1192, 64, 128), (46, 1328, 72, 128), (35, 5728, 8, 128)]
    got = probe("few", rows)
    assert [p[0] for p in got] == [1] * 5 + [0]
    assert all(splits > 0 and bool(few) == (us < other) for few, splits, us, other, _ in got), got


def test_gradient_pairs_of_few_bytes_stay_on_narrow_tiles(probe):
    """dA, dB, r > 64, over fewer than 44 MB of operands: 1480 x (5808 + 4920) r 72 12.5 us, 15.3 on 128x128 tiles; 8525 x (1144 + 960) r 80 19.8
    and 23.5; 4858 x (544 + 2640) r 128 16.8 and 19.2.  Above, as priced: 8192 x (4096 + 4096) r 128 41.6 on narrow tiles, 35.6."""
    small = [(1480, 5808, 4920, 72), (8525, 1144, 960, 80), (4858, 544, 2640, 128)]
    large = [(8192, 4096, 4096, 128), (8241, 7560, 376, 72), (8257, 1032, 2056, 72), (8193, 520, 3080, 128)]
    assert [p[0] for p in probe("pair", small + large)] == [0] * 3 + [1] * 4


def test_few_token_route_leaves_many_rows_of_large_layers(probe):
    """Every further 64 rows read W again and every 16 rows B: 245 x 4608 -> 9648 r 128 takes 74.2 us by the few-token route, 51.4 by T = X A
    and [X|T] [W;B], 256 x 10176 -> 7008 r 64 85.0 and 67.3, 170 x 7824 -> 10128 r 32 77.4 and 68.0; 93 x 2904 -> 8144 r 128 24.3 and 27."""
    large = [(245, 4608, 9648, 128), (256, 10176, 7008, 64), (170, 7824, 10128, 32), (256, 1752, 10152, 128)]
    assert [p[0] for p in probe("few", large)] == [0] * 4
    assert [p[0] for p in probe("few", [(93, 2904, 8144, 128), (32, 4096, 4096, 64), (64, 8192, 8192, 16)])] == [1] * 3


def test_masked_T_goes_to_tiles_where_they_are_faster(probe):
    """T = (X o m) A, r > 32.  us on the streaming kernel / on 128x64 tiles with their reduce: 1954 x 1280 r 64 10.5 / 12.3, 2582 x 2048 r 64 13.0 / 14.1,
    1713 x 1536 r 64 10.4 / 12.1, 3074 x 2304 r 48 13.0 / 13.9, 4628 x 1288 r 128 16.6 / 16.4 and a launch more; 700 x 3000 r 96 23.7 / 12.9, 1062 x 4864 r 128 25.6 / 15.6,
    5149 x 5120 r 40 34.8 / 19.3, 6568 x 640 r 128 14.5 / 11.9 (whole)."""
    stream = [(1954, 1280, 5760, 64), (2582, 2048, 768, 64), (1713, 1536, 9128, 64), (3074, 2304, 1792, 48), (4628, 1288, 2968, 128), (280, 2304, 768, 64)]
    tiles = [(700, 3000, 704, 96), (1062, 4864, 984, 128), (5149, 5120, 2816, 40), (6568, 640, 1280, 128)]
    assert [p[0] for p in probe("maskt", stream)] == [0] * 6
    assert [p[0] for p in probe("maskt", tiles)] == [1] * 4
