"""Static checks of the matrix-core kernel's machine code (no GPU needed: hipcc cross-compiles).

The kernel's speed rests on three properties of its K loop that a harmless-looking source change can
silently break, with results staying correct: (1) no full wait for outstanding loads (`s_waitcnt
vmcnt(0)`) inside a K step, which would serialise the LDS ring; (2) no per-lane loop around a load (the
compiler wraps a load whose scalar offset it cannot prove uniform in a `s_cbranch_execnz` loop);
(3) no register spills.  Both the dense and the int4 route are checked, in the NN and NT layouts; the K-tile-64 kernel and
the middle-sized one, every build (also those with a masked segment or a column scale), by the same properties.  No kernel of the
file, whatever it is, spills vector registers.
"""
import os
import re
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2312_03415_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    out = tmp_path_factory.mktemp("isa") / "gemm_bf16.s"
    p = subprocess.run([HIPCC, *FLAGS, "-S", "--cuda-device-only", os.path.join(CSRC, "gemm_bf16.hip"), "-o", str(out)],
                       capture_output=True, text=True)
    assert p.returncode == 0, p.stderr[-2000:]
    return out.read_text()


def kernel_text(asm, al, bl, ns, bq, plain=0):
    name = f"_ZN2rl14gemm_mc_kernelIDF16bLi{al}ELi{bl}ELi{ns}ELb{bq}ELi{plain}EEEvNS_8GemmArgsE"
    start = asm.index("\n" + name + ":")
    return name, asm[start:asm.index("s_endpgm", start)]


def test_no_kernel_spills_vector_registers(asm):
    names = re.findall(r"\.name:           (\S+)", asm)
    spills = re.findall(r"\.vgpr_spill_count:\s+(\d+)", asm)
    assert len(names) == len(spills) > 100
    assert not [n for n, s in zip(names, spills) if s != "0"]


def blocks(text):
    cur, out = [], []
    for line in text.split("\n"):
        if re.match(r"^\.LBB\d+_\d+:", line):
            out.append(cur)
            cur = []
        elif line.startswith("\t") and not line.strip().startswith((";", ".")):
            cur.append(line.strip())
    out.append(cur)
    return out


@pytest.mark.parametrize("al,bl,ns,bq,plain", [(0, 0, 3, 0, 0), (0, 1, 3, 0, 0), (1, 0, 3, 0, 0), (0, 0, 3, 1, 0), (0, 1, 3, 1, 0),
                                                (0, 0, 3, 0, 1), (0, 1, 3, 0, 1), (1, 0, 3, 0, 1), (0, 1, 3, 0, 2), (0, 0, 3, 1, 1)])
def test_k_loop_of_the_matrix_core_kernel(asm, al, bl, ns, bq, plain):
    name, text = kernel_text(asm, al, bl, ns, bq, plain)
    meta = asm[asm.index(".name:           " + name):]
    meta = meta[:meta.index(".wavefront_size")]
    assert re.search(r"\.vgpr_spill_count:\s+0\b", meta), "the kernel spills vector registers"
    # the two K steps of a tile: straight-line runs of MFMAs (the cursor's rare-event branch may cut one in two)
    ksteps = [b for b in blocks(text) if sum(i.startswith("v_mfma") for i in b) >= 3]
    assert sum(sum(i.startswith("v_mfma") for i in b) for b in ksteps) >= 32, "expected the 32 MFMAs of a K tile in a few straight-line blocks"
    assert len(ksteps) <= 4 * (2 if bq else 1), "the K steps are cut into many blocks: branches between the MFMAs"
    for b in ksteps:
        first = next(k for k, i in enumerate(b) if i.startswith("v_mfma"))
        last = max(k for k, i in enumerate(b) if i.startswith("v_mfma"))
        body = b[first:last + 1]
        assert not any(re.match(r"s_waitcnt\s+vmcnt\(0\)", i) for i in body), "full load wait inside a K step"
        assert not any(i.startswith("scratch_") for i in body), "spill traffic inside a K step"
    for b in blocks(text):
        if b and b[-1].startswith("s_cbranch_execnz"):
            assert not any(i.startswith(("buffer_load", "global_load")) for i in b), "a load sits in a per-lane (waterfall) loop"


@pytest.mark.parametrize("al,bl,plain", [(0, 0, 1), (0, 1, 1), (1, 0, 1), (0, 0, 0), (0, 1, 0), (0, 1, 2), (0, 0, 2),
                                         (0, 1, "segmask"), (0, 0, "colscale 1"), (0, 0, "colscale 3")])
def test_k_loop_of_the_matrix_core_kernel_with_k_tile_64(asm, al, bl, plain):
    """gemm_mc64_kernel: a K tile is two straight-line K steps of 64 MFMAs (16x16x32) with tied accumulators and nothing
    between them but the fragment reads, the 16 refill loads and, in the second, one wait + barrier; no spills, no
    accumulator traffic between the two register files, no load in a per-lane loop."""
    if plain == "segmask":
        name = "_ZN2rl24gemm_mc64_segmask_kernelIDF16bEEvNS_8GemmArgsE"
    elif str(plain).startswith("colscale"):
        name = f"_ZN2rl25gemm_mc64_colscale_kernelIDF16bLi{plain[-1]}EEEvNS_8GemmArgsE"
    else:
        name = f"_ZN2rl16gemm_mc64_kernelIDF16bLi{al}ELi{bl}ELi{plain}EEEvNS_8GemmArgsE"
    start = asm.index("\n" + name + ":")
    text = asm[start:asm.index("s_endpgm", start)]
    meta = asm[asm.index(".name:           " + name):]
    meta = meta[:meta.index(".wavefront_size")]
    assert re.search(r"\.vgpr_spill_count:\s+0\b", meta), "the kernel spills vector registers"
    ksteps = [b for b in blocks(text) if sum(i.startswith("v_mfma_f32_16x16x32") for i in b) >= 64]
    assert len(ksteps) == 2, "expected the two K steps of a tile as two straight-line blocks of 64 MFMAs"
    syncs = 0
    for b in ksteps:
        first = next(k for k, i in enumerate(b) if i.startswith("v_mfma"))
        last = max(k for k, i in enumerate(b) if i.startswith("v_mfma"))
        body = b[first:last + 1]
        assert sum(i.startswith("v_mfma") for i in body) == 64
        assert not any(i.startswith(("scratch_", "v_accvgpr")) for i in body), "spill or accumulator copies inside a K step"
        for i in body:
            m = re.match(r"v_mfma_f32_16x16x32_\w+\s+(a\[\d+:\d+\]), \S+, \S+, (a\[\d+:\d+\])", i)
            if i.startswith("v_mfma"):
                assert m and m.group(1) == m.group(2), "accumulator not tied: " + i
        waits = [i for i in body if re.match(r"s_waitcnt\s+vmcnt\(0\)", i)]
        assert len(waits) <= 1
        syncs += len(waits)
        n_loads = sum(i.startswith("buffer_load") for i in body)
        assert n_loads in (0, 16)
        assert len(body) <= 64 + 90, "too many instructions between the MFMAs of a K step"
    assert syncs == 1, "exactly one of the two K steps waits for the loads"
    for b in blocks(text):
        if b and b[-1].startswith("s_cbranch_execnz"):
            assert not any(i.startswith(("buffer_load", "global_load")) for i in b), "a load sits in a per-lane (waterfall) loop"


MT_BUILDS = [(al, bl, bm, bn, ns, 0) for al, bl in ((0, 0), (0, 1), (1, 0)) for bm, bn, ns in ((128, 128, 2), (128, 128, 4), (256, 128, 3), (128, 64, 3), (64, 128, 3))]


@pytest.mark.parametrize("al,bl,bm,bn,ns,xa", MT_BUILDS + [(0, 0, 64, 128, 3, 1), ("pair", 1, 0, 0, 0, 0), ("pair", 0, 0, 0, 0, 0), ("wide", 1, 0, 0, 0, 0), ("wide", 0, 0, 0, 0, 0)]
                         + [(al, bl, bm, bn, ns, opt) for al, bl, bm, bn, ns, _ in MT_BUILDS for opt in ("segmask", "colscale") if (al, bl) == ((0, 1) if opt == "segmask" else (0, 0))])
def test_k_loop_of_the_middle_sized_kernel(asm, al, bl, bm, bn, ns, xa):
    """gemm_mt_kernel: a K tile's two K steps are one straight-line block (its hand-issued LDS reads are in flight across the whole
    of it: a branch would let the compiler copy what has not arrived) with all its products, one wait for loads that leaves
    the younger ring stages in flight, and nothing spilled or moved between the register files."""
    if al == "pair":   # (bl = 1: Z1 = dY B^T ; Z2 = X A, else dA = X^T Z1 ; dB = Z2^T dY)
        name = "_ZN2rl19gemm_mt_pair_kernelIDF16bLi0ELi1ELi0ELi128ELi64ELi128ELi64EEEvNS_8GemmArgsES1_" if bl else \
            "_ZN2rl19gemm_mt_pair_kernelIDF16bLi1ELi0ELi0ELi128ELi64ELi64ELi128EEEvNS_8GemmArgsES1_"
        bodies, bm, bn, ns = 2, 128, 64, 3
    elif al == "wide":   # (the same on 128x128 tiles)
        name = f"_ZN2rl19gemm_mt_pair_kernelIDF16bLi{1 - bl}ELi{bl}ELi0ELi128ELi128ELi128ELi128EEEvNS_8GemmArgsES1_"
        bodies, bm, bn, ns = 2, 128, 128, 3
    elif xa in ("segmask", "colscale"):
        name = f"_ZN2rl{15 + len(xa)}gemm_mt_{xa}_kernelIDF16bLi{al}ELi{bl}ELi{bm}ELi{bn}ELi{ns}EEEvNS_8GemmArgsE"
        bodies = 1
    else:
        name = f"_ZN2rl14gemm_mt_kernelIDF16bLi{al}ELi{bl}ELi{bm}ELi{bn}ELi{ns}ELb{xa}EEEvNS_8GemmArgsE"
        bodies = 1
    start = asm.index("\n" + name + ":")
    text = asm[start:asm.index(".Lfunc_end", start)]
    meta = asm[asm.index(".name:           " + name):]
    meta = meta[:meta.index(".wavefront_size")]
    assert re.search(r"\.vgpr_spill_count:\s+0\b", meta), "the kernel spills vector registers"
    per_tile = 2 * (bm // 32) * (bn // 32)           # products of a wave, both K steps
    loads = (bm + bn) * 128 // 4096                  # of a wave and K tile
    ksteps = [b for b in blocks(text) if any(i.startswith("v_mfma") for i in b)]
    assert len(ksteps) == bodies, "a K tile is cut into several blocks"
    for b in ksteps:
        at = [k for k, i in enumerate(b) if i.startswith("v_mfma")]
        assert len(at) == per_tile and all("16x16x32" in b[k] for k in at)
        body = b[at[0]:at[-1] + 1]
        assert not any(i.startswith(("scratch_", "v_accvgpr")) for i in body), "spill or accumulator copies inside a K step"
        waits = [i for i in body if re.match(r"s_waitcnt.*vmcnt", i)]
        assert len(waits) == 1 and f"vmcnt({(ns - 2) * loads})" in waits[0], waits
        assert sum(i.startswith("s_barrier") for i in body) == 1
        assert len(body) <= 2 * per_tile + 66, "too many instructions between the products of a K tile"
    for b in blocks(text):   # (a per-lane loop reads one lane's offset at a time)
        assert not (any(i.startswith("v_readfirstlane") for i in b) and any(i.startswith(("buffer_load", "global_load")) for i in b)), \
            "a load sits in a per-lane (waterfall) loop"
