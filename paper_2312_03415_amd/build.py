"""Build librunlora.so (HIP for gfx950) and _autograd.so (the native autograd nodes, host code) in-tree:   python -m paper_2312_03415_amd.build [--force]

Objects go to paper_2312_03415_amd/_build/, the libraries to paper_2312_03415_amd/.
hipcc cross-compiles without a GPU.
"""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "librunlora.so")
EXT = os.path.join(HERE, "_autograd.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCES = ["gemm_bf16.hip", "gemm_f16.hip", "gemm_f32.hip", "gemm_host.hip", "schedule.cpp", "select.cpp", "api.hip", "probe.hip", "vera.hip", "dora.hip", "int4_panel.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-result",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _deps():
    return [os.path.join(CSRC, f) for f in os.listdir(CSRC)] + [os.path.join(HERE, "..", "include", "runlora.h")]


def _compile(src):
    obj = os.path.join(OBJ, src.rsplit(".", 1)[0] + ".o")
    cmd = [HIPCC, *FLAGS, "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
    p = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in p.stderr.splitlines() if "packed-fp32-ops" not in l)
    if p.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _ext_abi():
    """What _autograd.so is built against (it carries this text); it is rebuilt when one of them changes."""
    import torch
    return f"python {sys.implementation.cache_tag} torch {torch.__version__}"


def _ext_is_current():
    try:
        with open(EXT, "rb") as fh:
            return f"built for [{_ext_abi()}]".encode() in fh.read()
    except OSError:
        return False


def _compile_ext():
    """_autograd.so: a CPython extension against torch's headers; librunlora's entry points are handed to it at run time."""
    import sysconfig

    import torch
    root = os.path.dirname(torch.__file__)
    inc = os.path.join(root, "include")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", f'-DRL_BUILT_FOR="{_ext_abi()}"',
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), "-isystem", inc,
           "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"), "-isystem", "/opt/rocm/include",
           "-isystem", sysconfig.get_paths()["include"], os.path.join(CSRC, "autograd.cpp"), "-o", EXT,
           "-L" + os.path.join(root, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch", "-ltorch_python"]
    p = subprocess.run(cmd, capture_output=True, text=True)
    if p.returncode != 0:
        raise RuntimeError(f"g++ failed on autograd.cpp:\n{p.stderr}")


def build(force=False):
    if not force and _ext_is_current() and all(os.path.exists(f) and all(os.path.getmtime(f) >= os.path.getmtime(d) for d in _deps()) for f in (LIB, EXT)):
        return LIB
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES) + 1)) as ex:
        ext = ex.submit(_compile_ext)
        objs = list(ex.map(_compile, SOURCES))
        ext.result()
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs], check=True)
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv))
