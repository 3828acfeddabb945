"""Compile the HIP sources under csrc/ into paper_2412_19829_amd/libgformer_attn.so (gfx950), and the host code under
host/ into the extension module _decode_call.so.  The library needs hipcc alone; the module needs g++ and torch's headers,
and is left out with a warning where there is no torch."""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import warnings
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ_DIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libgformer_attn.so")
CALL_SRC = os.path.join(HERE, "host", "decode_call.cpp")
CALL = os.path.join(HERE, "_decode_call.so")

# packed-fp32 VALU forms are kept off for every device compilation unit
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _newest_input() -> float:
    deps = sources() + glob.glob(os.path.join(CSRC, "*.hpp")) + \
        glob.glob(os.path.join(HERE, "..", "include", "*.h")) + [CALL_SRC]
    return max(os.path.getmtime(p) for p in deps)


def _compile(src: str, extra) -> str:
    obj = os.path.join(OBJ_DIR, os.path.basename(src) + ".o")
    cmd = ["hipcc", *HIPCC_FLAGS, *extra, "-c", src, "-o", obj]
    subprocess.run(cmd, check=True)
    return obj


def _build_call() -> None:
    import sysconfig
    try:
        import torch
        from torch.utils.cpp_extension import include_paths
    except ImportError as e:
        warnings.warn(f"{CALL} is not built: {e}")
        return
    libs = os.path.join(os.path.dirname(torch.__file__), "lib")
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
                    f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
                    *(f"-isystem{p}" for p in [*include_paths(), sysconfig.get_paths()["include"]]),
                    CALL_SRC, "-o", CALL, f"-L{libs}", "-ltorch_python", "-ltorch_cpu", "-lc10"], check=True)


def build(force: bool = True, extra_flags=(), verbose: bool = False) -> str:
    if not force and all(os.path.exists(x) and os.path.getmtime(x) >= _newest_input() for x in (LIB, CALL)):
        return LIB
    os.makedirs(OBJ_DIR, exist_ok=True)
    srcs = sources()
    with ThreadPoolExecutor(max_workers=min(8, len(srcs) + 1)) as ex:
        call = ex.submit(_build_call)
        objs = list(ex.map(lambda s: _compile(s, list(extra_flags)), srcs))
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    subprocess.run(cmd, check=True)
    call.result()   # last: the library does not wait for the module, nor for what it may lack
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(force=True, extra_flags=sys.argv[1:], verbose=True)
