"""Builds libheart.so (the C-ABI HIP library) in-tree with hipcc for gfx950, and the extension module
_native.so that calls it for binding.py."""
from __future__ import annotations

import os
import subprocess
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libheart.so")
NATIVE = os.path.join(PKG, "_native.so")
NATIVE_SOURCE = os.path.join(CSRC, "native_calls.cpp")
SOURCES = ["heart_api.hip", "pool_qk.hip", "drift.hip", "mask_topp.hip", "attn_plan.hip",
           "block_sparse_attn.hip", "ubench.hip", "ebc.hip", "antidiag_scores.hip"]

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-fno-gpu-rdc", "-Wall", "-Wno-unused-function",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def sources():
    return [os.path.join(CSRC, s) for s in SOURCES]


def is_built() -> bool:
    """Both the library and the extension module are there."""
    return os.path.exists(LIB) and os.path.exists(NATIVE)


def _torch_mark() -> str:
    # (the extension module is bound to the C++ ABI of the torch that it was compiled against)
    import torch

    return f"built for torch {torch.__version__}"


def is_stale() -> bool:
    if not is_built():
        return True
    t = min(os.path.getmtime(LIB), os.path.getmtime(NATIVE))
    deps = [os.path.join(d, f) for d in (CSRC, os.path.join(ROOT, "include")) for f in os.listdir(d)]
    if any(os.path.getmtime(d) > t for d in deps):
        return True
    with open(NATIVE, "rb") as f:
        return _torch_mark().encode() not in f.read()


def _run(cmd, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in res.stdout.splitlines()
                    if "is not a recognized feature for this target" not in l)
    if res.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed:\n" + out)
    if verbose and out.strip():
        print(out)


def build(force: bool = True, verbose: bool = False) -> str:
    """Compile every HIP source into libheart.so and the extension module.  Raises on failure."""
    if not force and not is_stale():
        return LIB
    from torch.utils.cpp_extension import include_paths, library_paths

    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    obj = NATIVE[:-3] + ".o"
    incs = [f"-isystem{p}" for p in include_paths() + [sysconfig.get_paths()["include"], os.path.join(ROOT, "include")]]
    with ThreadPoolExecutor(2) as ex:
        jobs = [ex.submit(_run, [hipcc] + HIPCC_FLAGS + ["-o", LIB] + sources(), verbose),
                # (NDEBUG: without it pybind11's headers leave a thread-local counter, and a library with thread-local
                # data that a thread never touches puts all its other thread-locals on glibc's slow path: every torch
                # operation took 0.4 us longer once the module was imported)
                ex.submit(_run, ["g++", "-O2", "-DNDEBUG", "-std=c++17", "-fPIC", "-Wall", f'-DHEART_TORCH="{_torch_mark()}"',
                                 *incs, "-c", NATIVE_SOURCE, "-o", obj], verbose)]
        for j in jobs:
            j.result()
    # (torch's libraries are loaded already when the module is imported)
    _run(["g++", "-shared", obj, "-L" + PKG, "-l:libheart.so", *[f"-L{p}" for p in library_paths()], "-ltorch_python",
          "-ltorch_cpu", "-lc10", "-Wl,-rpath,$ORIGIN", "-o", NATIVE], verbose)
    os.remove(obj)
    return LIB


if __name__ == "__main__":
    build(force=True, verbose=True)
    print(LIB)
