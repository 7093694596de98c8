"""Build libhmy.so (the C-ABI library) in-tree with hipcc for gfx950."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libhmy.so")

SOURCES = ["model.cpp", "planner.cpp", "api.cpp", "engine.hip", "copy_engine.cpp", "elementwise.hip", "gemm.hip", "gemm_f32.hip", "attention.hip", "attention_f32.hip", "attention_mfma.hip", "gemm_tr.hip", "gemm_dma.hip", "gemm_tile.hip", "host_update.cpp"]

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-x", "hip",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-munsafe-fp-atomics", "-fno-math-errno", "-pthread", "-Wall", "-Wno-unused-function", "-Wno-unused-value",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


# plain host C++ (no device pass): the CPU-side update uses x86 target attributes
HOST_ONLY = {"host_update.cpp"}
HOST_FLAGS = ["-O3", "-std=c++17", "-fPIC", "-fno-math-errno", "-pthread", "-Wall",
              "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def _hostcxx() -> str:
    # hipcc would treat a .cpp as HIP and run a device pass over it
    cand = os.environ.get("HOSTCXX", "/opt/rocm/lib/llvm/bin/clang++")
    return cand if os.path.exists(cand) else "g++"


def _hipcc() -> str:
    return os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    if src in HOST_ONLY:
        cmd = [_hostcxx(), *HOST_FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    else:
        cmd = [_hipcc(), *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    msgs = "\n".join(l for l in (r.stdout + r.stderr).splitlines()
                     if "packed-fp32-ops" not in l)      # the host pass does not know the feature: harmless
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{msgs}")
    if msgs.strip():
        print(msgs, file=sys.stderr)
    return obj


def build(verbose: bool = True) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-pthread", "-o", LIB, *objs,
           "-L/opt/rocm/lib", "-lhsa-runtime64"]     # the runtime HIP itself runs on: copies on named copy engines
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout + r.stderr)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build()
