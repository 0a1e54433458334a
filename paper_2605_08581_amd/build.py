"""Build the HIP library for gfx950 in-tree (hipcc cross-compiles without a GPU)."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libprism.so")
BINDING = os.path.join(HERE, "_prism_torch.so")     # Python entry of the layer calls, against PyTorch's headers
SCHED_BINDING = os.path.join(HERE, "_prism_sched.so")  # Python entry of the control plane's per-request calls
SOURCES = ["prism_plan.cpp", "prism_api.cpp", "prism_sched.cpp", "prism_kernels.hip", "prism_attn64.hip", "prism_stream.hip"]
# packed fp32 VALU ops stay off: the kernels are written as ordinary float code
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-mllvm", "-amdgpu-mfma-vgpr-form",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    raise RuntimeError("hipcc not found")


def _compile(src: str, verbose: bool) -> str:
    obj_dir = os.path.join(HERE, "_build")
    os.makedirs(obj_dir, exist_ok=True)
    obj = os.path.join(obj_dir, os.path.splitext(src)[0] + ".o")
    cmd = [_hipcc()] + FLAGS + ["-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if verbose and err.strip():
        print(err, file=sys.stderr)
    return obj


def emit_assembly(src: str, out_dir: str) -> str:
    """Device-side assembly of one kernel source, with the flags of the build
    (for checks of what the compiler generated around the inline assembly)."""
    out = os.path.join(out_dir, os.path.splitext(src)[0] + ".s")
    cmd = [_hipcc()] + FLAGS + ["-x", "hip", "--cuda-device-only", "-S", os.path.join(CSRC, src), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc -S failed on {src}:\n{r.stderr}")
    return out


def _build_module(src: str, out: str, flags: list, libs: list) -> None:
    """A Python extension module of host code only."""
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", *flags, "-I", os.path.join(ROOT, "include"),
           "-isystem", sysconfig.get_paths()["include"], os.path.join(CSRC, src), "-o", out, *libs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed on {src}:\n" + r.stderr)


def _build_bindings() -> None:
    import torch
    base = os.path.dirname(torch.__file__)
    _build_module("prism_pysched.cpp", SCHED_BINDING, [], [])
    _build_module("prism_torch.cpp", BINDING,
                  ["-Wno-deprecated-declarations", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
                   f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
                   "-isystem", os.path.join(base, "include"), "-isystem", "/opt/rocm/include"],
                  ["-L", os.path.join(base, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10"])


def build(verbose: bool = False) -> str:
    """Compile every source, link libprism.so and the Python entries; always recompiles."""
    with ThreadPoolExecutor(max_workers=len(SOURCES) + 1) as ex:
        bindings = ex.submit(_build_bindings)
        objs = list(ex.map(lambda s: _compile(s, verbose), SOURCES))
        bindings.result()
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
