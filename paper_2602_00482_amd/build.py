"""Builds libdta.so (HIP kernels + C ABI) in-tree for gfx950 with hipcc, and dta_torch.so (its calls on torch
tensors, host code only) with the C++ compiler."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
LIB_PATH = os.path.join(PKG_DIR, "libdta.so")
PROBE_LIB_PATH = os.path.join(PKG_DIR, "libdta_probe.so")   # measurement kernels, not part of the product library
SOURCES = ["dta_tree.cpp", "dta_rollouts.cpp", "dta_plan.cpp", "dta_api.hip", "dta_f32_kernels.hip", "dta_f32_planes.hip", "dta_bf16_small.hip", "dta_bf16_fwd.hip", "dta_bf16_bwd.hip", "dta_noalloc.hip"]
PROBE_SOURCES = ["dta_probe.hip"]
TORCH_PATH = os.path.join(PKG_DIR, "dta_torch.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950", "-x", "hip",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(CSRC, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass warns that it does not know the packed-fp32 target feature; harmless
    err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    if verbose and err.strip():
        print(err, file=sys.stderr)
    return obj


def torch_stamp() -> str:
    """What dta_torch.so is built for; the module holds it."""
    import torch
    return f"torch {torch.__version__}, Python {sys.version_info.major}.{sys.version_info.minor}"


def _cxx():
    return shutil.which(os.environ.get("CXX", "g++"))


def build_torch() -> str:
    """Compile and link dta_torch.so (beside a built libdta.so)."""
    stamp = torch_stamp()
    import torch
    from torch.utils.cpp_extension import include_paths
    obj = os.path.join(CSRC, "dta_torch.o")
    inc = [f for d in include_paths("cuda") + [sysconfig.get_paths()["include"]] for f in ("-isystem", d)]
    cxx = _cxx() or "g++"
    cmd = [cxx, "-O2", "-std=c++17", "-fPIC", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DDTA_TORCH_BUILT_FOR="{stamp}"', *inc,
           "-I", os.path.join(ROOT, "include"), "-c", os.path.join(CSRC, "dta_torch.cpp"), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("compiling dta_torch.cpp failed:\n" + res.stderr)
    # libdta.so beside it; torch's own libraries are loaded by the `import torch` that comes first
    torch_lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = [cxx, "-shared", "-fPIC", obj, "-o", TORCH_PATH, "-L", PKG_DIR, "-l:libdta.so", "-Wl,-rpath,$ORIGIN",
           "-L", torch_lib, "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("linking dta_torch.so failed:\n" + res.stderr)
    return TORCH_PATH


def _can_build_torch() -> bool:
    if _cxx() is None:
        return False
    try:
        import torch  # noqa: F401
    except ImportError:
        return False
    return True


def build(verbose: bool = False) -> str:
    """Compile every source and link libdta.so, libdta_probe.so and, where torch and a C++ compiler
    are there, dta_torch.so; returns the path of libdta.so."""
    with ThreadPoolExecutor(max_workers=8) as pool:
        objs = list(pool.map(lambda s: _compile(s, verbose), SOURCES + PROBE_SOURCES))
    for out, group in ((LIB_PATH, objs[:len(SOURCES)]), (PROBE_LIB_PATH, objs[len(SOURCES):])):
        cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", *group, "-o", out]
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError("link failed:\n" + res.stderr)
    if _can_build_torch():
        build_torch()
    return LIB_PATH


def _sources():
    return [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith((".hip", ".cpp", ".h"))] + \
           [os.path.join(ROOT, "include", h) for h in ("dta.h", "dta_probe.h")]


def _stale() -> bool:
    """True when a source or header is newer than the built library (work-list
    records are shared between separately compiled host and device objects, so a
    half-rebuilt or outdated library must never be loaded)."""
    built = min(os.path.getmtime(LIB_PATH), os.path.getmtime(PROBE_LIB_PATH))
    return any(os.path.getmtime(d) > built for d in _sources() if os.path.basename(d) != "dta_torch.cpp")


def _torch_stale() -> bool:
    """True when dta_torch.so is missing, older than its source or built for another torch or Python."""
    if not os.path.exists(TORCH_PATH):
        return True
    built = os.path.getmtime(TORCH_PATH)
    if any(os.path.getmtime(d) > built
           for d in (os.path.join(CSRC, "dta_torch.cpp"), os.path.join(ROOT, "include", "dta.h"))):
        return True
    with open(TORCH_PATH, "rb") as f:
        return torch_stamp().encode() not in f.read()


def ensure_built() -> str:
    """Build what is not there or older than its sources (tests, the smoke run and the benchmark call this):
    everything with hipcc, or only dta_torch.so with the C++ compiler.  On a machine without the compilers what
    is there is used as it is; without dta_torch.so the Python wrappers make the calls."""
    if not all(os.path.exists(f) for f in (LIB_PATH, PROBE_LIB_PATH)):
        return build()
    if _stale() and os.path.exists(HIPCC):
        return build()
    if _can_build_torch() and _torch_stale():
        build_torch()
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose=True))
