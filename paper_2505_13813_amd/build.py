"""Builds libgrkan.so (HIP kernels + C ABI) in-tree for gfx950 with hipcc."""
from __future__ import annotations

import os
import shutil
import subprocess
from pathlib import Path

PKG = Path(__file__).resolve().parent
CSRC = PKG / "csrc"
LIB = PKG / "libgrkan.so"
SOURCES = [CSRC / "grkan_kernels.hip", CSRC / "grkan_plan.cpp", CSRC / "grkan_alg1_baseline.hip",
           CSRC / "grkan_linear.hip", CSRC / "grkan_linear_grad.hip", CSRC / "grkan_hidden.hip",
           CSRC / "grkan_product.hip", CSRC / "grkan_block.hip"]
HEADERS = [CSRC / "grkan_walk.h", CSRC / "grkan_plan.h", CSRC / "grkan_elem.h", CSRC / "grkan_tile.h", CSRC / "grkan_stage2.h",
           PKG.parent / "include" / "grkan.h",
           PKG.parent / "include" / "grkan_alg1.h"]

# the C++ autograd route of the PyTorch front end: host code only, over the C ABI of the library above
NATIVE = PKG / "_native.so"
NATIVE_SOURCES = [CSRC / "grkan_torch.cpp"]
NATIVE_HEADERS = [PKG.parent / "include" / "grkan.h"]

# packed-fp32 code generation is switched off on purpose (hipcc flag, device side)
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not Path(exe).exists():
        raise RuntimeError("hipcc not found; the GR-KAN library cannot be built")
    return exe


def is_stale() -> bool:
    if not LIB.exists():
        return True
    t = LIB.stat().st_mtime
    return any(p.stat().st_mtime > t for p in SOURCES + HEADERS)


def build_library(force: bool = True, verbose: bool = False) -> Path:
    """Compile the shared library.  `force=False` skips an up-to-date build."""
    if not force and not is_stale():
        return LIB
    tmp = LIB.with_name("libgrkan.so.tmp%d" % os.getpid())
    cmd = [hipcc(), *HIPCC_FLAGS, *map(str, SOURCES), "-o", str(tmp)]
    if verbose:
        print(" ".join(cmd))
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        tmp.unlink(missing_ok=True)
        raise RuntimeError("hipcc failed:\n" + res.stdout + res.stderr)
    os.replace(tmp, LIB)
    return LIB


def build_native(force: bool = True, verbose: bool = False) -> Path:
    """Compile the extension module (torch's headers, no device code).  libgrkan.so has to be there."""
    if not force and NATIVE.exists() and all(p.stat().st_mtime <= NATIVE.stat().st_mtime
                                             for p in NATIVE_SOURCES + NATIVE_HEADERS):
        return NATIVE
    import sysconfig

    import torch

    root = Path(torch.__file__).resolve().parent
    rocm = Path(hipcc()).resolve().parent.parent
    tmp = NATIVE.with_name("_native.so.tmp%d" % os.getpid())
    cmd = [shutil.which("g++") or "c++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           "-I%s" % (root / "include"), "-I%s" % (root / "include" / "torch" / "csrc" / "api" / "include"),
           "-I%s" % (rocm / "include"), "-I/opt/rocm/include", "-I%s" % sysconfig.get_paths()["include"],
           *map(str, NATIVE_SOURCES), "-o", str(tmp), "-L%s" % (root / "lib"), "-lc10", "-ltorch_cpu", "-ltorch",
           "-ltorch_python", "-lc10_hip", "-L%s" % PKG, "-l:libgrkan.so", "-Wl,-rpath,$ORIGIN"]
    if verbose:
        print(" ".join(cmd))
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        tmp.unlink(missing_ok=True)
        raise RuntimeError("g++ failed:\n" + res.stdout + res.stderr)
    os.replace(tmp, NATIVE)
    return NATIVE


if __name__ == "__main__":
    print(build_library(force=True, verbose=True))
    print(build_native(force=True, verbose=True))
