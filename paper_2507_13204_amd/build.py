"""Build libpgrad.so (the HIP kernels and the C ABI) for gfx950 with hipcc, and
_pgrad_torch.so (the autograd node, host code) with the C++ compiler.

Every .hip file under csrc/ is compiled to an object in parallel, then linked
into paper_2507_13204_amd/libpgrad.so next to this file; csrc/torch_node.cpp is
compiled beside them and linked against it and PyTorch.
"""
from __future__ import annotations

import concurrent.futures as cf
import glob
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(HERE, "libpgrad.so")
NODE = os.path.join(HERE, "_pgrad_torch.so")
ARCH = os.environ.get("PGRAD_ARCH", "gfx950")

HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

# Packed-FP32 instructions are disabled for all device code (the backend still
# vectorises FP32 code without them).
FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-munsafe-fp-atomics",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-I", os.path.join(ROOT, "include"),
]


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.basename(src) + ".o")
    cmd = [HIPCC, *FLAGS, "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def _compile_node() -> str:
    import sysconfig

    import torch
    from torch.utils import cpp_extension
    obj = os.path.join(BUILD, "torch_node.o")
    inc = cpp_extension.include_paths() + [sysconfig.get_paths()["include"], "/opt/rocm/include",
                                           os.path.join(ROOT, "include")]
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1",
           "-DUSE_ROCM=1", "-DTORCH_API_INCLUDE_EXTENSION_H", "-DTORCH_EXTENSION_NAME=_pgrad_torch",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           *[a for i in inc for a in ("-isystem", i)],
           "-c", os.path.join(CSRC, "torch_node.cpp"), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed for torch_node.cpp:\n{r.stdout}\n{r.stderr}")
    return obj


def _link_node(obj: str) -> None:
    from torch.utils import cpp_extension
    lib = cpp_extension.library_paths()[0]
    tmp = NODE + ".tmp"
    cmd = ["g++", "-shared", obj, f"-L{HERE}", "-l:libpgrad.so", f"-L{lib}", "-ltorch_python", "-ltorch_cpu", "-ltorch_hip",
           "-lc10", "-lc10_hip", "-Wl,-rpath,$ORIGIN", "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, NODE)


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    jobs = min(len(srcs) + 1, max(1, min(8, os.cpu_count() or 1)))
    with cf.ThreadPoolExecutor(jobs) as ex:
        node = ex.submit(_compile_node)
        objs = list(ex.map(_compile, srcs))
        node_obj = node.result()
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    _link_node(node_obj)
    if verbose:
        print(f"built {LIB} and {NODE}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
