"""Build the HIP library libfdbb.so for gfx950 and the native half of its
Python binding, in-tree.

    python -m paper_1809_09851_amd.build

Each translation unit under csrc/ is compiled to an object in parallel, then
all are linked into ``paper_1809_09851_amd/libfdbb.so``; binding.cpp becomes
the extension module ``_binding.so`` next to it.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIBRARY = os.path.join(HERE, "libfdbb.so")
BINDING = os.path.join(HERE, "_binding.so")
ARCH = os.environ.get("FDBB_OFFLOAD_ARCH", "gfx950")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    f"--offload-arch={ARCH}",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-Wall",
    "-Wno-unused-function",
    # Packed FP32 instructions stay off: the compiler must not turn ordinary
    # float code into v_pk_* forms.
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    f"-I{os.path.join(HERE, os.pardir, 'include')}",
]

SOURCES = [
    "fdbb_api.hip",
    "kernels_pointwise.hip",
    "kernels_char.hip",
    "kernels_fused.hip",
    "kernels_adjoint.hip",
    "kernels_batch.hip",
    "kernels_batch_fused.hip",
    "kernels_eigen.hip",
    "probes.hip",
    "fdbb_server.cpp",
]


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    # host-only C++ (the server) goes through hipcc as HIP so it sees the
    # HIP runtime headers; it holds no kernels
    lang = ["-x", "hip"] if src.endswith(".cpp") else []
    cmd = [HIPCC, *FLAGS, *lang, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def build_binding() -> str:
    """binding.cpp, host code only, against the installed torch."""
    import torch
    from torch.utils import cpp_extension
    tmp = BINDING + ".tmp"
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-o", tmp, os.path.join(CSRC, "binding.cpp"),
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           f"-I{sysconfig.get_paths()['include']}"]
    cmd += [f"-I{p}" for p in cpp_extension.include_paths()]
    cmd += [f"-L{p}" for p in cpp_extension.library_paths()]
    cmd += ["-ltorch_python", "-ltorch_cpu", "-lc10"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed for binding.cpp:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, BINDING)
    return BINDING


def build(jobs: int | None = None, verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    jobs = jobs or min(len(SOURCES), max(1, (os.cpu_count() or 2)))
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        binding = ex.submit(build_binding)
        objs = list(ex.map(_compile, SOURCES))
        binding.result()
    tmp = LIBRARY + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIBRARY)
    if verbose:
        print(f"built {LIBRARY} and {BINDING}")
    return LIBRARY


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
