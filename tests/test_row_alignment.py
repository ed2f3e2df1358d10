"""The wide accesses to rows and blocks in global memory are compiled for
pointers that are aligned to one value only, as packed and offset rows are:
the compiler's own intermediate code of the tile functions states the
alignment that each access relies on."""
import os
import re
import subprocess

import pytest

from paper_1809_09851_amd import build

SOURCE = """
#include "euler_tiles.hpp"
using namespace fdbb;
template <typename T, int P, int NT>
__global__ void rows(Args a) { tile_adjoint<1, T, P, NT>(a, (int64_t)blockIdx.x * blockDim.x * P); }
template <typename T, int P, int NT>
__global__ void blocks(Args a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    tile_fused<1, T, P, NT>(a, (int64_t)blockIdx.x * blockDim.x * P, ~0u, reinterpret_cast<T *>(smem));
}
template __global__ void rows<double, 2, kStoreRegular>(Args);
template __global__ void rows<float, 2, kStoreNT>(Args);
template __global__ void rows<float, 4, kStoreRegular>(Args);
template __global__ void blocks<double, 1, kStoreNT>(Args);
template __global__ void blocks<float, 4, kStoreRegular>(Args);
"""
ACCESS = re.compile(r"\b(load|store) <(\d+) x (double|float)>.*?ptr( addrspace\(\d+\))? .*?, align (\d+)")


@pytest.fixture(scope="module")
def accesses(tmp_path_factory):
    d = tmp_path_factory.mktemp("ir")
    src, out = os.path.join(d, "rows.hip"), os.path.join(d, "rows.ll")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", "-emit-llvm", f"-I{build.CSRC}", src, "-o", out],
                   check=True, capture_output=True)
    return [(m[0], int(m[1]), m[2], m[3].strip(), int(m[4])) for m in ACCESS.findall(open(out).read())]


def test_global_accesses_ask_for_one_values_alignment(accesses):
    kinds = set()
    for what, width, value, space, align in accesses:
        if space == "addrspace(3)":
            continue
        assert align == (8 if value == "double" else 4), (what, width, value, align)
        kinds.add((what, width, value))
    assert kinds >= {("load", 2, "double"), ("load", 2, "float"), ("load", 4, "float"),
                     ("store", 2, "double"), ("store", 2, "float"), ("store", 4, "float")}


def test_staged_runs_are_read_whole(accesses):
    """Blocks leave LDS in 16-byte reads: every staged run starts on 16 bytes."""
    assert {a for a in accesses if a[3] == "addrspace(3)" and a[0] == "load"} >= {
        ("load", 2, "double", "addrspace(3)", 16), ("load", 4, "float", "addrspace(3)", 16)}
