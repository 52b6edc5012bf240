"""Rules of the stencil's launch shapes, on the host: the library's own functions through a small
shared object (no device call)."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_0901_3163_amd")
SRC = r"""
#include "internal.hpp"
using namespace dl;
extern "C" {
int shape(const int* d, int v, int fp64) { return wilson_shape(make_lattice(d), v, fp64 != 0); }
int nbs(const int* d, int v) { return wilson_nbs(make_lattice(d), WilsonCfg{v, 0}); }
long grid(const int* d, int v, int fp64, int nrhs) { return wilson_grid(make_lattice(d), WilsonCfg{v, 0}, fp64 != 0, nrhs); }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    from paper_0901_3163_amd import deflan  # loads libdeflan.so
    cxx = shutil.which("g++")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    if cxx is None or not os.path.isdir(os.path.join(rocm, "include", "hip")):
        pytest.skip("no C++ compiler or HIP headers")
    d = tmp_path_factory.mktemp("shapes")
    (d / "shapes.cpp").write_text(SRC)
    so = d / "libshapes.so"
    subprocess.run([cxx, "-std=c++17", "-O1", "-w", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I",
                    os.path.join(rocm, "include"), "-I", os.path.join(PKG, "csrc"), str(d / "shapes.cpp"), "-o",
                    str(so), deflan.LIB_PATH, "-Wl,-rpath," + PKG], check=True)
    lib = ctypes.CDLL(str(so))
    lib.grid.restype = ctypes.c_long
    return lib


def dims4(*d):
    return (ctypes.c_int * 4)(*d)


BOXED = [(16, 16, 16, 32), (24, 24, 24, 48), (8, 8, 8, 8), (20, 20, 20, 40)]
NOBOX = [(3, 5, 7, 6), (26, 26, 26, 8)]  # no box of whole x rows fills half a block


@pytest.mark.parametrize("dims", BOXED + NOBOX)
@pytest.mark.parametrize("nrhs", [1, 2, 5, 64])
def test_grid_of_the_box_shapes(lib, dims, nrhs):
    """The blocks that the size check counts are the ones that are launched: FP64 has one right-hand
    side a block in every box shape, FP32 two in 24 to 26, the time-marching forms one."""
    d = dims4(*dims)
    for v in range(21, 27):
        pair = dims in BOXED and v >= 24
        assert lib.grid(d, v, 1, nrhs) == lib.nbs(d, v) * nrhs
        assert lib.grid(d, v, 0, nrhs) == lib.nbs(d, v) * ((nrhs + 1) // 2 if pair else nrhs)
        assert lib.shape(d, v, 0) == (v if dims in BOXED else 4 + (v - 21) % 3)
        assert lib.shape(d, v, 1) == ((21 if dims in BOXED else 4) + (v - 21) % 3)
