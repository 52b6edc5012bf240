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
int candidates(const int* d, int fp64, int nrhs, int* out) {
  int n = 0;
  for (const WilsonCfg& c : wilson_candidates(make_lattice(d), fp64 != 0, nrhs)) {
    out[2 * n] = c.variant;
    out[2 * n++ + 1] = c.order;
  }
  return n;
}
int max_nbs(const int* d) { return wilson_max_nbs(make_lattice(d)); }
int stride(const int* d, int lo, int fp64) { return wilson_red_stride(make_lattice(d), WilsonCfg{lo, 0}, WilsonCfg{fp64, 0}); }
int residual(const int* d, int v) { return wilson_residual_shape(make_lattice(d), WilsonCfg{v, 0}); }
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


# variants of one kernel (and rhs per block) by rising chunk length
CHUNKS = [({4: 4, 5: 8, 6: 16}), ({7: 8, 8: 16}), ({12: 8, 13: 16}), ({18: 8, 19: 16}), ({21: 4, 22: 8, 23: 16}),
          ({24: 4, 25: 8, 26: 16})]
RHS = {7: 4, 8: 4, 9: 8, 10: 2, 15: 2, 16: 4, 17: 2, 24: 2, 25: 2, 26: 2}


@pytest.mark.parametrize("dims", BOXED + NOBOX + [(4, 4, 4, 4), (16, 16, 16, 5), (64, 64, 64, 16)])
@pytest.mark.parametrize("fp64", [0, 1])
@pytest.mark.parametrize("nrhs", [1, 2, 3, 64])
def test_tuner_times_every_launch_once(lib, dims, fp64, nrhs):
    """Each (variant, order) that the fused reductions can hold launches the same blocks as exactly one
    of the shapes that are timed: the same kernel, effective chunk and rhs group, in the same order."""
    d = dims4(*dims)
    buf = (ctypes.c_int * 256)()
    n = lib.candidates(d, fp64, nrhs, buf)
    cands = [(buf[2 * i], buf[2 * i + 1]) for i in range(n)]

    def launch(v, o):
        v = lib.shape(d, v, fp64)
        for fam in CHUNKS:
            if v in fam:  # the shortest chunk that covers t, if this one does
                v = min(w for w in fam if w == v or (fam[v] >= dims[3] and fam[w] >= dims[3]))
        return v, 0 if o == 1 and nrhs <= RHS.get(v, 1) else o

    want = {launch(v, o) for v in range(27) for o in range(3) if lib.nbs(d, v) <= 16384}
    assert len(set(cands)) == n and set(cands) == want


@pytest.mark.parametrize("dims", BOXED + NOBOX + [(64, 64, 64, 96)])
def test_residual_follows_the_tuned_stencil(lib, dims):
    """The FP64 residual runs in the FP64 stencil's tuned shape where that has a residual form, else with
    the shortest chunks, and never on more blocks than the reduction's partials hold."""
    d = dims4(*dims)
    box = dims in BOXED
    for v in range(27):
        s = lib.shape(d, v, 1)
        got = lib.residual(d, v)
        if s in (4, 5, 6) or s >= 21:
            assert got == s
        elif dims == (64, 64, 64, 96):  # links above 4 GB: no box; 16384 partials hold chunks of 8 slices
            assert got == 5
        else:
            assert got == (21 if box else 4)
        assert s == got or lib.nbs(d, got) <= 16384


@pytest.mark.parametrize("dims", BOXED + NOBOX + [(64, 64, 64, 4), (64, 64, 64, 16), (64, 64, 64, 96)])
def test_partials_per_right_hand_side(lib, dims):
    """A buffer that serves every shape holds the widest grid that a fused reduction takes (16384 partials,
    which one hop per wave passes above a million sites); a solve in chosen shapes needs only theirs."""
    d = dims4(*dims)
    fits = [lib.nbs(d, v) for v in range(27) if lib.nbs(d, v) <= 16384]
    assert lib.max_nbs(d) == max(fits) <= 16384
    for lo in range(27):
        for hi in range(27):
            assert lib.stride(d, lo, hi) == max(lib.nbs(d, lo), lib.nbs(d, lib.residual(d, hi)))
    if dims == (16, 16, 16, 32):
        assert lib.max_nbs(d) == 2048 and lib.stride(d, 26, 22) == 64
