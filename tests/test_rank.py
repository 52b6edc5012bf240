"""Ranks of the eigenvalue keys (csrc/rank.hpp), compiled for the host: the kernels of the projected
problems index with them, so they have to be a permutation whatever the keys are."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def rank_lib(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    d = tmp_path_factory.mktemp("rank")
    src = d / "rank.cpp"
    src.write_text('#include "rank.hpp"\n'
                   'extern "C" int asc(int n, const double* k, int i) { return dl::key_rank(n, k, i); }\n'
                   'extern "C" int mag(int n, const double* k, int i) { return dl::key_rank_abs(n, k, i); }\n')
    so = d / "librank.so"
    subprocess.run([cxx, "-std=c++17", "-O2", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_0901_3163_amd", "csrc"), str(src), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so))


def keys_of(n, seed, odd):
    g = np.random.default_rng(seed)
    k = g.standard_normal(n)
    for v in odd:  # each special value at a few places, ties among them
        k[g.integers(0, n, max(1, n // 4))] = v
    return np.ascontiguousarray(k)


@pytest.mark.parametrize("fn,name", [("asc", "value"), ("mag", "magnitude")])
@pytest.mark.parametrize("n", [1, 2, 7, 64, 142, 510])
@pytest.mark.parametrize("odd", [(), (0.0, -0.0), (1.5, -1.5), (np.nan,), (np.inf, -np.inf, np.nan), (np.nan, -np.nan, 0.0)])
def test_ranks_are_a_permutation(rank_lib, fn, name, n, odd):
    f = getattr(rank_lib, fn)
    for k in [keys_of(n, 10 * n + len(odd), odd), np.full(n, odd[-1] if odd else 1.0)]:
        r = [f(n, k.ctypes.data_as(ctypes.c_void_p), i) for i in range(n)]
        assert sorted(r) == list(range(n))
        at = np.argsort(r)
        num = [i for i in at if not np.isnan(k[i])]
        assert np.isnan(k[at[len(num):]]).all()  # NaN last
        want = sorted(num, key=lambda i: (abs(k[i]), k[i], i) if fn == "mag" else (k[i], i))
        assert num == want
