"""Host-side check of the places that a merge of the dense eigensolver gives to
its poles (csrc/poles.hpp, the code of the kernels compiled for the host).

The kernels fill index maps at these places and read the maps in full, so the
places of the n poles have to be a permutation of 0 .. n - 1.  They are for
every ascending finite input; a NaN takes the place of another pole, and is
shown by finite_magnitude before the merges run."""
import ctypes as ct
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2210_17093_amd", "csrc")
SRC = """
#include "poles.hpp"
extern "C" void places(const double* d, int n1, int n, int* out) {
  for (int t = 0; t < n; ++t) out[t] = qsgw::merged_place(d, n1, n, t);
}
extern "C" double magnitude(double x) { return qsgw::finite_magnitude(x); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    tmp = tmp_path_factory.mktemp("poles")
    src, out = tmp / "poles.cpp", tmp / "libpoles.so"
    src.write_text(SRC)
    subprocess.run([cxx, "-std=c++17", "-O2", "-shared", "-fPIC", "-I" + CSRC, str(src), "-o",
                    str(out)], check=True)
    lib = ct.CDLL(str(out))
    lib.magnitude.restype = ct.c_double
    lib.magnitude.argtypes = [ct.c_double]
    return lib


def places(lib, d, n1):
    d = np.ascontiguousarray(d, dtype=np.float64)
    out = np.empty(len(d), dtype=np.int32)
    lib.places(d.ctypes.data_as(ct.c_void_p), n1, len(d), out.ctypes.data_as(ct.c_void_p))
    return out


@pytest.mark.parametrize("n", [2, 3, 17, 64, 100, 3072])
@pytest.mark.parametrize("kind", ["spread", "ties", "equal", "zeros"])
def test_places_are_a_permutation(lib, n, kind):
    rng = np.random.default_rng(n)
    d = rng.standard_normal(n)
    if kind == "ties":
        d = np.round(d, 1)
    elif kind == "equal":
        d[:] = 2.5
    elif kind == "zeros":
        d[:] = np.where(rng.random(n) < 0.5, 0.0, -0.0)
    n1 = n // 2
    d[:n1].sort()
    d[n1:].sort()
    at = places(lib, d, n1)
    assert sorted(at) == list(range(n))
    merged = np.empty(n)
    merged[at] = d
    assert np.all(np.diff(merged) >= 0)


def test_a_nan_takes_another_place_and_shows(lib):
    """Why the kernels replace a tridiagonal matrix that is not finite."""
    at = places(lib, np.full(100, np.nan), 50)
    assert 0 <= at.min() and at.max() < 100 and len(set(at)) == 50
    for x in (np.nan, -np.nan, np.inf, -np.inf):
        assert lib.magnitude(x) == np.inf
    for x in (0.0, -0.0, -2.5, 5e-324, 1.7e308):
        assert lib.magnitude(x) == abs(x)
