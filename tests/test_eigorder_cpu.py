"""The order of eigenvalues (csrc/eigorder.h): counting the places before each one is a
permutation whatever the diagonal holds, ascending with NaN last -- the kernels of
csrc/jacobi.h use it as an index."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2604_27451_amd", "csrc")
SHIM = r'''
#include "eigorder.h"
extern "C" void rank(int n, const double* v, int* perm) {
  for (int i = 0; i < n; ++i) {
    int r = 0;
    for (int j = 0; j < n; ++j) r += adc2::eig_before(v[j], j, v[i], i) ? 1 : 0;
    perm[r] = i;
  }
}
'''


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("eigorder")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run([gxx, "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "shim.cpp"), "-o",
                    str(d / "lib.so")], check=True)
    return ctypes.CDLL(str(d / "lib.so"))


NAN, INF = float("nan"), float("inf")


@pytest.mark.parametrize("v", [[NAN], [1.0, NAN], [NAN, 1.0], [NAN] * 5, [3.0, NAN, -1.0, NAN, -1.0],
                               [INF, NAN, -INF, INF], [0.0, -0.0, 0.0], [2.0] * 64,
                               list(np.where(np.arange(64) % 7, np.sin(np.arange(64)), NAN))])
def test_a_permutation_ascending_nan_last(lib, v):
    v = np.array(v)
    perm = np.full(len(v), -1, np.int32)
    lib.rank(len(v), v.ctypes.data_as(ctypes.c_void_p), perm.ctypes.data_as(ctypes.c_void_p))
    assert sorted(perm) == list(range(len(v)))
    assert np.array_equal(v[perm], np.sort(v, kind="stable"), equal_nan=True)
    same = np.nonzero(np.diff(v[perm]) == 0)[0]
    assert np.all(perm[same] < perm[same + 1])
