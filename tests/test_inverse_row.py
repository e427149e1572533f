"""The convolution rows of the 2D M1 solve (csrc/inverse_row.hpp, host code compiled here):
lengths that depend on the degree alone, whatever the cell width, and the inverse to rounding.

Tolerance: the entries are rounded to double (2^-53 of each) and the stencil times the row
adds sum |a| sum |c| of such errors at most; the cut entries are below that.
"""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest
from scipy.interpolate import BSpline

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2203_06513_amd", "csrc")
WRAP = """
#include "inverse_row.hpp"
extern "C" int row(int M, const double *mass, int n, double dx, double *out, int *hi) {
    const std::vector<double> r = ecpic2d::inverse_row(M, std::vector<double>(mass, mass + n), dx, *hi);
    for (size_t i = 0; i < r.size(); ++i) out[i] = r[i];
    return (int)r.size();
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("inverse_row")
    (d / "wrap.cpp").write_text(WRAP)
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "wrap.cpp"), "-o",
                    str(d / "row.so")], check=True)
    return C.CDLL(str(d / "row.so"))


def mass_row(d):
    b = BSpline.basis_element(np.arange(2 * d + 3), extrapolate=False)
    return b(np.arange(1.0, 2 * d + 2))


def row(lib, M, mass, dx):
    out, hi = np.zeros(M + 1), C.c_int(0)
    n = lib.row(M, C.c_void_p(mass.ctypes.data), len(mass), C.c_double(dx), C.c_void_p(out.ctypes.data), C.byref(hi))
    return out[:n], hi.value


@pytest.mark.parametrize("d,length", [(1, 65), (2, 101), (3, 135), (4, 169), (5, 205)])
@pytest.mark.parametrize("M", [8, 16, 64, 128, 256, 512])
def test_rows(lib, M, d, length):
    mass = mass_row(d)
    for dx in (1.0, 0.39269908169872414, 0.1, 1e-3, 7.3):
        r, hi = row(lib, M, mass, dx)
        assert len(r) == min(length, M)
        c = np.zeros(M)
        np.add.at(c, (hi - np.arange(len(r))) % M, r)
        a = np.zeros(M)
        np.add.at(a, np.arange(-d, d + 1) % M, dx * mass)
        prod = np.array([np.dot(a, c[(m - np.arange(M)) % M]) for m in range(M)])
        prod[0] -= 1.0
        # 4: the entries, the stencil, its product with dx and the sums here
        assert np.abs(prod).max() <= 4 * 2.0 ** -53 * np.abs(a).sum() * np.abs(c).sum()
