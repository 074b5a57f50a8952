"""The FP64 integrands' normal CDF as csrc/cdf_table.hpp has it, compiled for the
host, against 40-digit values.  Absolute bound: a cell's F within one ulp below
1/2 (5.6e-17 and erf's own ulp), one rounding each of the series' last
multiply-add and of the final addition: 2.5e-16."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2005_10494_amd", "csrc")
mp = pytest.importorskip("mpmath")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("cdf")
    src, so = d / "t.cpp", d / "t.so"
    src.write_text("""#include "cdf_table.hpp"
using namespace bmd;
static CdfCell cells[kCdfCells];
extern "C" int cells_of(double* at) {
    for (int j = 0; j < kCdfCells; ++j) { cells[j] = cdf_cell(j); at[j] = static_cast<double>(j) / kCdfPerUnit; }
    return kCdfCells;
}
extern "C" void table(const double* x, double* out, int n) {
    for (int i = 0; i < n; ++i) out[i] = norm_cdf_table(x[i], cells);
}
""")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-shared", "-fPIC", "-D__host__=",
                           "-D__device__=", "-D__forceinline__=inline", "-I", CSRC, str(src), "-o", str(so)])
    return ctypes.CDLL(str(so))


def _cells(lib):
    at = np.zeros(4096)
    n = lib.cells_of(at.ctypes.data_as(ctypes.c_void_p))
    return at[:n]


def _eval(fn, x):
    x = np.ascontiguousarray(x, dtype=np.float64)
    out = np.empty_like(x)
    fn(x.ctypes.data_as(ctypes.c_void_p), out.ctypes.data_as(ctypes.c_void_p), len(x))
    return out


def _points(at):
    """Random ones, every cell's middle (where the neighbours meet) and both sides of it."""
    mid = 0.5 * (at[1:] + at[:-1])
    x = np.concatenate([np.random.default_rng(0).uniform(0, 9, 2000), at, mid, mid - 1e-9, mid + 1e-9, [8.5, 8.4999999]])
    return np.concatenate([x, -x])


def test_table_cdf_of_the_header(lib):
    mp.mp.dps = 40
    at = _cells(lib)
    assert at[0] == 0.0 and at[-1] == 8.5
    x = _points(at)
    got = _eval(lib.table, x)
    assert max(abs(mp.mpf(g) - mp.ncdf(mp.mpf(v))) for g, v in zip(got, x)) <= 2.5e-16
    far = np.array([1e6, 1e300, np.inf])
    assert np.all(_eval(lib.table, far) == 1.0) and np.all(_eval(lib.table, -far) == 0.0)
