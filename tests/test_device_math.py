"""The device's own FP64 functions that are plain IEEE arithmetic, compiled for the
host from the same source text and compared with 80-bit values."""
import ctypes
import os
import re
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def exp_le0(tmp_path_factory):
    """(x[n]) -> exp_le0(x) and expl(x) rounded to 80 bits minus it, in units in the last place."""
    with open(os.path.join(ROOT, "paper_2010_08454_amd", "csrc", "device.h")) as f:
        body = re.search(r"double exp_le0\(double x\) \{.*?\n\}\n", f.read(), re.S).group(0)
    d = tmp_path_factory.mktemp("device_math")
    src, lib = d / "exp.cpp", d / "libexp.so"
    src.write_text("#include <cmath>\nusing std::fma;\nstatic " + body + """
extern "C" void run(const double *x, long n, double *y, double *err) {
    for (long i = 0; i < n; ++i) {
        y[i] = exp_le0(x[i]);
        const long double ref = expl((long double)x[i]);
        int e;
        frexpl(ref, &e);
        const long double ulp = ldexpl(1.0L, (e < -1021 ? -1021 : e) - 53);
        err[i] = (double)(((long double)y[i] - ref) / ulp);
    }
}
""")
    subprocess.run(["g++", "-O2", "-mfma", "-ffp-contract=off", "-shared", "-fPIC", "-o", str(lib), str(src)], check=True)
    run = ctypes.CDLL(str(lib)).run
    P = ctypes.POINTER(ctypes.c_double)

    def call(x):
        x = np.ascontiguousarray(x, np.float64)
        y, err = np.empty_like(x), np.empty_like(x)
        run(x.ctypes.data_as(P), ctypes.c_long(x.size), y.ctypes.data_as(P), err.ctypes.data_as(P))
        return y, err
    return call


def test_exp_le0_error(exp_le0):
    """In units in the last place of a result in [1/sqrt 2, 1) 2^k (above 1 a unit is
    twice that): the last sum rounds by 1/2, the one before, of size 0.35 at most, by
    1/4, and the square, the polynomial, its product (at most 0.06 in all) and the
    carried error of the reduction by less than 1/6 together."""
    g = np.random.default_rng(0)
    half = (np.arange(-1074, 0) + 0.5) * np.log(2.0)           # where the reduction changes k
    near = np.concatenate([np.nextafter(half, -np.inf), half, np.nextafter(half, np.inf)])
    x = np.concatenate([g.uniform(-708.0, 0.0, 2_000_000), -10.0 ** g.uniform(-320, 2.85, 500_000), near[near > -708.0]])
    y, err = exp_le0(x)
    assert np.max(np.abs(err)) < 0.92
    assert np.max(y) <= 1.0 and np.min(y) > 0.0


def test_exp_le0_ends(exp_le0):
    """1 at both zeros and at arguments that round to it, subnormal results within a
    unit of their own, zero below them, and NaN kept."""
    y, _ = exp_le0([0.0, -0.0, -1e-300, -1e-17, 1e-17, -np.inf, -800.0, -746.0, np.nan])
    np.testing.assert_array_equal(y, [1.0, 1.0, 1.0, 1.0, 1.0, 0.0, 0.0, 0.0, np.nan])
    y, err = exp_le0(np.linspace(-745.0, -708.0, 200_001))
    assert np.max(np.abs(err)) <= 1.5 and np.all(y >= 0.0)
