"""The kernels' FP64 reciprocal, root and quotient on the CPU, from estimates
off by as much as the hardware's may be, against exact rationals: no less exact
than the division and the root they stand for."""
import ctypes
import os
import subprocess
from fractions import Fraction
from math import isqrt, ulp

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
OFF = [0.0, 2.0 ** -22, -2.0 ** -22, 2.0 ** -24, -1.3 * 2.0 ** -24]   # relative errors of the estimate


@pytest.fixture(scope="module")
def fp64(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("fp64") / "fp64.so")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.check_call([hipcc, "-std=c++17", "-O2", "-mfma", "-fPIC", "-shared", "--offload-host-only", "-o", out,
                           os.path.join(HERE, "fp64_host.hip")])
    L = ctypes.CDLL(out)
    for f in (L.rcp64_of, L.rsqrt64_of, L.div64_of):
        f.argtypes, f.restype = [ctypes.c_double] * 2, ctypes.c_double
    return L


def _numbers(n):
    rng = np.random.default_rng(6)
    return [float(v) for v in np.exp(rng.uniform(-4, 16, n))] + [1.0, 2.0, 3.0, 750.0, np.nextafter(2.0, 0)]


def _ulps(got, exact):
    return float(abs(Fraction(got) - exact) / Fraction(ulp(float(exact))))


@pytest.mark.parametrize("off", OFF)
def test_reciprocal(fp64, off):
    worst = max(_ulps(fp64.rcp64_of(x, (1.0 / x) * (1 + off)), 1 / Fraction(x)) for x in _numbers(4000))
    assert worst <= 0.5001   # a correctly rounded division: 0.5


@pytest.mark.parametrize("off", OFF)
def test_reciprocal_root(fp64, off):
    worst = 0.0
    for x in _numbers(2000):
        # 1 / sqrt(n / d) to 120 bits
        n, d = Fraction(x).numerator, Fraction(x).denominator
        exact = Fraction(isqrt((d << 400) // n), 1 << 200)
        worst = max(worst, _ulps(fp64.rsqrt64_of(x, x ** -0.5 * (1 + off)), exact))
    assert worst <= 1.25   # two correctly rounded operations: up to 1.5


def test_quotient(fp64):
    rng = np.random.default_rng(8)
    worst = 0.0
    for d in _numbers(4000):
        n = float(rng.uniform(-1000, 1000))
        worst = max(worst, _ulps(fp64.div64_of(n, d), Fraction(n) / Fraction(d)))
    assert worst <= 0.5001
