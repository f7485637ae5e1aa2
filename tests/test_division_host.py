"""div_by(a, b, 1 / b), the short 1-D run's quotient dt / dx, is IEEE division bit for
bit: random operands over many binades, divisors whose mantissas are all ones, powers
of two, small integers and their reciprocals (the cell sizes of real grids), dividends
close to multiples of them, zero.
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1210_5246_amd", "csrc")

SRC = r"""
#include "csh_device.h"
extern "C" void quotients(long n, const double* a, const double* b, double* out)
{
    for (long i = 0; i < n; ++i) out[i] = csh::div_by(a[i], b[i], 1.0 / b[i]);
}
"""
_D = ctypes.POINTER(ctypes.c_double)


@pytest.fixture(scope="module")
def quotients(tmp_path_factory):
    d = tmp_path_factory.mktemp("division")
    src, so = str(d / "c.hip"), str(d / "c.so")
    with open(src, "w") as f:
        f.write(SRC)
    subprocess.run(["/opt/rocm/bin/hipcc", "-O2", "-std=c++17", "-fPIC", "-shared", "--offload-arch=gfx950",
                    "-ffp-contract=off", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", CSRC, src,
                    "-o", so], check=True, capture_output=True)
    f = ctypes.CDLL(so).quotients
    f.argtypes = [ctypes.c_long, _D, _D, _D]

    def call(a, b):
        a, b = (np.ascontiguousarray(x, dtype=np.float64) for x in np.broadcast_arrays(a, b))
        out = np.empty(a.shape)
        f(a.size, *(x.ctypes.data_as(_D) for x in (a, b, out)))
        return out
    return call


def _check(quotients, a, b):
    np.testing.assert_array_equal(quotients(a, b), np.asarray(a) / np.asarray(b))


def test_random_operands(quotients):
    g = np.random.default_rng(1)
    for _ in range(4):
        a, b = (np.ldexp(1.0 + g.random(500000), g.integers(-60, 20, 500000)) for _ in range(2))
        _check(quotients, a, b)


def test_cell_sizes(quotients):
    g = np.random.default_rng(2)
    n = np.arange(1, 961, dtype=np.float64)
    for b in (1.0 / n, n, 0.7 / n):
        _check(quotients, np.exp(g.uniform(-40, 3, (400, n.size))), b)
        _check(quotients, 0.0, b)


def test_hard_mantissas(quotients):
    g = np.random.default_rng(3)
    u = 2.0 ** -52
    near = np.concatenate([2.0 - u * np.arange(1, 400), 1.0 + u * np.arange(400), 1.5 + u * np.arange(-200, 200)])
    _check(quotients, near[:, None], near[None, :])
    b = 1.0 + g.random(300000)
    # dividends next to the midpoints between two quotients
    m = (1.0 + g.integers(0, 2 ** 52, b.size) * u) * b
    for k in (-1, 0, 1):
        _check(quotients, m * (1.0 + u / 2) + k * np.spacing(m), b)
        _check(quotients, np.nextafter(m, np.inf if k > 0 else 0.0), b)
