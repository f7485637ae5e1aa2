"""Where the sweeps' arithmetic rounds (the kernels' functions run on the CPU, against
the same formulas in extended precision).

The centre of a cell's face states, base - k A d, is a state less a small increment:
it rounds at the state's size once, so its error is that of rounding the exact result,
whatever the increment's own roundings (at a fiftieth of the size here) add: 1.1 times
it at most (two roundings at that size would give 1.41 times).

The CFL rate's roundings fall either way from state to state: over many states at
rest its mean error is a small part of a rounding, whatever the cell sizes (over
40000 states the mean of a few roundings scatters by 0.01 of one; a factor rounded
once per grid turns every rate, and so every timestep, by up to one).
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
#include "csh3_device.h"
using namespace csh;
template <int N>
static d3::V10 sub3(const double* b, double k, const double* w, const double* d)
{
    d3::V10 B, W, D;
    for (int m = 0; m < 10; ++m) B.v[m] = b[m], W.v[m] = w[m], D.v[m] = d[m];
    return d3::sub_jac<N>(B, k, W, rcp(w[0]), D);
}
// base - k A d along the axis, [n][6] or [n][10]
extern "C" void centres(int dim, int axis, int n, double k, const double* base, const double* W, const double* D,
                        double* out)
{
    for (int c = 0; c < n; ++c) {
        if (dim == 3) {
            const double *b = base + 10 * c, *w = W + 10 * c, *d = D + 10 * c;
            const d3::V10 o = axis == 0 ? sub3<0>(b, k, w, d) : axis == 1 ? sub3<1>(b, k, w, d) : sub3<2>(b, k, w, d);
            for (int m = 0; m < 10; ++m) out[10 * c + m] = o.v[m];
        } else {
            auto at = [&](const double* a) -> Prim<double> {
                a += 6 * c;
                return {a[0], a[1], a[2], a[3], a[4], a[5]};
            };
            const Prim<double> o = sub_jac_x(at(base), k, at(W), rcp(W[6 * c]), at(D));
            const double v[6] = {o.r, o.u, o.v, o.pxx, o.pxy, o.pyy};
            for (int m = 0; m < 6; ++m) out[6 * c + m] = v[m];
        }
    }
}
// CFL rates of [n][6] or [n][10] states
extern "C" void rates(int dim, int n, const double* ih, const double* W, double* out)
{
    for (int c = 0; c < n; ++c) {
        if (dim == 3) {
            d3::V10 w;
            for (int m = 0; m < 10; ++m) w.v[m] = W[10 * c + m];
            out[c] = d3::signal_rate(w, ih);
        } else {
            const double* a = W + 6 * c;
            const Prim<double> w = {a[0], a[1], a[2], a[3], a[4], a[5]};
            out[c] = dim == 2 ? signal_rate<double, true>(w, ih[0], ih[1]) : signal_rate<double, false>(w, ih[0], 0.0);
        }
    }
}
"""
_D = ctypes.POINTER(ctypes.c_double)


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("state_rounding")
    src, so = str(d / "c.hip"), str(d / "c.so")
    with open(src, "w") as f:
        f.write(SRC)
    subprocess.run(["/opt/rocm/bin/hipcc", "-O2", "-std=c++17", "-fPIC", "-shared", "--offload-arch=gfx950",
                    "-ffp-contract=off", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", CSRC, src,
                    "-o", so], check=True, capture_output=True)
    return ctypes.CDLL(so)


def p(a):
    assert a.dtype == np.float64 and a.flags.c_contiguous
    return a.ctypes.data_as(_D)


def tri(i, j, d):
    i, j = min(i, j), max(i, j)
    return 1 + d + i * d - i * (i - 1) // 2 + (j - i)


def states(g, n, d):
    """n random primitive states [n, 6 or 10], P = rho L L^T."""
    L = np.tril(g.uniform(-0.5, 0.5, (n, d, d)), -1) + np.eye(d) * g.uniform(0.3, 1.2, (n, 1, d))
    P = L @ L.transpose(0, 2, 1)
    rho = g.uniform(0.1, 2.0, (n, 1))
    return np.concatenate([rho, g.uniform(-1.0, 1.0, (n, d)), rho * np.stack(
        [P[:, i, j] for i in range(d) for j in range(i, d)], axis=1)], axis=1)


def jacobian_times(W, D, n, d):
    """A D along axis n, component by component."""
    w, x = W.T, D.T
    un, dn = w[1 + n], x[1 + n]
    out = [un * x[0] + w[0] * dn] + [un * x[1 + i] + x[tri(i, n, d)] / w[0] for i in range(d)]
    for i in range(d):
        for j in range(i, d):
            out.append(un * x[tri(i, j, d)] + w[tri(i, j, d)] * dn + w[tri(i, n, d)] * x[1 + j] +
                       w[tri(j, n, d)] * x[1 + i])
    return np.stack(out, axis=1)


@pytest.mark.parametrize("dim,axis", [(2, 0), (3, 0), (3, 1), (3, 2)])
def test_the_centre_rounds_once(lib, dim, axis):
    g, n, k = np.random.default_rng(10 * dim + axis), 20000, 0.37
    W, base = states(g, n, dim), states(g, n, dim)
    D = 0.02 * g.uniform(-1.0, 1.0, W.shape)
    out = np.empty_like(W)
    lib.centres(dim, axis, n, ctypes.c_double(k), p(base), p(W), p(D), p(out))
    ext = np.longdouble
    exact = base.astype(ext) - ext(k) * jacobian_times(W.astype(ext), D.astype(ext), axis, dim)
    off = np.sqrt(np.mean(((out - exact).astype(np.float64)) ** 2, axis=0))
    once = np.sqrt(np.mean((exact.astype(np.float64) - exact).astype(np.float64) ** 2, axis=0))
    print(off / once)
    assert (off <= 1.1 * once).all()


@pytest.mark.parametrize("dim", [1, 2, 3])
def test_the_rate_is_not_biased(lib, dim):
    d, n, ext = max(dim, 2), 40000, np.longdouble
    g = np.random.default_rng(70 + dim)
    for _ in range(12):
        ih = np.round(np.exp(g.uniform(np.log(30), np.log(5000), 3)))
        W = states(g, n, d)
        W[:, 1:1 + d] = 0.0
        out = np.empty(n)
        lib.rates(dim, n, p(ih), p(W), p(out))
        w = W.astype(ext)
        exact = sum(np.sqrt(3 * w[:, tri(k, k, d)] / w[:, 0]) * ext(ih[k]) for k in range(dim))
        bias = float(np.mean((out - exact) / exact)) * 2.0 ** 53
        assert abs(bias) <= 0.05, (ih[:dim], bias)
