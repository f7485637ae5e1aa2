"""The CFL rate's fused validity test (checked_rate, 1-D, 2-D and 3-D) accepts
and rejects what physical() does, run on the CPU through a small harness: every
component set to zero, negative, tiny, huge, infinite and NaN values in states
that are otherwise positive-definite, and states on either side of each minor.
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
// out: per state physical and the checked test; W primitive, [n][m]
extern "C" void check(int dim, int n, const double* W, int* phys, int* chk)
{
    for (int k = 0; k < n; ++k) {
        bool bad = false;
        if (dim == 3) {
            d3::V10 w;
            for (int m = 0; m < 10; ++m) w.v[m] = W[10 * k + m];
            const double ih[3] = {3.0, 5.0, 7.0};
            d3::checked_rate(w, ih, bad);
            phys[k] = d3::physical(w);
        } else {
            const double* w = W + 6 * k;
            const Prim<double> p = {w[0], w[1], w[2], w[3], w[4], w[5]};
            const Cons<double> U = to_cons(p);
            if (dim == 2) checked_rate<double, true>(U, 3.0, 5.0, bad);
            else checked_rate<double, false>(U, 3.0, 0.0, bad);
            phys[k] = physical(to_prim(U));
        }
        chk[k] = !bad;
    }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("checked_rate")
    src, so = str(d / "c.hip"), str(d / "c.so")
    with open(src, "w") as f:
        f.write(SRC)
    subprocess.run(["/opt/rocm/bin/hipcc", "-O2", "-std=c++17", "-fPIC", "-shared", "--offload-arch=gfx950",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", CSRC, src, "-o", so],
                   check=True, capture_output=True)
    return ctypes.CDLL(so)


@pytest.mark.parametrize("dim", [1, 2, 3])
def test_same_verdict_as_physical(lib, dim):
    g = np.random.Generator(np.random.PCG64(dim))
    d = 3 if dim == 3 else 2
    m = 10 if dim == 3 else 6
    tri = [(i, j) for i in range(d) for j in range(i, d)]
    base = []
    for _ in range(200):
        L = np.tril(g.uniform(-0.5, 0.5, (d, d))) + np.diag(g.uniform(0.5, 1.0, d))
        P = L @ L.T
        base.append([g.uniform(0.1, 2.0), *g.normal(0, 1, d), *(P[i, j] for i, j in tri)])
    states = [list(b) for b in base]
    bads = [0.0, -0.0, -1.0, -1e-3, 1e-300, 1e300, np.inf, -np.inf, np.nan]
    for b in base[:40]:
        for f in range(m):
            for v in bads:
                if f in range(1, 1 + d) and abs(v) == 1e300:
                    continue  # overflows the conserved form, not a state
                s = list(b)
                s[f] = v
                states.append(s)
        for f, (i, j) in enumerate(tri):  # pairs of signs, and Pij^2 about Pii Pjj
            if i != j:
                lim = np.sqrt(b[1 + d + tri.index((i, i))] * b[1 + d + tri.index((j, j))])
                for v in (0.999, 1.001, -1.001):
                    s = list(b)
                    s[1 + d + f] = v * lim
                    states.append(s)
        s = list(b)
        s[0], s[1 + d] = -s[0], -s[1 + d]
        states.append(s)
        states.append([-x for x in b])
    W = np.ascontiguousarray(states)
    phys, chk = (np.zeros(len(W), np.int32) for _ in range(2))
    lib.check(dim, len(W), W.ctypes.data_as(ctypes.c_void_p), phys.ctypes.data_as(ctypes.c_void_p),
              chk.ctypes.data_as(ctypes.c_void_p))
    assert phys[:200].all() and 0.3 < 1 - phys.mean() < 0.99
    diff = np.nonzero(phys != chk)[0]
    assert not len(diff), (len(diff), W[diff[:5]], phys[diff[:5]])
