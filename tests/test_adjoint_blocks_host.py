"""The blocks of the device's 2-D reverse step, its own phases run on the CPU block by
block and thread by thread (tests/host/adjoint_host.hip), against the reverse step cell
by cell: both block widths (12 x 12 and 28 x 12 outputs), grids of one block and of one
more or less cell or row, thin grids, grids narrower than the ring, every pair of
boundary kinds, the potential on.  Both sides sum the same terms in another order:
1e-12 of the largest value.
"""
import ctypes

import numpy as np
import pytest

import oracle
import test_adjoint_host as th
import workloads as wl

SHAPES = [(1, 2), (2, 2), (3, 40), (40, 3), (11, 12), (12, 11), (12, 12), (12, 13), (13, 12), (24, 25), (25, 24),
          (27, 12), (28, 12), (28, 13), (29, 12), (56, 24), (57, 23), (61, 37)]
BOTH = [(0, 0), (1, 1), (0, 1), (1, 0)]


def _blocks(width, g, dt, U, lam):
    f = th.lib().host_adjoint_step_blocks
    f.argtypes = [ctypes.c_int] + th.lib().host_adjoint_step.argtypes
    out = np.full_like(U, np.nan)
    assert f(width, *th.geo(g), dt, g.vc, g.rc, g.x0, g.y0, th.p(U), th.p(lam), th.p(out)) == 0
    return out


def _case(nx, ny, bc, vc):
    W = np.ascontiguousarray(wl.periodic(64, 71).W[:, :ny, :nx])
    W[1:3] *= 2.0
    g = oracle.Grid(nx, ny, 1.0 / nx, 1.2 / ny, *bc, -0.4, -0.55, vc, 0.1)
    U = oracle.cons_field(W)
    return g, U, 0.8 / oracle.max_signal_speed(g, U), np.random.default_rng(nx + 100 * ny).standard_normal(U.shape)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("width", [16, 32])
def test_blocks_equal_the_cells(shape, width):
    for bc in BOTH:
        g, U, dt, lam = _case(*shape, bc, 0.8 if bc[0] or bc[1] else 0.0)
        ref = th.host_adjoint(g, dt, U, lam)
        assert np.abs(_blocks(width, g, dt, U, lam) - ref).max() <= 1e-12 * np.abs(ref).max(), bc


@pytest.mark.parametrize("width", [16, 32])
def test_a_nan_reaches_only_the_cells_of_its_stencil(width):
    """A NaN adjoint near each boundary, each corner and each edge of a block: the same
    cells are NaN as in the reverse step cell by cell, nothing else is touched."""
    nx, ny = 31, 27
    for bc in BOTH:
        g, U, dt, lam0 = _case(nx, ny, bc, 0.0)
        for j, i in ((10, 3), (10, nx - 4), (3, 12), (ny - 4, 12), (0, 0), (ny - 1, nx - 1), (12, 11), (11, 28), (24, 14)):
            lam = lam0.copy()
            lam[:, j, i] = np.nan
            ref, got = th.host_adjoint(g, dt, U, lam), _blocks(width, g, dt, U, lam)
            np.testing.assert_array_equal(np.isnan(got), np.isnan(ref))
