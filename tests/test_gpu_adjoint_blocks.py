"""The 2-D reverse pass at the edges of its blocks (12 x 12 and 28 x 12 outputs)
against the CPU pass over the same per-cell bodies: grids of one block and one
more cell or row, thin grids, both block widths, every pair of boundary kinds,
the potential on.  Both sides sum the same terms in another order: 1e-12 of the
largest value, as in test_gpu_adjoint.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1210_5246_amd as csh
import test_adjoint_host as th
import workloads as wl

pytestmark = pytest.mark.gpu

SMALL = [(1, 2), (2, 3), (5, 2), (12, 12), (13, 12), (12, 13), (24, 25), (29, 23), (3, 40), (40, 3)]
# the smallest square that takes the wide blocks has 265 .. 276 cells a side
CASES = [(s, bc) for s in SMALL for bc in ((0, 0), (1, 1), (0, 1), (1, 0))]
CASES += [((276, 270), (1, 1)), ((275, 276), (0, 1)), ((281, 266), (1, 0)), ((276, 276), (0, 0))]


@pytest.mark.parametrize("shape,bc", CASES)
def test_blocks(shape, bc):
    nx, ny = shape
    n = max(64, nx, ny)
    W = np.ascontiguousarray(wl.periodic(n, 71).W[:, :ny, :nx])
    W[1:3] *= 2.0
    g = oracle.Grid(nx, ny, 1.0 / nx, 1.2 / ny, *bc, -0.4, -0.55, 0.8 if bc != (0, 0) else 0.0, 0.1)
    U = oracle.cons_field(W)
    dt = 0.8 / oracle.max_signal_speed(g, U)
    lam = np.random.default_rng(nx + ny).standard_normal(U.shape)
    ref = th.host_adjoint(g, dt, U, lam)
    print("adjoint blocks", shape, bc, flush=True)
    G = csh.Grid(torch.from_numpy(W).cuda(), g.dx, g.dy, bc)
    if g.vc:
        G.set_potential(g.vc, g.rc, g.x0, g.y0)
    got = G.adjoint_step(dt, torch.from_numpy(U).cuda(), torch.from_numpy(lam).cuda()).cpu().numpy()
    assert np.abs(got - ref).max() / np.abs(ref).max() < 1e-12


def test_a_nan_reaches_only_the_cells_of_its_stencil():
    """NaN adjoints three cells from each boundary of an outflow grid: the same cells
    are NaN as in the CPU pass, the boundary cells not among them."""
    nx, ny = 24, 20
    W = np.ascontiguousarray(wl.periodic(64, 72).W[:, :ny, :nx])
    g = oracle.Grid(nx, ny, 1.0 / nx, 1.2 / ny, 1, 1, 0.0, 0.0, 0.0, 0.0)
    U = oracle.cons_field(W)
    dt = 0.8 / oracle.max_signal_speed(g, U)
    for j, i in ((10, 3), (10, nx - 4), (3, 12), (ny - 4, 12)):
        lam = np.random.default_rng(i).standard_normal(U.shape)
        lam[:, j, i] = np.nan
        ref = th.host_adjoint(g, dt, U, lam)
        G = csh.Grid(torch.from_numpy(W).cuda(), g.dx, g.dy, (1, 1))
        got = G.adjoint_step(dt, torch.from_numpy(U).cuda(), torch.from_numpy(lam).cuda()).cpu().numpy()
        assert np.isfinite(ref[:, 10, [0, nx - 1]]).all() and np.isfinite(ref[:, [0, ny - 1], 12]).all()
        np.testing.assert_array_equal(np.isnan(got), np.isnan(ref))
