"""The CFL rate's reduction: wavefront maxima, partial maxima per workgroup class, their combination.

One cell is made much faster than the rest; wherever it lies (lane of a
wavefront, wavefront, workgroup, part of the slot) the standalone rate, and the
rate fused into a step of a uniform state, must find it.  Tolerance: the rate is
a few products and one square root good to ~4e-15 each, 1e-13 relative.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1210_5246_amd as csh

pytestmark = pytest.mark.gpu


def _uniform(ny, nx):
    W = np.zeros((6, ny, nx))
    W[0], W[3], W[5], W[4] = 1.0, 1.0, 0.5, 0.1
    return W


@pytest.mark.parametrize("nx,ny", [(1, 1), (59, 1), (3000, 1), (64, 2), (121, 37), (700, 66)])
def test_hot_cell_found_wherever_it_lies(nx, ny):
    og = oracle.Grid(nx, ny, 1.0 / nx, 1.0 / ny, 0, 0)
    rng = np.random.Generator(np.random.PCG64(nx + ny))
    cells = {0, nx * ny - 1} | {int(c) for c in rng.integers(0, nx * ny, 24)}
    g = None
    for cell in sorted(cells):
        W = _uniform(ny, nx)
        j, i = divmod(cell, nx)
        W[1, j, i] = 7.0
        Wd = torch.from_numpy(W if ny > 1 else W[:, 0].copy()).cuda()
        if g is None:
            g = csh.Grid(Wd, 1.0 / nx, 1.0 / ny, (0, 0))
        else:
            g.set_state(Wd)
        s = oracle.max_signal_speed(og, oracle.cons_field(W))
        assert abs(g.max_signal_speed() - s) <= 1e-13 * s, cell
        # a step of dt = 0 leaves the state: the rate fused into it is the same
        g.step(0.0)
        assert abs(g.last_signal_speed() - s) <= 1e-13 * s, cell


def test_hot_cell_3d():
    n = (31, 14, 9)
    for cell in (0, 17, 31 * 14 * 4 + 31 * 7 + 29, 31 * 14 * 9 - 1):
        W = np.zeros((10, n[2], n[1], n[0]))
        W[0], W[4], W[7], W[9] = 1.0, 1.0, 0.5, 0.25
        W.reshape(10, -1)[2, cell] = 5.0
        og = oracle.Grid3(*n, 1.0 / n[0], 1.0 / n[1], 1.0 / n[2])
        s = oracle.max_signal_speed3(og, oracle.cons3_field(W))
        g = csh.Grid3(torch.from_numpy(W).cuda(), (1.0 / n[0], 1.0 / n[1], 1.0 / n[2]))
        assert abs(g.max_signal_speed() - s) <= 1e-13 * s, cell
        g.step(0.0)
        assert abs(g.last_signal_speed() - s) <= 1e-13 * s, cell
