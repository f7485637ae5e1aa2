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


def test_many_handles_keep_their_own_rate_and_flag():
    """More handles than a page of host cells holds, some freed in between."""
    W = torch.from_numpy(_uniform(4, 70)).cuda()
    grids = []
    for k in range(150):
        Wk = W.clone()
        Wk[1, 2, 3] = 2.0 + k
        grids.append((k, csh.Grid(Wk, 1.0 / 70, 0.25, (0, 0))))
        if k % 3 == 2:
            grids.pop(0)
    U = grids[5][1].U.clone()
    U[0, 1, 1] = -1.0
    grids[5][1].step(1e-5, U)
    s0 = None
    for n, (k, g) in enumerate(grids):
        if n == 5:
            with pytest.raises(csh.NonPhysicalState):
                g.last_signal_speed()
            continue
        s = g.max_signal_speed()
        s0 = s - 70.0 * k if s0 is None else s0
        assert abs(s - (s0 + 70.0 * k)) <= 1e-12 * s, k


@pytest.mark.parametrize("nx,ny", [(40, 30), (1200, 700)])
def test_log_buffer_and_replay(nx, ny):
    """A run repeated with other log buffers and lengths gives the same state and log
    (recorded steps on the small grid, plain launches on the large one)."""
    Wd = torch.from_numpy(_uniform(ny, nx)).cuda()
    Wd[1] += 0.1 * torch.sin(torch.arange(nx, device="cuda") * 0.1)
    g = csh.Grid(Wd, 1.0 / nx, 1.0 / ny, (0, 0))
    first = None
    for n in (7, 7, 3, 7, 12, 7):
        U = g.set_state(Wd)
        log = torch.full((n + 2,), -1.0, dtype=torch.float64, device="cuda")
        g.run_cfl(n, 0.8, dt_log=log)
        torch.cuda.synchronize()
        assert (log[:n] > 0).all() and (log[n:] == -1.0).all()
        if n == 7:
            if first is None:
                first = (U.clone(), log.clone())
            assert torch.equal(U, first[0]) and torch.equal(log, first[1])
        else:
            assert torch.equal(log[:3], first[1][:3])
