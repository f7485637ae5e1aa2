"""Parity of the 2-D sweep at the edges of its work decomposition.

Small grids: a workgroup of four wavefronts stacked on one strip, with a flux
exchange between them (every count of rows that leaves wavefronts with none,
one, two or more rows, first and last segments ragged).  Larger ones: a
wavefront per segment.  One step against the oracle, <= 1e-12 per field as in
test_gpu_parity; the fluxes likewise.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1210_5246_amd as csh
import workloads as wl
from parity import max_rel_error

pytestmark = pytest.mark.gpu
TOL1 = 1e-12


def _workload(nx, ny, bc):
    w = wl.periodic(64, 31)
    reps = (1, -(-ny // 64), -(-nx // 64))
    w.W = np.ascontiguousarray(np.tile(w.W, reps)[:, :ny, :nx])
    # not the tile's own period: every strip and segment holds other values
    w.W[0] *= 1.0 + 0.2 * np.sin(np.arange(ny)[:, None] * 0.013 + np.arange(nx)[None, :] * 0.021)
    return w.W, 1.0 / nx, 1.3 / ny


def _check(nx, ny, bc, potential=False, scheme="muscl"):
    W, dx, dy = _workload(nx, ny, bc)
    pot = (0.7, 0.1, -0.5, -0.65) if potential else (0.0, 0.0, 0.0, 0.0)
    og = oracle.Grid(nx, ny, dx, dy, *bc, pot[2], pot[3], pot[0], pot[1])
    U0 = oracle.cons_field(W)
    dt = 0.8 / oracle.max_signal_speed(og, U0)
    solver = "hllc" if scheme == "hllc" else "hll"
    ref = oracle.step(og, dt, U0, solver)
    g = csh.Grid(torch.from_numpy(W).cuda(), dx, dy, bc)
    g.set_scheme(scheme)
    if potential:
        g.set_potential(*pot)
    print("sweep split", nx, ny, bc, scheme, flush=True)
    assert max_rel_error(g.step(dt).cpu().numpy(), ref) <= TOL1
    assert g.last_signal_speed() == pytest.approx(oracle.max_signal_speed(og, ref), rel=1e-13)
    Fx, Fy = g.fluxes(dt)
    ox, oy = oracle.fluxes(og, dt, U0, solver)
    for got, want in ((Fx, ox), (Fy, oy)):
        scale = np.abs(want).reshape(6, -1).max(axis=1)[:, None]
        d = np.abs(got.cpu().numpy() - want).reshape(6, -1)
        assert (d <= TOL1 * np.maximum(scale, np.abs(want).max() * 1e-3)).all()


@pytest.mark.parametrize("ny", [2, 3, 4, 5, 6, 7, 13])
@pytest.mark.parametrize("bc", [(0, 0), (1, 1)])
def test_stacked_segments(ny, bc):
    _check(61, ny, bc, potential=bc == (1, 1))


@pytest.mark.parametrize("rows", [1, 2, 3, 4, 6, 7, 9, 10, 23])
def test_stacked_segments_of_any_length(rows, monkeypatch):
    monkeypatch.setenv("CSH_ROWS", str(rows))
    _check(67, 23, (1, 0), potential=True, scheme="hllc" if rows % 2 else "muscl")


@pytest.mark.parametrize("nx,ny,bc", [(61, 17001, (0, 1)), (60, 40007, (1, 0))])
def test_wavefront_per_segment(nx, ny, bc):
    _check(nx, ny, bc, potential=True)


def test_wavefront_per_segment_short(monkeypatch):
    """Segments of two rows: every one of them a boundary of the row ring."""
    monkeypatch.setenv("CSH_ROWS", "2")
    _check(61, 17001, (0, 0))
