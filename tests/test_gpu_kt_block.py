"""Parity of the 2-D Kurganov-Tadmor step of a workgroup per segment.

Grids up to one round of workgroups (FP64) or a few (FP32): eight wavefronts
share the rows of a segment in both stages.  Segment heights from one row (most
wavefronts idle) to the tallest, ragged last segments, strips narrower than the
halo and grids shorter than it.  One step against the oracle: <= 1e-12 per
field as in test_gpu_kt; FP32 <= 2e-5 (inputs rounded at 6e-8, ~300 roundings
of that size per cell at most in line).
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1210_5246_amd as csh
import workloads as wl
from parity import max_rel_error

pytestmark = pytest.mark.gpu


def _check(nx, ny, bc, potential=False, dtype=torch.float64, tol=1e-12):
    w = wl.periodic(64, 32)
    W = np.ascontiguousarray(np.tile(w.W, (1, -(-ny // 64), -(-nx // 64)))[:, :ny, :nx])
    # not the tile's own period: every strip and segment holds other values
    W[0] *= 1.0 + 0.2 * np.sin(np.arange(ny)[:, None] * 0.013 + np.arange(nx)[None, :] * 0.021)
    W = W.astype(np.float32 if dtype is torch.float32 else np.float64).astype(np.float64)
    dx, dy = 1.0 / nx, 1.3 / ny
    pot = (0.7, 0.1, -0.5, -0.65) if potential else (0.0, 0.0, 0.0, 0.0)
    og = oracle.Grid(nx, ny, dx, dy, *bc, pot[2], pot[3], pot[0], pot[1])
    U0 = oracle.cons_field(W)
    dt = 0.8 / oracle.max_signal_speed(og, U0)
    ref = oracle.step_kt(og, dt, U0)
    g = csh.Grid(torch.from_numpy(W).to("cuda", dtype), dx, dy, bc)
    g.set_scheme("kt")
    if potential:
        g.set_potential(*pot)
    print("kt block", nx, ny, bc, dtype, flush=True)
    assert max_rel_error(g.step(dt).double().cpu().numpy(), ref) <= tol
    rate = 1e-13 if dtype is torch.float64 else tol
    assert g.last_signal_speed() == pytest.approx(oracle.max_signal_speed(og, ref), rel=rate)


@pytest.mark.parametrize("ny", [2, 3, 4, 5, 8, 11, 12, 13, 29])
@pytest.mark.parametrize("bc", [(0, 0), (1, 1)])
def test_short_grids(ny, bc):
    _check(57, ny, bc, potential=bc == (1, 1))


@pytest.mark.parametrize("nx", [1, 2, 3, 55, 56, 112, 113])
@pytest.mark.parametrize("bc", [(0, 1), (1, 0)])
def test_narrow_grids(nx, bc):
    _check(nx, 37, bc)


# rows per segment 4 .. 52: one share of 1 .. 7 rows each, even and uneven
@pytest.mark.parametrize("nx,ny", [(300, 200), (500, 300), (512, 512), (900, 500), (100, 4001), (1000, 700)])
def test_tall_segments(nx, ny):
    _check(nx, ny, (1, 1), potential=True)
    _check(nx, ny, (0, 0))


@pytest.mark.parametrize("nx,ny", [(113, 33), (900, 900), (1400, 1400)])
def test_fp32_one_or_two_workgroups_on_a_cu(nx, ny):
    _check(nx, ny, (0, 1), dtype=torch.float32, tol=2e-5)
