"""FP32 (and the Kurganov-Tadmor run of a short 1-D grid) in the work decompositions
that other tests take in FP64 or with one scheme only.

* 2-D Kurganov-Tadmor: the march of a wavefront per segment, which FP32 grids of more
  than three rounds of workgroups take, at segments shorter than its halo.
* 2-D sweep: the stacked segments of four wavefronts, which every FP32 grid takes, at
  ragged heights and narrow strips; both solvers, the fluxes too.
* Whole 1-D runs in one launch: every scheme in FP32, Kurganov-Tadmor with the potential
  and an end time in both types.

One FP32 step against the oracle on the rounded input: <= 2e-5 as in
test_gpu_kt_block (a few hundred roundings of 6e-8 in line); runs of 20 FP32 steps
5e-4 and FP64 runs 1e-10 as in test_gpu_line_run.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1210_5246_amd as csh
import workloads as wl
from parity import max_rel_error

pytestmark = pytest.mark.gpu
TOL1 = 2e-5


def _grid(nx, ny, bc, scheme, dtype=torch.float32):
    w = wl.periodic(64, 31)
    W = np.ascontiguousarray(np.tile(w.W, (1, -(-ny // 64), -(-nx // 64)))[:, :ny, :nx])
    # not the tile's own period: every strip and segment holds other values
    W[0] *= 1.0 + 0.2 * np.sin(np.arange(ny)[:, None] * 0.013 + np.arange(nx)[None, :] * 0.021)
    W = torch.from_numpy(W).to(dtype)
    dx, dy, pot = 1.0 / nx, 1.3 / ny, (0.7, 0.1, -0.5, -0.65)
    og = oracle.Grid(nx, ny, dx, dy, *bc, pot[2], pot[3], pot[0], pot[1])
    U0 = oracle.cons_field(np.ascontiguousarray(W.double().numpy()))
    g = csh.Grid(W.cuda(), dx, dy, bc)
    g.set_scheme(scheme)
    g.set_potential(*pot)
    return g, og, U0, 0.8 / oracle.max_signal_speed(og, U0)


@pytest.mark.parametrize("rows", [1, 2, 3, 5, 40])
@pytest.mark.parametrize("bc", [(0, 0), (1, 1), (0, 1)])
def test_kt_march(rows, bc, monkeypatch):
    monkeypatch.setenv("CSH_KT_ROWS", str(rows))
    g, og, U0, dt = _grid(127, 43, bc, "kt")
    print("fp32 kt march", rows, bc, flush=True)
    ref = oracle.step_kt(og, dt, U0)
    assert max_rel_error(g.step(dt).double().cpu().numpy(), ref) <= TOL1
    assert g.last_signal_speed() == pytest.approx(oracle.max_signal_speed(og, ref), rel=TOL1)


def _sweep(nx, ny, bc, scheme):
    g, og, U0, dt = _grid(nx, ny, bc, scheme)
    print("fp32 sweep", nx, ny, bc, scheme, flush=True)
    solver = "hllc" if scheme == "hllc" else "hll"
    ref = oracle.step(og, dt, U0, solver)
    assert max_rel_error(g.step(dt).double().cpu().numpy(), ref) <= TOL1
    assert g.last_signal_speed() == pytest.approx(oracle.max_signal_speed(og, ref), rel=TOL1)
    for got, want in zip(g.fluxes(dt), oracle.fluxes(og, dt, U0, solver)):
        scale = np.abs(want).reshape(6, -1).max(axis=1)[:, None]
        d = np.abs(got.double().cpu().numpy() - want).reshape(6, -1)
        assert (d <= TOL1 * np.maximum(scale, np.abs(want).max() * 1e-3)).all()


@pytest.mark.parametrize("nx,ny", [(61, 2), (61, 3), (61, 5), (61, 6), (61, 7), (61, 13), (1, 37), (2, 37), (59, 37),
                                   (60, 37), (121, 37), (61, 17001)])
@pytest.mark.parametrize("scheme", ["muscl", "hllc"])
def test_stacked_sweep(nx, ny, scheme):
    _sweep(nx, ny, (1, 0), scheme)


@pytest.mark.parametrize("rows", [1, 2, 3, 4, 6, 7, 9, 23])
def test_stacked_sweep_of_any_length(rows, monkeypatch):
    monkeypatch.setenv("CSH_ROWS", str(rows))
    _sweep(67, 23, (0, 1), "muscl")


@pytest.mark.parametrize("n", [2, 60, 61, 300, 960])
@pytest.mark.parametrize("scheme", ["muscl", "hllc", "kt"])
@pytest.mark.parametrize("dtype,tol", [(torch.float32, 5e-4), (torch.float64, 1e-10)])
def test_line_run(n, scheme, dtype, tol):
    W = np.tile(wl.periodic(64, 24).W[:, 3, :], (1, -(-n // 64)))[:, :n]
    W = torch.from_numpy(np.ascontiguousarray(W * (1.0 + 0.1 * np.sin(0.02 * np.arange(n))))).to(dtype)
    og = oracle.Grid(n, 1, 1.0 / n, 1.0, 1, 1, -0.5, 0.0, 0.6, 0.1)
    U0 = oracle.cons_field(np.ascontiguousarray(W.double().numpy()))
    t_end = 12.5 * 0.8 / oracle.max_signal_speed(og, U0)  # in the thirteenth of about twenty steps
    print("line run", n, scheme, dtype, flush=True)
    for end in (0.0, t_end):
        ref, dts = oracle.run_cfl(og, U0, nsteps=20, cfl=0.8, t_end=end or None, scheme=scheme)
        g = csh.Grid(W.cuda(), 1.0 / n, 1.0, (1, 1))
        g.set_scheme(scheme)
        g.set_potential(0.6, 0.1, -0.5)
        got = g.run_cfl(20, 0.8, end).cpu().numpy()
        assert max_rel_error(g.U.double().cpu().numpy(), ref) <= tol
        assert abs(got.sum() - np.sum(dts)) <= tol * np.sum(dts)
