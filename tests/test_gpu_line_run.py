"""Whole runs of short 1-D grids (one workgroup, one launch) against the oracle.

Sizes at the edges of the 60-cell wavefronts and of the path itself (960 cells;
961 takes a launch per step), all schemes, both boundary kinds, both types.
Tolerances as in test_gpu_parity: 1e-10 after up to 100 FP64 steps, timesteps
1e-11 (each follows from a state good to 1e-12 or so); FP32 5e-4 after 20 steps.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1210_5246_amd as csh
import workloads as wl
from parity import max_rel_error

pytestmark = pytest.mark.gpu


def _fields(n):
    W = np.tile(wl.periodic(64, 24).W[:, 3, :], (1, -(-n // 64)))[:, :n]
    return np.ascontiguousarray(W * (1.0 + 0.1 * np.sin(0.02 * np.arange(n))) if n > 64 else W)


@pytest.mark.parametrize("n", [1, 2, 3, 5, 59, 60, 61, 121, 256, 959, 960, 961])
@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("scheme", ["muscl", "hllc", "kt"])
def test_run_cfl(n, bc, scheme):
    W = _fields(n)
    og = oracle.Grid(n, 1, 1.0 / n, 1.0, bc, bc)
    steps = 25
    ref, dts = oracle.run_cfl(og, oracle.cons_field(W), nsteps=steps, cfl=0.8, scheme=scheme)
    print("line run", n, bc, scheme, flush=True)
    g = csh.Grid(torch.from_numpy(W).cuda(), 1.0 / n, 1.0, (bc, bc))
    g.set_scheme(scheme)
    U0 = g.U.clone()
    got = g.run_cfl(steps, 0.8)
    assert np.allclose(got.cpu().numpy(), dts, rtol=1e-11, atol=0)
    assert max_rel_error(g.U.cpu().numpy(), ref) <= 1e-10
    # the handle goes on as after single steps: rate, then a step from it
    s = oracle.max_signal_speed(og, ref)
    assert g.last_signal_speed() == pytest.approx(s, rel=1e-10)
    nxt, _ = oracle.run_cfl(og, ref, nsteps=1, cfl=0.8, scheme=scheme)
    out = g.step(0.8 / s)
    assert max_rel_error(out.cpu().numpy(), nxt) <= 1e-10
    assert g.last_signal_speed() == pytest.approx(oracle.max_signal_speed(og, nxt), rel=1e-10)
    # the recorded timesteps replay the run bit for bit, and so do the kept states
    V = U0.clone()
    g.run_dts(got, V)
    assert torch.equal(V, g.U)
    states, log = g.run_cfl_states(steps, 0.8, U0=U0)
    assert torch.equal(states[-1], g.U) and torch.equal(log, got)


@pytest.mark.parametrize("steps", [1, 2, 40])
def test_end_time(steps):
    """Clipped at t_end; the steps after it have dt = 0 and keep the state."""
    w = wl.sod(100)
    og = oracle.Grid(100, 1, 0.01, 1.0, 1, 1)
    U0 = oracle.cons_field(w.W)
    t_end = 0.03
    ref, dts = oracle.run_cfl(og, U0, nsteps=steps, cfl=0.8, t_end=t_end)
    g = csh.Grid(torch.from_numpy(w.W).cuda(), 0.01, 1.0, (1, 1))
    got = g.run_cfl(steps, 0.8, t_end).cpu().numpy()
    assert np.allclose(got[:len(dts)], dts, rtol=1e-9, atol=1e-14)
    assert (np.abs(got[len(dts):]) <= 1e-14).all()
    assert max_rel_error(g.U.cpu().numpy(), ref) <= 1e-10


def test_potential_fp32_and_flag():
    n = 130
    W = _fields(n)
    og = oracle.Grid(n, 1, 1.0 / n, 1.0, 1, 1, -0.5, 0.0, 0.6, 0.1)
    ref, dts = oracle.run_cfl(og, oracle.cons_field(W), nsteps=20, cfl=0.8)
    for dtype, tol in ((torch.float64, 1e-10), (torch.float32, 5e-4)):
        g = csh.Grid(torch.from_numpy(W).cuda().to(dtype), 1.0 / n, 1.0, (1, 1))
        g.set_potential(0.6, 0.1, -0.5)
        g.run_cfl(20, 0.8)
        assert max_rel_error(g.U.double().cpu().numpy(), ref) <= tol
    U = g.U.clone()
    U[0, 77] = -U[0, 77]
    g.run_cfl(2, 0.8, U=U)
    with pytest.raises(csh.NonPhysicalState):
        g.last_signal_speed()
