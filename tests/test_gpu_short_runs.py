"""Runs of a few steps, which are launched one by one on every grid, beside the longer
ones of the same handle, which small grids record: states, timesteps and the handle's
rate equal those of the kept-state run bit for bit, before and after a recorded run, and
a short run can be captured into the caller's own graph and replayed.
"""
import numpy as np
import pytest
import torch

import paper_1210_5246_amd as csh
import workloads as wl

pytestmark = pytest.mark.gpu


def _grid(shape, scheme):
    W = wl.periodic(64, 24).W
    if shape[0] == 1:
        W = np.tile(W[:, 3, :], (1, -(-shape[1] // 64)))[:, :shape[1]]
        W = W * (1.0 + 0.1 * np.sin(0.02 * np.arange(shape[1])))
    else:
        W = W[:, :shape[0], :shape[1]]
    g = csh.Grid(torch.from_numpy(np.ascontiguousarray(W)).cuda(), 1.0 / shape[1], 1.0 / shape[0], (1, 0))
    g.set_scheme(scheme)
    return g


@pytest.mark.parametrize("shape", [(20, 23), (64, 64), (1, 961), (1, 1500)])
@pytest.mark.parametrize("scheme", ["muscl", "kt"])
def test_runs_of_any_length(shape, scheme):
    print("short runs", shape, scheme, flush=True)
    g = _grid(shape, scheme)
    U0 = g.U.clone()
    states, dts = g.run_cfl_states(12, 0.4, U0=U0)
    rates = []
    for n in range(1, 13):
        g.run_cfl_states(n, 0.4, U0=U0)
        rates.append(g.last_signal_speed())
    for n in (1, 2, 3, 4, 5, 12, 1, 2, 3, 4, 12, 5):  # recorded and launched in turn
        U = U0.clone()
        log = g.run_cfl(n, 0.4, U=U)
        assert torch.equal(U, states[n - 1]) and torch.equal(log, dts[:n]), n
        assert g.last_signal_speed() == rates[n - 1]
        V = U0.clone()
        g.run_dts(dts[:n].clone(), V)
        assert torch.equal(V, U), n
    t_end = float(dts[:2].sum()) + 0.3 * float(dts[2])
    U = U0.clone()
    log = g.run_cfl(4, 0.4, t_end, U=U).cpu().numpy()
    assert log[3] == 0.0 and log.sum() == pytest.approx(t_end, rel=1e-14)


def test_a_short_run_in_the_callers_graph():
    print("short run captured", flush=True)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        g = _grid((64, 64), "muscl")
        U0, U, log = g.U.clone(), g.U, torch.empty(3, dtype=torch.float64, device="cuda")
        g.run_cfl(3, 0.4, dt_log=log)  # allocates the work buffer
        s.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            g.run_cfl(3, 0.4, dt_log=log)
        for k in range(4):
            U.copy_(U0 * (1.0 + 0.1 * k))
            log.zero_()
            graph.replay()
            s.synchronize()
            want, dts = g.run_cfl_states(3, 0.4, U0=U0 * (1.0 + 0.1 * k))
            s.synchronize()
            assert torch.equal(U, want[2]) and torch.equal(log, dts)
