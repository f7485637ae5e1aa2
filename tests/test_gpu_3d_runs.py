"""The 3-D sweep on small grids, whose columns are cut into equal runs of planes.

One run per column, uneven runs, runs of one and two planes, and a grid past the
rule's line (equal shares that span columns).  One step against the oracle,
<= 1e-12 as in test_gpu_3d; the rate to 1e-13 checks that no cell is left out.
"""
import pytest

import oracle
import test_gpu_3d as t3

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(217, 185, 4), (61, 47, 33), (56, 60, 51), (5, 7, 300), (30, 13, 127), (100, 100, 40)])
@pytest.mark.parametrize("bc", [(0, 0, 0), (1, 0, 1)])
def test_runs_of_a_column(n, bc):
    W, g, h = t3.workload(n, 83, bc)
    U0 = oracle.cons3_field(W)
    dt = 0.8 / oracle.max_signal_speed3(g, U0)
    ref = oracle.step3(g, dt, U0)
    print("3d runs", n, bc, flush=True)
    G = t3.gpu(W, h, bc)
    assert t3.rel_err(G.step(dt).cpu().numpy(), ref) <= 1e-12
    assert G.last_signal_speed() == pytest.approx(oracle.max_signal_speed3(g, ref), rel=1e-13)
