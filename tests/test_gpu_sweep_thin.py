"""The 2-D sweep and its fluxes on wide grids of few rows, at the edges of the rule that
gives each of their strips a wavefront of its own (more than 512 strips of 60 columns,
at most eight rows): parity with the oracle as in test_gpu_sweep_split, FP32 as in
test_gpu_fp32_plans.
"""
import pytest

import test_gpu_fp32_plans as f32
import test_gpu_sweep_split as f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(30720, 2), (30721, 2), (30739, 3), (31001, 5), (40001, 8), (31001, 9)])
@pytest.mark.parametrize("bc,scheme", [((0, 0), "muscl"), ((1, 1), "hllc"), ((1, 0), "muscl")])
def test_wide_grids_of_few_rows(nx, ny, bc, scheme):
    f64._check(nx, ny, bc, potential=bc != (0, 0), scheme=scheme)


@pytest.mark.parametrize("nx,ny", [(30721, 2), (31001, 8)])
def test_fp32(nx, ny):
    f32._sweep(nx, ny, (1, 0), "muscl")
