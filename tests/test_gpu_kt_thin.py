"""The Kurganov-Tadmor step on wide grids of few rows, which FP64 takes by the march with
segments shorter than eight rows and FP32 by either kernel: one step against the oracle,
tolerances as in test_gpu_kt_block.
"""
import pytest
import torch

from test_gpu_kt_block import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(14337, 2), (16001, 3), (30001, 5), (20003, 7), (60001, 8), (16007, 13)])
@pytest.mark.parametrize("bc", [(0, 0), (1, 1)])
def test_wide_grids_of_few_rows(nx, ny, bc):
    _check(nx, ny, bc, potential=bc == (1, 1))
    _check(nx, ny, bc, dtype=torch.float32, tol=2e-5)
