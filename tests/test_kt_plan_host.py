"""Which kernel takes the 2-D Kurganov-Tadmor step (kt_plan, called in the library on the
CPU): in FP64 the block kernel where one round of its workgroups holds the grid, never
in more (the march was faster at every size measured, by up to two times on wide grids
of few rows); segments no taller than the grid; no more workgroups than planned.
"""
import ctypes
import random
import re
import subprocess

import pytest

import paper_1210_5246_amd as csh


class Plan(ctypes.Structure):
    _fields_ = [("block", ctypes.c_bool), ("rows", ctypes.c_int)]


@pytest.fixture(scope="module")
def plan():
    names = subprocess.run(["nm", "-D", csh.LIB_PATH], capture_output=True, text=True, check=True).stdout
    f = getattr(csh.lib(), re.search(r"\b(_Z\w*7kt_plan\w*)", names).group(1))
    f.restype, f.argtypes = Plan, [ctypes.c_int, ctypes.c_int, ctypes.c_bool]
    return lambda nx, ny, f64: (lambda p: (p.block, p.rows))(f(nx, ny, f64))


def _workgroups(nx, ny, rows):
    return -(-nx // 56) * -(-ny // rows)


@pytest.mark.parametrize("nx,ny", [(100000, 2), (120000, 3), (30000, 5), (60000, 8), (120000, 20), (30000, 64),
                                   (1024, 1024), (1500, 1500), (4096, 4096)])
def test_the_march_where_the_blocks_take_more_than_a_round(plan, nx, ny):
    assert not plan(nx, ny, True)[0]


@pytest.mark.parametrize("nx,ny", [(100, 100), (512, 512), (1000, 700), (900, 500), (4000, 48), (57, 2), (10000, 2)])
def test_the_block_in_one_round(plan, nx, ny):
    assert plan(nx, ny, True)[0] and plan(nx, ny, False)[0]


def test_any_grid(plan):
    g = random.Random(5)
    for _ in range(3000):
        nx, ny = (round(2 ** g.uniform(0, 17)) for _ in range(2))
        ny = max(2, min(ny, (1 << 28) // nx))
        for f64 in (True, False):
            block, rows = plan(nx, ny, f64)
            assert 1 <= rows <= min(ny, 52 if block else 96), (nx, ny, f64)
            if block:
                assert _workgroups(nx, ny, rows) <= (256 if f64 else 3 * 512), (nx, ny, f64)
