"""Every tube of a batch is advanced once, whatever the number of tubes, workgroups
that start at once and workgroup size: each tube equals bitwise a batch of that tube
alone (one tube has one schedule).  Counts below, at and above one and two tubes per
compute unit (256 of them), and more tubes than workgroups that start at once.
"""
import numpy as np
import pytest
import torch

import paper_1210_5246_amd as csh
import workloads as wl

pytestmark = pytest.mark.gpu

LENGTHS = (1, 2, 59, 61, 130, 7)


def _primitive(n, seed):
    return wl.periodic(64, seed).W.reshape(6, -1)[:, :n]


def _alone(n, W, steps):
    b = csh.Batch(torch.from_numpy(np.ascontiguousarray(W)).cuda(), np.array([0, n]))
    dts = b.run(steps, 0.8, threads=64)
    return b.U.cpu().numpy(), dts.cpu().numpy()[0]


@pytest.mark.parametrize("threads", [None, 64, 1024])
@pytest.mark.parametrize("ntubes", [1, 255, 257, 512, 700, 1100])
def test_every_tube_advances(ntubes, threads):
    print("batch orders", ntubes, threads, flush=True)
    steps = 3
    parts = [_primitive(n, 90 + k) for k, n in enumerate(LENGTHS)]
    want = [_alone(n, W, steps) for n, W in zip(LENGTHS, parts)]
    which = np.random.default_rng(ntubes).integers(len(LENGTHS), size=ntubes)
    off = np.concatenate([[0], np.cumsum([LENGTHS[k] for k in which])])
    b = csh.Batch(torch.from_numpy(np.ascontiguousarray(np.concatenate([parts[k] for k in which], axis=1))).cuda(), off)
    dts = b.run(steps, 0.8, threads=threads or 0).cpu().numpy()
    U = b.U.cpu().numpy()
    for j, k in enumerate(which):
        np.testing.assert_array_equal(U[:, off[j]:off[j + 1]], want[k][0])
        np.testing.assert_array_equal(dts[j], want[k][1])
