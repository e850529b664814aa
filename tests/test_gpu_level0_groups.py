"""Level-0 groups whose members fill part of a row, whole rows and several rows
of the percolation pass, in every alignment, with labels dropped between them
and some groups spanning the box; exact results of the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2412_18629_amd as rs
from test_gpu_phase import compare

pytestmark = pytest.mark.gpu
BOX = 100.0
SIZES = [1, 20, 63, 64, 65, 19, 1023, 1024, 1025, 130, 2500, 40]


@pytest.mark.parametrize("shift", [0, 1, 37])
def test_level0_groups(shift):
    rng = np.random.default_rng(shift)
    sizes = [3] * shift + SIZES
    xs, grp = [], []
    for g, n in enumerate(sizes):
        at = rng.normal(size=(n, 6)) * np.array([0.3] * 3 + [30.0] * 3)
        if g % 3 == 1:   # a chain along one axis, across the periodic face
            at[:, g % 2] += np.linspace(0, BOX * (0.3 + 0.1 * (g % 5)), n)
        xs.append(at + np.array([*(rng.random(3) * BOX), 0, 0, 0]))
        grp.append(np.full(n, g))
    x, grp = np.concatenate(xs).astype(np.float32), np.concatenate(grp)
    x[:, :3] %= np.float32(BOX)
    x[:, :3][x[:, :3] >= np.float32(BOX)] = 0.0
    order = rng.permutation(grp.size)
    x, grp = x[order], grp[order]
    first = np.full(len(sizes), grp.size)
    np.minimum.at(first, grp, np.arange(grp.size))
    arrs, labels = [np.ascontiguousarray(c) for c in x.T], first[grp].astype(np.int32)
    ref = oracle.phase_fof(*arrs, BOX, labels)
    dev = [torch.from_numpy(a).cuda() for a in arrs]
    compare(rs.rs_phase_fof_batch(*dev, BOX, torch.from_numpy(labels).cuda()), ref)
