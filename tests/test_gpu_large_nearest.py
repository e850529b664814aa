"""Nearest-neighbour search of groups above the small-node limit whose members
reach very differently far: a dense core with a power-law tail (a tile's
outliers are left to the search of single queries), and separate clumps of
one, a few and many leaves.  Sizes leave a lone member or a full tile at the
end; exact and bracketed searches.  Bit-identical to the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2412_18629_amd as rs
from paper_2412_18629_amd import learn
from test_gpu_phase import compare

pytestmark = pytest.mark.gpu
BOX = 100.0


def _points(kind, rng, n):
    if kind == "tail":
        u = rng.random(n) ** 6
    else:
        u = (rng.random(n) < 0.02) * rng.random(n)
    d = rng.normal(size=(n, 6))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    at = np.zeros((n, 6))
    if kind == "clumps":
        c = rng.integers(0, 40, n) ** 2 // 40
        at[:, :3] = rng.normal(size=(40, 3))[c] * 3.0
        at[:, 3:] = rng.normal(size=(40, 3))[c] * 300.0
        at += rng.normal(size=(n, 6)) * np.array([0.05] * 3 + [5.0] * 3)
    at += d * u[:, None] * np.array([4.0] * 3 + [400.0] * 3)
    return at + np.array([rng.random() * BOX, 50.0, 0.5, 0, 0, 0])


@pytest.mark.parametrize("kind", ["tail", "clumps"])
@pytest.mark.parametrize("sizes", [(2049,), (2112, 4097), (20000, 2240)], ids=str)
def test_nearest_of_uneven_groups(kind, sizes):
    rng = np.random.default_rng(sum(sizes) + len(kind))
    x = np.concatenate([_points(kind, rng, n) for n in sizes]).astype(np.float32)
    x[:, :3] %= np.float32(BOX)
    x[:, :3][x[:, :3] >= np.float32(BOX)] = 0.0
    first = np.concatenate([np.full(n, sum(sizes[:g])) for g, n in enumerate(sizes)])
    arrs, labels = [np.ascontiguousarray(c) for c in x.T], first.astype(np.int32)
    ref = oracle.phase_fof(*arrs, BOX, labels)
    dev = [torch.from_numpy(a).cuda() for a in arrs]
    lab = torch.from_numpy(labels).cuda()
    compare(rs.rs_phase_fof_batch(*dev, BOX, lab), ref)
    compare(rs.rs_phase_fof_batch(*dev, BOX, lab, flags=rs.RS_LEARNED,
                                  model=learn.load_model()), ref)
