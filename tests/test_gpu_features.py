"""The 24 proposer features of every node, computed here in 64 bits from the
members that parent and deepest give, for nodes of one wavefront (64 members),
of a workgroup (65, 300, 2048) and of the large-node pipeline (2049, 5000),
inside the box and across its faces, in the batched and the plain form.
ln N, the dispersion shares and the level are exact up to the fp32 rounding of
the result (2^-23 relative; the shares divide exact integers); the two
histograms are counts over N, where a member within 1e-5 of a bin's edge, some
twenty roundings of the fp32 radius, may fall to either side."""
import numpy as np
import pytest
import torch

import paper_2412_18629_amd as rs
from test_gpu_small_nodes import BOX, _clump

pytestmark = pytest.mark.gpu
SIZES = [64, 65, 300, 2048, 2049, 5000]
EDGES = np.array([0.25, 0.5, 0.75, 1.0, 1.5, 2.0, 3.0])


def _members(parent, deepest):
    """Member indices of every node: the particles at or below it."""
    own = [np.nonzero(deepest == k)[0] for k in range(parent.size)]
    for k in range(parent.size - 1, -1, -1):
        if parent[k] >= 0:
            own[parent[k]] = np.concatenate([own[parent[k]], own[k]])
    return [np.sort(m) for m in own]


def _bins(r, sigma):
    """Smallest and largest counts per bin that the edges' tolerance allows."""
    t = r / sigma
    lo = np.searchsorted(EDGES, t * (1 - 1e-5), side="right")
    hi = np.searchsorted(EDGES, t * (1 + 1e-5), side="right")
    sure = np.bincount(lo[lo == hi], minlength=8)
    return sure, sure + np.bincount(lo[lo != hi], minlength=8) + np.bincount(hi[lo != hi],
                                                                            minlength=8)


def _check(feat, x, v, members, level):
    n = len(members)
    q = np.rint(x[members].astype(np.float64) * 2.0 ** 20)
    d = q - q[0]                     # members ascend: the first is the reference
    L = np.rint(BOX * 2.0 ** 20)
    d = (d - L * (2 * d > L) + L * (2 * d <= -L)) * 2.0 ** -20
    w = np.rint(v[members].astype(np.float64) * 2.0 ** 10) * 2.0 ** -10
    assert abs(feat[0] - np.log(n)) <= 2.0 ** -22 * np.log(n)
    assert feat[23] == level
    for cols, y, hist in ((slice(1, 4), d, feat[7:15]), (slice(4, 7), w, feat[15:23])):
        var = y.var(0)
        assert np.allclose(feat[cols], var / var.sum(), rtol=1e-6, atol=1e-7), (n, level)
        radius = np.sqrt(((y - y.mean(0)) ** 2).sum(1))
        low, high = _bins(radius, np.sqrt(var.sum()))
        count = np.rint(hist.astype(np.float64) * n)
        assert np.allclose(hist * n, count, atol=1e-2)
        assert count.sum() == n
        assert ((low <= count) & (count <= high)).all(), (n, level, low, count, high)


@pytest.mark.parametrize("flags", [rs.RS_BATCHED, rs.RS_PLAIN], ids=["batched", "plain"])
@pytest.mark.parametrize("where", ["inside", "face"])
def test_features(where, flags):
    rng = np.random.default_rng(7)
    pos, vel = [], []
    for n in SIZES:
        centre = rng.uniform(10, BOX - 10, 3)
        if where == "face":
            centre = np.array([0.05, BOX - 0.1, centre[2]])
        p, u = _clump(rng, n, centre)
        # axes of different extent, so that no two of them can change places
        pos.append((centre + ((p - centre + BOX / 2) % BOX - BOX / 2) * [1.0, 0.5, 2.0]) % BOX)
        vel.append(u * [0.3, 1.0, 0.6])
    x = np.concatenate(pos).astype(np.float32)
    x[x >= np.float32(BOX)] = 0.0
    v = np.concatenate(vel).astype(np.float32)
    first = np.concatenate([np.full(n, sum(SIZES[:g])) for g, n in enumerate(SIZES)])
    dev = [torch.from_numpy(np.ascontiguousarray(c)).cuda() for c in (*x.T, *v.T)]
    tree = rs.rs_phase_fof_batch(*dev, BOX, torch.from_numpy(first.astype(np.int32)).cuda(),
                                 flags=flags | rs.RS_FEATURES)
    parent, deepest, level, size = (tree[k].cpu().numpy()
                                    for k in ("parent", "deepest", "level", "size"))
    feat = tree["features"].cpu().numpy()
    members = _members(parent, deepest)
    assert sorted(size[level == 0]) == SIZES and (level > 0).sum() > 20
    for k, m in enumerate(members):
        assert len(m) == size[k]
        _check(feat[k].astype(np.float64), x, v, m, level[k])
