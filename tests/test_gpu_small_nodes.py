"""Groups at the edges of the small-node kernels -- one wavefront up to 64
members, 16- and 64-wide tiles beyond, the size buckets 256, 1024 and 2048 --
of every kind whose pairs take another path there: compact clumps, clumps
across the periodic faces, groups that percolate, lattices (every nearest
distance tied) and sets with duplicate points.  Bit-identical to the
oracle."""
import numpy as np
import pytest

import paper_2412_18629_amd as rs
from test_gpu_phase import compare, run_both

pytestmark = pytest.mark.gpu
BOX = 100.0
SIZES = [10, 33, 63, 64, 65, 66, 79, 80, 81, 127, 128, 129, 255, 256, 257, 400, 1008, 1023, 1024,
         1025, 1500, 2047, 2048]


def _clump(rng, n, centre):
    """A Gaussian clump with two colder, denser clumps inside it."""
    pos, vel = rng.normal(0, 0.3, (n, 3)), rng.normal(0, 150.0, (n, 3))
    for k, (off, v) in enumerate(((0.4, 200.0), (-0.3, -150.0))):
        m = n // 4
        s = slice(k * m, (k + 1) * m)
        pos[s] = off + rng.normal(0, 0.02, (m, 3))
        vel[s] = v + rng.normal(0, 20.0, (m, 3))
    return (pos + centre) % BOX, vel


def _lattice(n, centre):
    side = int(np.ceil(n ** (1 / 3)))
    g = np.stack(np.meshgrid(*[np.arange(side)] * 3, indexing="ij"), -1).reshape(-1, 3)[:n]
    return (g * 0.0625 + centre) % BOX, np.zeros((n, 3))


def _group(kind, rng, n):
    centre = rng.uniform(5, BOX - 5, 3)
    if kind == "compact":
        return _clump(rng, n, centre)
    if kind == "face":
        return _clump(rng, n, np.where(rng.random(3) < 0.7, 0.0, centre))
    if kind == "percolating":
        pos, vel = _clump(rng, n, centre)
        far = rng.random(n) < 0.2
        pos[far] = rng.uniform(0, BOX, (int(far.sum()), 3))
        return pos, vel
    if kind == "lattice":
        return _lattice(n, np.floor(centre))
    pos, vel = _clump(rng, n, centre)
    twin = rng.integers(0, n, n // 3)
    pos[:n // 3], vel[:n // 3] = pos[twin], vel[twin]
    return pos, vel


@pytest.mark.parametrize("kind", ["compact", "face", "percolating", "lattice", "duplicates"])
@pytest.mark.parametrize("kw", [{}, {"min_group": 2, "min_sub": 2, "f": 0.95}],
                         ids=["default", "min_sub2"])
def test_small_nodes_match_oracle(kind, kw):
    rng = np.random.default_rng(len(kind))
    pos, vel, group = [], [], []
    for g, n in enumerate(SIZES):
        p, v = _group(kind, rng, n)
        pos.append(p)
        vel.append(v)
        group.append(np.full(n, g))
    pos = np.concatenate(pos).astype(np.float32)
    pos[pos >= np.float32(BOX)] = 0.0
    vel = np.concatenate(vel).astype(np.float32)
    group = np.concatenate(group)
    order = rng.permutation(group.size)
    pos, vel, group = pos[order], vel[order], group[order]
    first = np.full(len(SIZES), group.size)
    np.minimum.at(first, group, np.arange(group.size))
    labels = first[group].astype(np.int32)
    got, ref = run_both([*pos.T, *vel.T], BOX, labels, **kw)
    assert (ref["size"] > 64).sum() > 10
    compare(got, ref)
    if kind == "percolating":
        assert ref["wide"].any()


def test_features_unchanged_between_forms():
    # a 64-member node's features come from one wavefront, a 65-member one's
    # from a workgroup: both against the plain form of the same set
    rng = np.random.default_rng(5)
    sets = [_clump(rng, n, rng.uniform(5, 95, 3)) for n in (64, 65, 300)]
    pos = np.concatenate([s[0] for s in sets]).astype(np.float32)
    vel = np.concatenate([s[1] for s in sets]).astype(np.float32)
    labels = np.repeat([0, 64, 129], [64, 65, 300]).astype(np.int32)
    a, _ = run_both([*pos.T, *vel.T], BOX, labels, flags=rs.RS_BATCHED | rs.RS_FEATURES)
    b, _ = run_both([*pos.T, *vel.T], BOX, labels, flags=rs.RS_PLAIN | rs.RS_FEATURES)
    fa, fb = a["features"].cpu().numpy(), b["features"].cpu().numpy()
    assert np.array_equal(fa, fb)
    size = a["size"].cpu().numpy()
    assert np.allclose(fa[:, 0], np.log(size), rtol=1e-6)
    assert np.allclose(fa[:, 7:15].sum(1), 1.0, rtol=1e-5)
    assert np.allclose(fa[:, 15:23].sum(1), 1.0, rtol=1e-5)
