"""Seed assignment at the edges of its screened path: seed counts around the
plain loop's limit (8), a 16-seed block and a 2048-seed run, for groups in
the box, across its faces, wider than half the box (no screening), and with
coinciding seeds (ties to the smaller node).  Identical to the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2412_18629_amd as rs

pytestmark = pytest.mark.gpu
L = 100.0
COUNTS = [2, 8, 9, 16, 17, 33, 300, 2048, 2049, 4100]


def _hierarchy(kind, rng, own=130):
    """One two-level group per count: `own` particles of the level-0 node and
    two particles in each of its leaves."""
    pos, vel, deep = [], [], []
    level, parent, size, a, c, first = [], [], [], [], [], []
    for k in COUNTS:                      # level-0 nodes
        level.append(0); parent.append(-1); size.append(own + 2 * k); a.append(1.0); c.append(1e-4)
    leaf_xy = []
    for g, k in enumerate(COUNTS):
        centre = np.zeros(3) if kind == "face" else rng.uniform(10, 90, 3)
        spread = 40.0 if kind == "wide" else 1.0
        p = centre + rng.uniform(-spread, spread, (k, 3))
        v = rng.normal(0, 200.0, (k, 3))
        s = rng.uniform(0.01, 0.3, k)     # sigma of each seed
        if kind == "ties":
            p[k // 2:], v[k // 2:], s[k // 2:] = p[:k - k // 2], v[:k - k // 2], s[:k - k // 2]
        leaf_xy.append((p, v))
        for j in range(k):
            level.append(1); parent.append(g); size.append(2)
            a.append(1.0 / s[j] ** 2); c.append(1.0 / (300.0 * s[j]) ** 2)
        pos.append(centre + rng.uniform(-1.2 * spread, 1.2 * spread, (own, 3)))
        vel.append(rng.normal(0, 250.0, (own, 3)))
        deep.append(np.full(own, g))
    node = len(COUNTS)
    for p, v in leaf_xy:
        pos.append(np.repeat(p, 2, 0)); vel.append(np.repeat(v, 2, 0))
        deep.append(np.repeat(np.arange(node, node + len(p)), 2))
        node += len(p)
    pos = (np.concatenate(pos) % L).astype(np.float32)
    pos[pos >= L] = 0.0
    vel = np.concatenate(vel).astype(np.float32)
    deep = np.concatenate(deep).astype(np.int32)
    parent = np.array(parent, np.int32)
    first = np.full(len(parent), len(deep), np.int32)
    np.minimum.at(first, deep, np.arange(len(deep), dtype=np.int32))
    np.minimum.at(first, parent[parent >= 0], first[parent >= 0])
    return pos, vel, dict(level=np.array(level, np.int32), parent=parent, min_index=first,
                          size=np.array(size, np.int32), deepest=deep,
                          a=np.array(a, np.float32), c=np.array(c, np.float32))


@pytest.mark.parametrize("kind", ["inside", "face", "wide", "ties"])
def test_many_seeds_match_oracle(kind):
    pos, vel, t = _hierarchy(kind, np.random.default_rng(len(kind)))
    dev = [torch.from_numpy(np.ascontiguousarray(q)).cuda() for q in [*pos.T, *vel.T]]
    T = {k: torch.from_numpy(v).cuda() for k, v in t.items()}
    T["n_levels"] = 2
    props = rs.rs_halo_props(*dev, L, T)
    got = rs.rs_seed_assign(*dev, L, T, props).cpu().numpy()
    ref = oracle.seed_assign(*pos.T, *vel.T, L, t["parent"], t["deepest"], t["a"], t["c"],
                             props.cpu().numpy())
    assert np.array_equal(got, ref), (np.nonzero(got != ref)[0][:5], kind)
