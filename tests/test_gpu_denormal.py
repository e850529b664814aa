"""Squared distances in the denormal range, which the pair arithmetic keeps:
coinciding positions whose velocities differ by 1e-23 to 1e-18 km/s, and clumps
of that size about the origin beside an ordinary one.  Nodes of every size
class and the seeds, bit-identical to the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2412_18629_amd as rs
from paper_2412_18629_amd import learn
from test_gpu_phase import compare

pytestmark = pytest.mark.gpu
BOX = 100.0


def _groups(kind, scale, sizes):
    rng = np.random.default_rng(int(-np.log10(scale)))
    pos, vel = [], []
    for n in sizes:
        centre = rng.uniform(5, BOX - 5, 3)
        p, v = np.tile(centre, (n, 1)), rng.normal(0, 1, (n, 3)) * scale
        if kind == "origin":
            # two thirds about the origin, the rest an ordinary clump beside it
            m = 2 * n // 3
            p[:m] = np.abs(rng.normal(0, 1, (m, 3))) * scale
            p[m:] = np.abs(rng.normal(0.2, 0.05, (n - m, 3)))
            v[m:] = rng.normal(0, 100.0, (n - m, 3))
        pos.append(p)
        vel.append(v)
    x = np.concatenate([np.concatenate(pos), np.concatenate(vel)], 1).astype(np.float32)
    first = np.concatenate([np.full(n, sum(sizes[:g])) for g, n in enumerate(sizes)])
    return [np.ascontiguousarray(c) for c in x.T], first.astype(np.int32)


@pytest.mark.parametrize("scale", [1e-22, 1e-21, 1e-18])
@pytest.mark.parametrize("kind", ["velocity", "origin"])
def test_hierarchy_and_seeds(kind, scale):
    for sizes, kw in (([64, 65, 256, 300, 1030, 2049], {}),
                      ([64, 65, 300, 1030], {"min_sub": 2, "f": 0.9})):
        arrs, labels = _groups(kind, scale, sizes)
        dev = [torch.from_numpy(a).cuda() for a in arrs]
        lab = torch.from_numpy(labels).cuda()
        ref = oracle.phase_fof(*arrs, BOX, labels, brute_max=4000, **kw)
        tree = rs.rs_phase_fof_batch(*dev, BOX, lab, **kw)
        compare(tree, ref)
        compare(rs.rs_phase_fof_batch(*dev, BOX, lab, flags=rs.RS_LEARNED,
                                      model=learn.load_model(), **kw), ref)
        props = rs.rs_halo_props(*dev, BOX, tree)
        want = oracle.seed_assign(*arrs, BOX, *[ref[k] for k in ("parent", "deepest", "a", "c")],
                                  props.cpu().numpy())
        assert np.array_equal(rs.rs_seed_assign(*dev, BOX, tree, props).cpu().numpy(), want)
