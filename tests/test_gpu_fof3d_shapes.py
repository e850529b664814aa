"""The 3D pass at the limits of its launch shapes -- counts read on the device
up to 65536 particles, one thread per octant and neighbour cell, octant pairs
deferred above 128 member pairs, 2048-slot tiles -- on clustered and
unclustered boxes, a grid of a few cells and one without auto-linking, and
the range error that the short path finds after its launches.  Labels
identical to the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import paper_2412_18629_amd as rs
from paper_2412_18629_amd import synth

pytestmark = pytest.mark.gpu


def _run(pos, box, ll):
    dev = [torch.from_numpy(np.ascontiguousarray(c)).cuda() for c in pos]
    lab, ng = rs.rs_fof3d(*dev, box, ll)
    ref = oracle.fof3d(*pos, box, ll)
    assert np.array_equal(lab.cpu().numpy(), ref)
    assert ng == np.unique(ref).size


@pytest.mark.parametrize("n", [1, 2, 2047, 2048, 2049, 65535, 65536, 65537, 300001])
@pytest.mark.parametrize("kind", ["clustered", "uniform"])
def test_sizes(n, kind):
    cfg = synth.scaled(synth.CONFIGS["c32"], n)
    if kind == "clustered" and n > 2:
        pos = [a.numpy() for a in synth.generate(cfg, n)[:3]]
    else:
        pos = [a.numpy() for a in synth.random_uniform(n, cfg.box, n)[:3]]
    _run(pos, cfg.box, cfg.link_len)


@pytest.mark.parametrize("cells", [1, 2, 3, 4])
def test_coarse_grids(cells):
    # ll is about box / cells: every octant holds many particles (heavy pairs)
    # and, below three cells, neighbours coincide and nothing is auto-linked
    rng = np.random.default_rng(cells)
    pos = [rng.uniform(0, 10, 3000).astype(np.float32) for _ in range(3)]
    for c in pos:
        c[c >= 10] = 0
    _run(pos, 10.0, 0.99 * 10 / cells if cells > 2 else 0.2 * 10 / cells + 1.5)


def test_range_error_leaves_labels():
    x = torch.rand(5000, device="cuda")
    y, z = x.flip(0).contiguous(), x.clone()
    z[4321] = float("nan")
    lab = torch.full((5000,), -7, dtype=torch.int32, device="cuda")
    with pytest.raises(rs.RsError) as e:
        rs.rs_fof3d(x, y, z, 1.0, 0.01, labels=lab)
    assert e.value.status == rs.RS_ERANGE and bool((lab == -7).all())
