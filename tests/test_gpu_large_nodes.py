"""Groups just above the small-node limit and a few times it, of the kinds
whose pairs take another path in the large-node searches: compact clumps,
clumps across the periodic faces, groups that percolate (no culling), lattices
(every nearest distance tied, leaves of equal points' boxes touching) and sets
with duplicate points; exact and bracketed searches, 32- and 64-bit member
offsets.  Bit-identical to the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2412_18629_amd as rs
from paper_2412_18629_amd import learn
from test_gpu_phase import compare
from test_gpu_small_nodes import BOX, _group

pytestmark = pytest.mark.gpu
SIZES = [2049, 2050, 2112, 2113, 3000, 6001]


def _set(kind):
    rng = np.random.default_rng(100 + len(kind))
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
    return [*pos.T, *vel.T], first[group].astype(np.int32)


@pytest.mark.parametrize("wide", ["", "1"], ids=["offsets32", "offsets64"])
@pytest.mark.parametrize("kind", ["compact", "face", "percolating", "lattice", "duplicates"])
def test_large_nodes_match_oracle(kind, wide, monkeypatch):
    if wide:
        monkeypatch.setenv("RS_DEBUG_WIDE_OFFSETS", "1")
    arrs, labels = _set(kind)
    ref = oracle.phase_fof(*arrs, BOX, labels)
    assert (ref["size"] > 2048).sum() >= len(SIZES)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in arrs]
    lab = torch.from_numpy(labels).cuda()
    compare(rs.rs_phase_fof_batch(*dev, BOX, lab), ref)
    compare(rs.rs_phase_fof_batch(*dev, BOX, lab, flags=rs.RS_LEARNED,
                                  model=learn.load_model()), ref)
