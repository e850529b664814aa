"""Grouping of the members by 32-bit keys around the sizes where the sort
changes its form (one workgroup, tiles of 4096, tiles of 8192) and just off
whole tiles: level-0 groups from labels with gaps, and their members' records
as the halo properties read them.  Bit-identical to the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2412_18629_amd as rs
from test_gpu_phase import compare
from test_gpu_props import _bits, _props_both

pytestmark = pytest.mark.gpu
BOX = 100.0


@pytest.mark.parametrize("n", [1, 8191, 8192, 8193, 12288, 12289, 65535])
def test_group_records(n):
    rng = np.random.default_rng(n)
    arrs = [(rng.random(n) * BOX).astype(np.float32) for _ in range(3)]
    for a in arrs:
        a[a >= np.float32(BOX)] = 0.0
    arrs += [(rng.normal(size=n) * 200).astype(np.float32) for _ in range(3)]
    # groups of 1 to about 60 members, the label being the smallest index
    g = rng.integers(0, max(n // 30, 1), n)
    first = np.full(g.max() + 1, n)
    np.minimum.at(first, g, np.arange(n))
    labels = first[g].astype(np.int32)
    ref = oracle.phase_fof(*arrs, BOX, labels)
    dev = [torch.from_numpy(a).cuda() for a in arrs]
    compare(rs.rs_phase_fof_batch(*dev, BOX, torch.from_numpy(labels).cuda()), ref)
    if ref["size"].size:
        got, want = _props_both(arrs, BOX, ref)
        assert np.array_equal(_bits(got), _bits(want))
