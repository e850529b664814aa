"""Large nodes whose pairs the screening cannot tell apart: two or three compact
clumps far apart (each below the resolution of the search tree's cells), also
across the periodic face, such clumps beside an ordinary one, and coinciding
members; exact and bracketed searches, 32- and 64-bit member offsets.
Bit-identical to the oracle, and not slower than the pairs themselves explain."""
import time

import numpy as np
import pytest
import torch

import oracle
import paper_2412_18629_amd as rs
from paper_2412_18629_amd import learn
from test_gpu_phase import compare
from test_gpu_small_nodes import BOX, _clump

pytestmark = pytest.mark.gpu
SIZES = [2049, 2500, 4100, 6001]


def _clumps(rng, n, centre, number):
    """`number` clumps of 1e-3 Mpc and 0.3 km/s, 10 Mpc and 1000 km/s apart."""
    which = rng.integers(0, number, n)[:, None] - (number - 1) / 2
    pos, vel = rng.normal(0, 1e-3, (n, 3)), rng.normal(0, 0.3, (n, 3))
    return (pos + 10.0 * which + centre) % BOX, vel + 1000.0 * which


def _group(kind, rng, n):
    centre = rng.uniform(20, BOX - 20, 3)
    if kind == "two":
        return _clumps(rng, n, centre, 2)
    if kind == "three":
        return _clumps(rng, n, centre, 3)
    if kind == "face":
        return _clumps(rng, n, np.array([5.0, 50.0, BOX - 5.0]), 2)
    if kind == "mixed":
        pos, vel = _clump(rng, n, centre)
        m = n // 2
        pos[:m], vel[:m] = _clumps(rng, m, centre + 3.0, 2)
        return pos, vel
    pos, vel = _clump(rng, n, centre)          # few distinct points
    pick = rng.integers(0, 20, n)
    return pos[pick], vel[pick]


def _set(kind, sizes, seed):
    rng = np.random.default_rng(seed)
    groups = [_group(kind, rng, n) for n in sizes]
    x = np.concatenate([np.concatenate([g[0] for g in groups]),
                        np.concatenate([g[1] for g in groups])], 1).astype(np.float32)
    x[:, :3][x[:, :3] >= np.float32(BOX)] = 0.0
    first = np.concatenate([np.full(n, sum(sizes[:g])) for g, n in enumerate(sizes)])
    return [np.ascontiguousarray(c) for c in x.T], first.astype(np.int32)


@pytest.mark.parametrize("wide", ["", "1"], ids=["offsets32", "offsets64"])
@pytest.mark.parametrize("kind", ["two", "three", "face", "mixed", "few points"])
def test_matches_oracle(kind, wide, monkeypatch):
    if wide:
        monkeypatch.setenv("RS_DEBUG_WIDE_OFFSETS", "1")
    arrs, labels = _set(kind, SIZES, len(kind))
    dev = [torch.from_numpy(a).cuda() for a in arrs]
    lab = torch.from_numpy(labels).cuda()
    for f in (0.7, 0.95):
        ref = oracle.phase_fof(*arrs, BOX, labels, f=f, brute_max=10000)
        compare(rs.rs_phase_fof_batch(*dev, BOX, lab, f=f), ref)
        compare(rs.rs_phase_fof_batch(*dev, BOX, lab, f=f, flags=rs.RS_LEARNED,
                                      model=learn.load_model()), ref)


def test_time_of_compact_clumps():
    """Two clumps of 50000 members (all 2.5e9 pairs tested) within 2.7 times an
    ordinary node's time."""
    def best(groups):
        x = np.concatenate([np.concatenate([g[k] for g in groups]) for k in (0, 1)], 1)
        dev = [torch.from_numpy(np.ascontiguousarray(c)).cuda() for c in x.astype(np.float32).T]
        lab = torch.zeros(len(x), dtype=torch.int32, device="cuda")
        times = []
        for _ in range(5):
            torch.cuda.synchronize()
            t = time.perf_counter()
            rs.rs_phase_fof_batch(*dev, BOX, lab)
            times.append(time.perf_counter() - t)
        return min(times)

    rng = np.random.default_rng(2)
    centre = np.array([50.0, 50.0, 50.0])
    ordinary = best([_clump(rng, 100000, centre)])
    assert best([_clumps(rng, 100000, centre, 2)]) < 2.7 * ordinary
