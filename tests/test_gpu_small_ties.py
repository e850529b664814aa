"""Small nodes whose nearest neighbours the screening leaves undecided: lattices
and lines of equal spacing (also across the periodic face), two compact clumps
far apart, and clumps of which about half the members are tied, where the
search changes from single members to every pair.  Bit-identical to the
oracle, and not slower than the pairs themselves explain."""
import time

import numpy as np
import pytest
import torch

import paper_2412_18629_amd as rs
from test_gpu_phase import compare, run_both
from test_gpu_small_nodes import BOX, _clump, _lattice

pytestmark = pytest.mark.gpu
SIZES = [65, 127, 128, 129, 256, 257, 600, 1024, 1025, 2048]


def _group(kind, rng, n):
    centre = rng.uniform(20, BOX - 20, 3)
    if kind == "lattice":
        return _lattice(n, np.floor(centre))
    if kind == "face":
        return _lattice(n, np.array([BOX - 0.25, 50.0, 0.0]))
    if kind == "line":
        pos = np.tile(np.floor(centre), (n, 1))
        pos[:, 0] += 0.0078125 * np.arange(n)
        return pos % BOX, np.zeros((n, 3))
    if kind == "two clumps":
        pos, vel = rng.normal(0, 1e-3, (n, 3)), rng.normal(0, 0.3, (n, 3))
        side = np.where(rng.random(n) < 0.5, 1, -1)[:, None]
        return (pos + 5 * side + centre) % BOX, vel + 500.0 * side
    # about half of the members in triples of coinciding points
    tied = n // 2 + {"half less": -3, "half": 0, "half more": 3}[kind]
    pos, vel = _clump(rng, n, centre)
    first = np.arange(tied) // 3
    pos[:tied], vel[:tied] = pos[first], vel[first]
    return pos, vel


def _set(kind, sizes, seed):
    rng = np.random.default_rng(seed)
    groups = [_group(kind, rng, n) for n in sizes]
    x = np.concatenate([np.concatenate([g[0] for g in groups]),
                        np.concatenate([g[1] for g in groups])], 1).astype(np.float32)
    x[:, :3][x[:, :3] >= np.float32(BOX)] = 0.0
    first = np.concatenate([np.full(n, sum(sizes[:g])) for g, n in enumerate(sizes)])
    return [np.ascontiguousarray(c) for c in x.T], first.astype(np.int32)


@pytest.mark.parametrize("kind", ["lattice", "face", "line", "two clumps", "half less", "half",
                                  "half more"])
@pytest.mark.parametrize("kw", [{}, {"min_sub": 2, "f": 0.95}], ids=["default", "min_sub2"])
def test_matches_oracle(kind, kw):
    arrs, labels = _set(kind, SIZES, len(kind))
    got, ref = run_both(arrs, BOX, labels, **kw)
    compare(got, ref)


def test_time_of_tied_and_percolating_nodes():
    """A node of 2048 members whose pairs all have to be evaluated (2.1 million
    tests) within twice and a half the time of an ordinary one."""
    def best(arrs, labels):
        dev = [torch.from_numpy(a).cuda() for a in arrs]
        lab = torch.from_numpy(labels).cuda()
        times = []
        for _ in range(5):
            torch.cuda.synchronize()
            t = time.perf_counter()
            rs.rs_phase_fof_batch(*dev, BOX, lab)
            times.append(time.perf_counter() - t)
        return min(times)

    rng = np.random.default_rng(1)
    sizes = [2048] * 64
    plain = [_clump(rng, 2048, rng.uniform(20, 80, 3)) for _ in sizes]
    _, labels = _set("line", sizes, 0)

    def arrays(groups):
        x = np.concatenate([np.concatenate([g[k] for g in groups]) for k in (0, 1)], 1)
        return [np.ascontiguousarray(c) for c in x.astype(np.float32).T]

    ordinary = best(arrays(plain), labels)
    box = [(rng.uniform(0, 99.9, (2048, 3)), rng.normal(0, 100.0, (2048, 3))) for _ in sizes]
    assert best(arrays(box), labels) < 2.5 * ordinary
    assert best(*_set("two clumps", sizes, 2)) < 2 * ordinary
    assert best(*_set("line", sizes, 3)) < 2 * ordinary
