"""The 3D pass on one dense clump, where most octant pairs are deferred to the
second pass: labels identical to the oracle's over the link lengths where the
clump falls apart, in a periodic box and in a sub-box, also with a queue of a
few entries; and no link length among them takes many times another's time."""
import time

import numpy as np
import pytest
import torch

import oracle
import paper_2412_18629_amd as rs

pytestmark = pytest.mark.gpu
BOX = 100.0


def _clump(n):
    rng = np.random.default_rng(n)
    pos = rng.normal(BOX / 2, BOX / 200, (3, n)).astype(np.float32)
    return [np.ascontiguousarray(np.clip(c, 0, np.float32(BOX * 0.999))) for c in pos]


@pytest.mark.parametrize("queue", ["", "100"], ids=["room", "full"])
@pytest.mark.parametrize("b", [0.05, 0.1, 0.15, 0.2, 0.28])
def test_labels(b, queue, monkeypatch):
    n = 20000
    if queue:
        monkeypatch.setenv("RS_DEBUG_HEAVY_QUEUE", queue)
    host, ll = _clump(n), BOX / n ** (1 / 3) * b
    dev = [torch.from_numpy(c).cuda() for c in host]
    ref = oracle.fof3d(*host, BOX, ll)
    assert np.array_equal(rs.rs_fof3d(*dev, BOX, ll)[0].cpu().numpy(), ref)
    lo, hi = [0.0] * 3, [BOX] * 3
    want = oracle.fof3d_subbox(*host, n, lo, hi, 0.0, ll)
    got, _ = rs.rs_fof3d_subbox(*dev, n, lo, hi, 0.0, ll)
    assert np.array_equal(got.cpu().numpy(), want[0] if isinstance(want, tuple) else want)


@pytest.mark.parametrize("n", [60000, 400000])
def test_time_over_link_lengths(n):
    dev = [torch.from_numpy(c).cuda() for c in _clump(n)]

    def best(b):
        times = []
        for _ in range(4):
            torch.cuda.synchronize()
            t = time.perf_counter()
            rs.rs_fof3d(*dev, BOX, BOX / n ** (1 / 3) * b)
            times.append(time.perf_counter() - t)
        return min(times)

    times = [best(b) for b in (0.15, 0.2, 0.24, 0.28)]
    assert max(times) < 5 * min(times), times
