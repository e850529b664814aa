"""The sort's three shapes -- one workgroup up to 8192 pairs, 4096-key tiles,
8192-key tiles from 2^24 pairs -- at their limits and with tile counts that
do and do not fill the rounds over the XCDs, against a stable argsort."""
import numpy as np
import pytest
import torch

import paper_2412_18629_amd as rs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1023, 1024, 1025, 8191, 8192, 8193, 4096 * 128, 4096 * 256 + 1,
                               (1 << 24) - 1, 1 << 24, (1 << 24) + 8193])
@pytest.mark.parametrize("bits", [7, 24, 42, 64])
def test_shapes(n, bits):
    g = torch.Generator(device="cuda").manual_seed(n + bits)
    keys = torch.randint(-(1 << 63), (1 << 63) - 1, (n,), generator=g, dtype=torch.int64,
                         device="cuda")
    keys[: n // 3] &= 0xFFF          # long runs of equal digits
    vals = torch.arange(n, dtype=torch.int32, device="cuda")
    ko, vo = rs.rs_sort_pairs(keys, vals, bits)
    k = keys.cpu().numpy().view(np.uint64)
    mask = np.uint64((1 << bits) - 1) if bits < 64 else np.uint64(0xFFFFFFFFFFFFFFFF)
    order = np.argsort(k & mask, kind="stable")
    assert np.array_equal(vo.cpu().numpy(), order.astype(np.int32))
    assert np.array_equal(ko.cpu().numpy().view(np.uint64), k[order])
