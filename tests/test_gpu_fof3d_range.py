"""Coordinates out of range: every particle (wrong units), one, or NaN, on
grids with and without auto-linking, in the three 3D entry points and on both
sides of the size up to which the host reads the error only at the end.  The
call reports RS_ERANGE, leaves the labels alone and tests no pair."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2412_18629_amd as rs

pytestmark = pytest.mark.gpu
BOX = 10.0


def _noalloc(pos, ll, lab):
    rc = rs.load().rs_fof3d_noalloc(*[ctypes.c_void_p(c.data_ptr()) for c in pos],
                                    pos[0].numel(), BOX, float(ll),
                                    ctypes.c_void_p(lab.data_ptr()), None,
                                    ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    if rc != rs.RS_OK:
        raise rs.RsError(rc, "rs_fof3d_noalloc")


CALLS = {
    "box": lambda pos, ll, lab: rs.rs_fof3d(*pos, BOX, ll, labels=lab),
    "noalloc": _noalloc,
    "subbox": lambda pos, ll, lab: rs.rs_fof3d_subbox(*pos, pos[0].numel(), [0.0] * 3, [BOX] * 3,
                                                      0.0, ll, labels=lab),
}


@pytest.mark.parametrize("n,ll", [(1, 0.3), (2000, 0.3), (2000, BOX / 2.5), (65537, 0.3)])
@pytest.mark.parametrize("bad", ["units", "one", "nan"])
@pytest.mark.parametrize("call", list(CALLS))
def test_nothing_is_tested(call, bad, n, ll):
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    pos = [torch.rand(n, generator=g, device="cuda") * 9.99 for _ in range(3)]
    if bad == "units":
        pos = [c * 1000.0 + BOX for c in pos]
    else:
        pos[2][n // 2] = float("nan") if bad == "nan" else float(np.nextafter(np.float32(0), -1))
    lab = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    rs.rs_profile_enable(2)
    try:
        with pytest.raises(rs.RsError) as e:
            CALLS[call](pos, ll, lab)
        tested = rs.rs_profile_get("pairs_fof3d")[2]
    finally:
        rs.rs_profile_enable(0)
    assert e.value.status == rs.RS_ERANGE
    assert bool((lab == -7).all())
    assert tested == 0
