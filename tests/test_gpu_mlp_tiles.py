"""The minibatch kernel at the edges of its 32-sample tiles and past the
largest number of workgroups (512), against the fp64 reference.  Bounds: a
chain of at most 24 + 64 + 64 fp32 multiply-adds per element and fp32 sums
over at most a workgroup's samples give errors of a few hundred 2^-24 of an
element's summed magnitudes; 1e-4 of the largest element covers that with the
cancellation of random rows."""
import numpy as np
import pytest
import torch

import paper_2412_18629_amd as rs
from oracle import mlp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 31, 32, 33, 63, 65, 1000, 512 * 32 + 1, 40007])
def test_minibatch_tiles_match_oracle(n):
    rng = np.random.default_rng(n)
    p = (mlp.init(n) + rng.normal(0, 0.02, mlp.NPARAM)).astype(np.float32)
    X = rng.normal(0, 1, (n, mlp.NIN)).astype(np.float32)
    t = rng.normal(0, 1, n).astype(np.float32)
    P, Xd, T = (torch.from_numpy(a).cuda() for a in (p, X, t))
    g, loss = rs.rs_mlp_grad(P, Xd, T)
    ref = mlp.grad(p.astype(np.float64), X.astype(np.float64), t.astype(np.float64))
    assert np.abs(g.cpu().numpy() - ref).max() <= 1e-4 * np.abs(ref).max() + 1e-7
    want = mlp.loss(p, X, t)
    assert abs(loss.item() - want) <= 1e-4 * max(1.0, want)
    y = rs.rs_mlp_forward(P, Xd).cpu().numpy()
    y_ref, _ = mlp.forward(p, X)
    assert np.abs(y - y_ref).max() <= 1e-5 * max(1.0, np.abs(y_ref).max())
    again, loss2 = rs.rs_mlp_grad(P, Xd, T)
    assert torch.equal(g, again) and torch.equal(loss, loss2)
