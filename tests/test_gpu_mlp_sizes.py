"""Selector training kernels at the edges of their tiles: batches around the
samples of one workgroup (8) and the samples a gradient workgroup has in
flight (256), one output up to all of them, and an empty mask."""
import numpy as np
import pytest

from oracle import mlp as OM
from paper_1210_2536_amd import capi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_out", [1, capi.K_COUNT])
@pytest.mark.parametrize("B", [1, 7, 8, 9, 63, 255, 256, 257, 1025])
def test_mlp_backward_sizes(B, n_out):
    import torch
    from paper_1210_2536_amd import spmv as G
    rng = np.random.default_rng([63, B, n_out])
    flat = rng.normal(0, 0.3, OM.n_params(n_out)).astype(np.float32)
    z = rng.normal(size=(B, 12)).astype(np.float32)
    t = rng.normal(size=(B, n_out)).astype(np.float32)
    mask = (rng.random((B, n_out)) < (0.0 if B == 63 else 0.8)).astype(np.float32)
    p64 = OM.unflatten(flat.astype(np.float64), n_out)
    s_ref, cache = OM.forward(p64, z.astype(np.float64))
    g_ref = OM.flatten(OM.backward(p64, cache, s_ref, t.astype(np.float64),
                                   mask.astype(np.float64)))
    l_ref = OM.loss(s_ref, t.astype(np.float64), mask.astype(np.float64))
    P, Z = torch.from_numpy(flat).cuda(), torch.from_numpy(z).cuda()
    # a float32 chain of k operations is within k 2^-24 of the sum of its
    # terms' magnitudes: 12 + 64 + 64 forward, 64 + n_out back, batch sums
    tol = (12 + 64 + 64 + 64 + n_out + B) * 2.0 ** -24
    s = G.mlp_forward(P, Z, n_out).cpu().numpy()
    assert np.linalg.norm(s - s_ref) <= tol * np.linalg.norm(s_ref) + 1e-30
    args = (P, Z, torch.from_numpy(t).cuda(), torch.from_numpy(mask).cuda(), n_out)
    g, loss = G.mlp_backward(*args)
    assert np.linalg.norm(g.cpu().numpy() - g_ref) <= tol * np.linalg.norm(g_ref) + 1e-30
    assert abs(float(loss.item()) - l_ref) <= tol * l_ref
    g2, _ = G.mlp_backward(*args)
    assert torch.equal(g, g2)   # fixed summation order
