"""Power Doppler without a filtered ensemble at every K of the norm-difference path, and at frame
counts around the 4 frames it loads ahead.

The subspace is given exactly (a Gram matrix with eigenvalues 2^-i, independent of the ensemble),
the sums are FP64 and the result is rounded to FP32 once: off by at most 2^-23 of the mean power
before the projection."""
import numpy as np
import pytest

from helpers import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('K', range(18))
@pytest.mark.parametrize('nt,nv', [(18, 300), (19, 257), (20, 1), (23, 64), (130, 1000)])
def test_pd_norm(gpu, K, nt, nv):
    import torch
    rng = np.random.default_rng(1000 * nt + K)
    q, _ = np.linalg.qr(rng.standard_normal((nt, nt)) + 1j * rng.standard_normal((nt, nt)))
    G = (q * 2.0 ** -np.minimum(np.arange(nt), 30.0)) @ q.conj().T
    G = 0.5 * (G + G.conj().T)
    x = (rng.standard_normal((nt, nv)) + 1j * rng.standard_normal((nt, nv))).astype(np.complex64)
    sws = torch.empty(gpu.svd_workspace_size(nv, nt), dtype=torch.uint8, device='cuda')
    sigma = torch.empty(nt, dtype=torch.float64, device='cuda')
    k = torch.zeros(1, dtype=torch.int32, device='cuda')
    pd, pd2 = torch.full((nv,), -1.0, device='cuda'), torch.full((nv,), -1.0, device='cuda')
    gpu.svd_clutter_filter(dev(x), dev(G), sws, sigma, k, K, pd=pd)
    gpu.svd_filter_apply(dev(x), sws, k, pd=pd2)       # the rank read on the device
    assert k.item() == K
    x64, v = x.astype(np.complex128), q[:, :K]
    want = np.mean(np.abs(x64 - v.conj() @ (v.T @ x64)) ** 2, axis=0)
    power = np.mean(np.abs(x64) ** 2, axis=0)
    if K <= 16:
        assert np.all(np.abs(pd.cpu().numpy() - want) <= 2.0 ** -23 * power)
    else:   # the explicit projection, FP32 products
        assert np.all(np.abs(pd.cpu().numpy() - want) <= 1e-4 * power)
    assert torch.equal(pd, pd2)
