"""Orthogonalisation of clustered eigenvectors: Gram matrices with repeated eigenvalues,
whose leading subspace (cut between two clusters) has a unique projector.

The filter applied to the identity returns I - conj(V) V^T.  Its FP32 products of
|V| <= 1 sum K <= 64 terms: 64 * 2^-23 < 1e-5 per entry."""
import numpy as np
import pytest

from helpers import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('n', [24, 64, 65, 130, 257])
@pytest.mark.parametrize('sizes', [(1, 7, 4), (12,), (3, 1, 1, 59)])
def test_clustered_subspace(gpu, n, sizes):
    import torch
    K = sum(sizes)
    if K >= n:
        pytest.skip('the cluster fills the space')
    rng = np.random.default_rng(n + K)
    q, _ = np.linalg.qr(rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n)))
    lam = np.concatenate([np.full(m, 100.0 / (i + 1)) for i, m in enumerate(sizes)] + [np.linspace(1.0, 0.1, n - K)])
    G = (q * lam) @ q.conj().T
    G = 0.5 * (G + G.conj().T)
    iq = dev(np.eye(n, dtype=np.complex64))
    sws = torch.empty(gpu.svd_workspace_size(n, n), dtype=torch.uint8, device='cuda')
    sigma = torch.empty(n, dtype=torch.float64, device='cuda')
    k = torch.zeros(1, dtype=torch.int32, device='cuda')
    status = torch.full((1,), -1, dtype=torch.int32, device='cuda')
    filt = torch.empty(n, n, dtype=torch.complex64, device='cuda')
    pd = torch.empty(n, device='cuda')
    gpu.svd_clutter_filter(iq, dev(G), sws, sigma, k, K, iq_filt=filt, pd=pd, status=status)
    assert status.item() == 0 and k.item() == K
    v = q[:, :K]
    want = np.eye(n) - v.conj() @ v.T
    assert np.abs(filt.cpu().numpy() - want).max() < 1e-5
