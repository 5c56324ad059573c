"""The clutter projection over several voxel blocks per workgroup (above 65536 voxels), with odd
voxel counts, frame counts around its 16-frame batches, and an ensemble that is stored past the
caches (more than 256 MB, whole lines).

FP32 sums of n_t and 2 K products of values whose sizes Cauchy-Schwarz bounds by the voxel's norm:
off by at most (n_t + 2 K) 2^-23 of it.  The subspace itself is determined by G (of unit norm,
rounded to FP64) to a small multiple, taken as 20, of n_t 2^-53 / gap (Davis-Kahan)."""
import numpy as np
import pytest

from helpers import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('nt,nv,K', [(16, 65537, 3), (17, 131072 + 48, 16), (47, 70001, 17), (33, 66000, 33 - 1),
                                     (100, 65536 + 15, 64), (64, (1 << 19) + 16, 5), (400, 3000, 40)])
def test_projection(gpu, nt, nv, K):
    import torch
    rng = np.random.default_rng(nt)
    q, _ = np.linalg.qr(rng.standard_normal((nt, nt)) + 1j * rng.standard_normal((nt, nt)))
    lam = 2.0 ** -(np.arange(nt) * 40.0 / nt)
    G = (q * lam) @ q.conj().T
    G = 0.5 * (G + G.conj().T)
    x = torch.randn(nt, nv, dtype=torch.complex64, device='cuda', generator=torch.Generator('cuda').manual_seed(nt))
    sws = torch.empty(gpu.svd_workspace_size(nv, nt), dtype=torch.uint8, device='cuda')
    sigma = torch.empty(nt, dtype=torch.float64, device='cuda')
    k = torch.zeros(1, dtype=torch.int32, device='cuda')
    filt, pd = torch.full_like(x, float('nan')), torch.full((nv,), float('nan'), device='cuda')
    gpu.svd_clutter_filter(x, dev(G), sws, sigma, k, K, iq_filt=filt, pd=pd)
    assert k.item() == K and not bool(torch.isnan(torch.view_as_real(filt)).any()) and not bool(torch.isnan(pd).any())
    at = np.unique(np.concatenate([np.arange(min(nv, 200)), np.arange(max(nv - 200, 0), nv), rng.integers(0, nv, 500)]))
    got, gpd = filt[:, at].cpu().numpy(), pd[at].cpu().numpy()
    x64, v = x[:, at].cpu().numpy().astype(np.complex128), q[:, :K]
    want = x64 - v.conj() @ (v.T @ x64)
    norm = np.linalg.norm(x64, axis=0)
    gap = lam[K - 1] - lam[K] if K < nt else 1.0
    tol = (nt + 2 * K) * 2.0 ** -23 + 20 * nt * 2.0 ** -53 / gap
    assert np.all(np.abs(got - want) <= tol * norm)
    np.testing.assert_allclose(gpd, np.mean(np.abs(got.astype(np.complex128)) ** 2, axis=0), rtol=(nt + 4) * 2.0 ** -23)
