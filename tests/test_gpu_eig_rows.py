"""The tridiagonalisation of one launch a step (above 128 frames) at the edges of its 64-column
chunks, against LAPACK.

Householder reductions and the methods on T are backward stable: eigenvalues are off by a small
multiple of n 2^-53 ||G||, taken as 20.  G is rank-deficient in one case (whole zero columns on
the way), diagonal in another (no reflector at all)."""
import numpy as np
import pytest

from helpers import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('kind', ['full', 'rank3', 'diagonal'])
@pytest.mark.parametrize('n', [128, 129, 191, 192, 193, 208, 209, 256, 257, 449, 512])
def test_eigenvalues(gpu, n, kind):
    import torch
    rng = np.random.default_rng(n)
    x = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    if kind == 'diagonal':
        G = np.diag(rng.uniform(0.0, 5.0, n)).astype(np.complex128)
    else:
        x = x[:, :3] if kind == 'rank3' else x
        G = x @ x.conj().T
        G = 0.5 * (G + G.conj().T)
    want = np.linalg.eigvalsh(G)[::-1]
    sws = torch.full((gpu.svd_workspace_size(n, n) + 4096,), 0xff, dtype=torch.uint8, device='cuda')
    sigma = [torch.empty(n, dtype=torch.float64, device='cuda') for _ in range(2)]
    k = torch.zeros(1, dtype=torch.int32, device='cuda')
    status = torch.full((1,), -1, dtype=torch.int32, device='cuda')
    iq, pd = dev(np.eye(n, dtype=np.complex64)), torch.empty(n, device='cuda')
    for s in sigma:
        gpu.svd_clutter_filter(iq, dev(G), sws[:-4096], s, k, 2, pd=pd, status=status)
        assert status.item() == 0
    assert torch.equal(sigma[0], sigma[1])
    assert bool((sws[-4096:] == 0xff).all())
    got = sigma[0].cpu().numpy() ** 2
    assert np.abs(got - np.maximum(want, 0.0)).max() < 20 * n * 2.0 ** -53 * want[0]


@pytest.mark.parametrize('n', [2, 3, 7, 8, 9, 10, 16, 17, 18, 63, 127, 255, 512])
def test_leading_projector(gpu, n):
    """Inverse iteration in batches of 8 rows and the back-transformation 4 reflectors ahead at
    the ends of both.  Eigenvalues 2^-i: the leading projector is off by a few n 2^-53 / gap, and
    the filter applied to the identity adds FP32 products of K <= 3 terms: 1e-5 covers both."""
    import torch
    rng = np.random.default_rng(n)
    q, _ = np.linalg.qr(rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n)))
    G = (q * 2.0 ** -np.minimum(np.arange(n), 40.0)) @ q.conj().T
    G = 0.5 * (G + G.conj().T)
    K = min(3, n - 1)
    sws = torch.full((gpu.svd_workspace_size(n, n),), 0xff, dtype=torch.uint8, device='cuda')
    sigma = torch.empty(n, dtype=torch.float64, device='cuda')
    k = torch.zeros(1, dtype=torch.int32, device='cuda')
    status = torch.full((1,), -1, dtype=torch.int32, device='cuda')
    filt, pd = torch.empty(n, n, dtype=torch.complex64, device='cuda'), torch.empty(n, device='cuda')
    gpu.svd_clutter_filter(dev(np.eye(n, dtype=np.complex64)), dev(G), sws, sigma, k, K, iq_filt=filt, pd=pd, status=status)
    assert status.item() == 0 and k.item() == K
    v = q[:, :K]
    assert np.abs(filt.cpu().numpy() - (np.eye(n) - v.conj() @ v.T)).max() < 1e-5
