"""Gram matrix at the edges of its stages, tiles and voxel ranges: one tile shared by four
wavefronts (up to 32 frames) or several, stages cut short, rows on 8-byte boundaries (odd
voxel counts), few and many voxel ranges.

Per entry, relative to sqrt(G_ii G_jj) (Cauchy-Schwarz bounds sum |x||y| by it): FP32 sums of
at most 64 voxels x 2 products are off by at most 128 * 2^-24; the two-term split adds
2 * 2^-17 and has 4 times the products."""
import numpy as np
import pytest

from helpers import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('mode,tol', [(0, 128 * 2.0 ** -24), (3, 2.0 ** -16 + 512 * 2.0 ** -24)])
@pytest.mark.parametrize('nt', [1, 20, 32, 33, 100])
@pytest.mark.parametrize('nv', [1, 6, 63, 64, 255, 256, 257, 2050, 20001, 70000])
def test_gram_edges(gpu, mode, tol, nt, nv):
    import torch
    rng = np.random.default_rng(nt * 100003 + nv)
    x = (rng.standard_normal((nt, nv)) + 1j * rng.standard_normal((nt, nv))).astype(np.complex64)
    x *= np.exp(rng.standard_normal((nt, 1))).astype(np.float32)
    g = torch.empty(nt, nt, dtype=torch.complex128, device='cuda')
    ws = torch.full((gpu.gram_workspace_size(nv, nt, mode),), 0xff, dtype=torch.uint8, device='cuda')
    gpu.casorati_gram(dev(x), g, ws, mode)
    x64 = x.astype(np.complex128)
    want = x64.conj() @ x64.T
    d = np.sqrt(np.diagonal(want).real)
    got = g.cpu().numpy()
    assert np.max(np.abs(got - want) / np.outer(d, d)) < tol
    np.testing.assert_array_equal(got, got.conj().T)


@pytest.mark.parametrize('nt', [1, 20, 33, 100])
@pytest.mark.parametrize('nv', [1, 257, 4096, 20001, 70000])
def test_gram_smallest_workspace(gpu, nt, nv):
    """A workspace of one partial sum per 2048 voxels, fewer than the voxel ranges that fill
    the chip, is taken, nothing is written past it, and a byte less is refused."""
    import torch
    rng = np.random.default_rng(nt * 100003 + nv)
    x = (rng.standard_normal((nt, nv)) + 1j * rng.standard_normal((nt, nv))).astype(np.complex64)
    nb = -(-nt // 32)
    splits = -(-(-(-nv // 2048)) // 8) * 8
    least = splits * nb * (nb + 1) // 2 * 32 * 32 * 16
    assert least <= gpu.gram_workspace_size(nv, nt, 0)
    ws = torch.full((least + 4096,), 0x5a, dtype=torch.uint8, device='cuda')
    g = torch.empty(nt, nt, dtype=torch.complex128, device='cuda')
    gpu.casorati_gram(dev(x), g, ws[:least], 0)
    assert bool((ws[least:] == 0x5a).all())
    x64 = x.astype(np.complex128)
    want = x64.conj() @ x64.T
    d = np.sqrt(np.diagonal(want).real)
    assert np.max(np.abs(g.cpu().numpy() - want) / np.outer(d, d)) < 128 * 2.0 ** -24
    with pytest.raises(RuntimeError, match='workspace too small'):
        gpu.casorati_gram(dev(x), g, ws[:least - 1], 0)
