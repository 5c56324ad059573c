"""Gathering series of more frames than a launch has block rows for."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('n_t', [1, 8, 9, 524280, 524281, 524297, 1048569])
def test_frames(gpu, n_t):
    import torch
    src = torch.randn((2, n_t, 3), dtype=torch.complex64, device='cuda')
    idx = torch.tensor([5, 0, 2, 3], device='cuda')
    dst = torch.zeros((n_t, 4), dtype=torch.complex64, device='cuda')
    gpu.lcf_gather(src, idx, dst)
    assert torch.equal(dst, torch.stack([src[1, :, 2], src[0, :, 0], src[0, :, 2], src[1, :, 0]], 1))
