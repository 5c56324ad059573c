"""Projections onto planes of 2^28 pixels and more."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('plane', [0, 1])   # over z, over y
@pytest.mark.parametrize('rows', [16384, 16385])
def test_large_planes(gpu, plane, rows):
    import torch
    vol = torch.rand((1, rows, 16384) if plane == 0 else (rows, 1, 16384), device='cuda')
    out = torch.zeros((rows, 16384), device='cuda')
    gpu.mip(vol, plane, out)
    assert torch.equal(out, vol.view(rows, 16384))
