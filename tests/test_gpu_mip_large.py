"""Projections onto planes of few and many pixels, and of 2^28 and more."""
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


@pytest.mark.parametrize('pixels', [(1, 1), (3, 67), (1, 32768), (1, 32769), (524288, 1), (7, 74899), (1025, 1023)])
@pytest.mark.parametrize('n', [1, 3, 17, 70])
def test_planes_of_few_and_many_pixels(gpu, pixels, n):
    """16, 4 and 1 wavefronts for 64 pixels, with fewer planes than wavefronts; a maximum is exact."""
    import torch
    ny, nx = pixels
    vol = torch.randn((n, ny, nx), device='cuda')
    out = torch.zeros((ny, nx), device='cuda')
    gpu.mip(vol, 0, out)
    assert torch.equal(out, vol.amax(0))
    gpu.mip(vol.view(ny, n, nx), 1, out)
    assert torch.equal(out, vol.view(ny, n, nx).amax(1))
