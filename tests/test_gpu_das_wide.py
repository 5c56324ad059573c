"""Delays of windows beyond 248 rows carry the fraction bits of narrow ones.

One element and one transmit; a constant record demodulated at 0.45 of the sampling rate, so
that neighbouring samples are almost opposite (|b| = 1, steps of 2) and the interpolation shows
an error of its fraction twice over.  A voxel of a coarse grid (wide window) and the same voxel
alone (narrow) go through the same arithmetic: with 24 fraction bits they differ by the rounding
of the voxel's coordinates alone, 2^-24 of a sample at a rounding boundary, 2^-23 in the sum;
with 22 bits by up to 2 * 2^-23 of a sample, 2^-21 in the sum (5e-7)."""
import numpy as np
import pytest

from helpers import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('interp', [0, 1])
def test_wide_and_narrow_windows_agree(gpu, interp):
    import torch
    probe = gpu.make_probe(1, 1, 3e-4, 3e-4, 14.0625e6, 31.25e6, 1540.0)
    tx = gpu.make_tx([(0.05, -0.03)])
    n, d, z0, T = (40, 40, 24), 1.5e-3, 6e-3, 3001
    rf = dev(np.ones((1, 1, 1, T), dtype=np.float32))
    ws = torch.empty(gpu.das_workspace_size(probe, tx, 1, T), dtype=torch.uint8, device='cuda')

    def beamform(grid, count):
        iq = torch.empty((1, count), dtype=torch.complex64, device='cuda')
        gpu.das_beamform(probe, tx, grid, rf, iq, ws, interp)
        return iq.cpu().numpy()[0]

    grid = gpu.make_grid(*n, 0.0, 0.0, z0, d, d, d)
    assert gpu.das_launch_shape(probe, tx, grid, 1, T, interp)[3] == 1
    wide = beamform(grid, n[0] * n[1] * n[2]).reshape(n[2], n[1], n[0])
    worst = 0.0
    for ix, iy, iz in np.random.default_rng(0).integers(0, (40, 40, 12), (300, 3)):
        iz *= 2   # (the second voxel of a pair takes its transmit delay and phase from the first)
        one = gpu.make_grid(1, 1, 1, ix * d, iy * d, z0 + iz * d, d, d, d)
        assert gpu.das_launch_shape(probe, tx, one, 1, T, interp)[3] == 0
        worst = max(worst, abs(beamform(one, 1)[0] - wide[iz, iy, ix]))
    print('largest difference', worst)
    assert worst < 2.0 ** -23
