"""Delay-and-sum over its launch shapes against the oracle: every number of frames of a block
and of transmits of a pass that a kernel is compiled for, both interpolations, workgroups
of one, four and sixteen element groups (with fewer elements than groups, and numbers that
they do not divide), grids smaller than a tile, odd records, windows beyond 248 rows.

Tolerance as for the other beamforming tests (1e-4 relative L2)."""
import numpy as np
import pytest

from fqscene import get_config
from helpers import dev, gpu_das, rel_l2
from oracle import native

pytestmark = pytest.mark.gpu

C1 = get_config('c1').acq
TILTS = tuple((float(a), float(b)) for a, b in np.random.default_rng(0).uniform(-6, 6, (11, 2)))


def check(acq, interp, seed):
    rng = np.random.default_rng(seed)
    rf = rng.standard_normal((acq.n_frames, acq.n_angles, acq.n_elem, acq.n_samples)).astype(np.float32)
    iq = gpu_das(acq, dev(rf), interp).cpu().numpy()
    want = native.das_from_bb(acq, native.rf2iq(rf, acq.fc, acq.fs), interp)
    assert rel_l2(iq, want) < 1e-4


@pytest.mark.parametrize('frames', [1, 2, 3, 4, 5, 6, 7, 8, 9])
@pytest.mark.parametrize('grid', [(7, 5, 3), (40, 40, 17), (64, 64, 70)])   # 16, 4 and 1 groups
def test_frames(gpu, frames, grid):
    nx, ny, nz = grid
    n = 5 if grid[0] < 64 else 3
    acq = C1.with_(nx=nx, ny=ny, nz=nz, n_frames=frames, nx_el=n, ny_el=7, z0=6e-3, tilts_deg=TILTS[:2], n_samples=767)
    check(acq, frames % 2, frames)


@pytest.mark.parametrize('angles', [1, 2, 3, 4, 5, 6, 7, 8, 9, 11])
@pytest.mark.parametrize('grid', [(9, 6, 5), (33, 20, 35)])
@pytest.mark.parametrize('elems', [(2, 3), (6, 11)])
def test_transmits(gpu, angles, grid, elems):
    nx, ny, nz = grid
    acq = C1.with_(nx=nx, ny=ny, nz=nz, n_frames=3, nx_el=elems[0], ny_el=elems[1], z0=6e-3, tilts_deg=TILTS[:angles])
    check(acq, angles % 2, angles)


@pytest.mark.parametrize('interp', [0, 1])
def test_wide_windows(gpu, interp):
    acq = C1.with_(nx=40, ny=40, nz=24, dx=1.5e-3, dy=1.5e-3, dz=1.5e-3, n_frames=2, nx_el=2,
                   ny_el=3, z0=6e-3, tilts_deg=TILTS[:3], n_samples=3001)
    check(acq, interp, 5)
