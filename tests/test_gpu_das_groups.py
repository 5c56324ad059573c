"""Delay-and-sum with 1, 4 and 16 element groups a workgroup for every block length and both
interpolations, each case checked to take the launch it is meant for, against the oracle
(tolerance as for the other beamforming tests, 1e-4 relative L2)."""
import numpy as np
import pytest

from fqscene import get_config
from helpers import dev, gpu_das, rel_l2, structs
from oracle import native

pytestmark = pytest.mark.gpu

C1 = get_config('c1').acq
TILTS = tuple((float(a), float(b)) for a, b in np.random.default_rng(0).uniform(-6, 6, (9, 2)))


def check(gpu, acq, interp, frames, groups):
    probe, tx, grid, _ = structs(acq)
    assert gpu.das_launch_shape(probe, tx, grid, acq.n_frames, acq.n_samples, interp)[::2][:2] == (frames, groups)
    rf = np.random.default_rng(1).standard_normal((acq.n_frames, acq.n_angles, acq.n_elem, acq.n_samples)).astype(np.float32)
    iq = gpu_das(acq, dev(rf), interp).cpu().numpy()
    assert rel_l2(iq, native.das_from_bb(acq, native.rf2iq(rf, acq.fc, acq.fs), interp)) < 1e-4


@pytest.mark.parametrize('frames', [1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize('interp', [0, 1])
@pytest.mark.parametrize('groups,grid', [(16, (7, 5, 3)), (4, (48, 40, 20)), (1, (64, 64, 70))])
def test_block_lengths(gpu, frames, interp, groups, grid):
    nx, ny, nz = grid
    el = (11, 6) if groups == 4 else (3, 3)   # 4 does not divide 66; fewer elements than 16 groups
    acq = C1.with_(nx=nx, ny=ny, nz=nz, n_frames=frames, nx_el=el[0], ny_el=el[1], z0=6e-3, tilts_deg=TILTS[:5],
                   n_samples=767)
    check(gpu, acq, interp, frames, groups)


@pytest.mark.parametrize('angles', [1, 2, 3, 4, 5, 6, 7, 8, 9])
@pytest.mark.parametrize('interp', [0, 1])
@pytest.mark.parametrize('frames', [1, 8])
def test_transmits_over_four_groups(gpu, angles, interp, frames):
    acq = C1.with_(nx=40, ny=40, nz=40, n_frames=frames, nx_el=11, ny_el=6, z0=6e-3, tilts_deg=TILTS[:angles],
                   n_samples=766)
    check(gpu, acq, interp, frames, 4)
