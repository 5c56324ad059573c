"""Voxels whose delays lie past the record, just so or far."""
import numpy as np
import pytest

from fqscene import get_config
from helpers import dev, gpu_das, rel_l2
from oracle import native

pytestmark = pytest.mark.gpu

C1 = get_config('c1').acq


@pytest.mark.parametrize('frames', [1, 3, 8])
@pytest.mark.parametrize('wraps', [1, 2])
def test_row_offsets_beyond_32_bits(gpu, frames, wraps):
    """A delay of 2^32 bytes of rows and a few rows more is outside the record like any other."""
    rows = wraps * 2 ** 32 / (8 * frames) + 100
    acq = C1.with_(nx=3, ny=2, nz=5, n_frames=frames, nx_el=2, ny_el=2, tilts_deg=((0.0, 0.0),), n_samples=600,
                   z0=0.5 * rows * C1.c / C1.fs)
    rf = np.random.default_rng(0).standard_normal((frames, 1, 4, 600)).astype(np.float32)
    assert not gpu_das(acq, dev(rf)).cpu().numpy().any()


@pytest.mark.parametrize('nx', [3, 40])
@pytest.mark.parametrize('interp', [0, 1])
@pytest.mark.parametrize('samples', [300, 301])
def test_grid_across_the_end_of_the_record(gpu, nx, interp, samples):
    """Planes a third of a row apart around the depth of the last sample (its last taps, and the
    first plane without any); tolerance as for the other beamforming tests."""
    dz = C1.c / C1.fs / 6
    acq = C1.with_(nx=nx, ny=4, nz=61, dz=dz, n_frames=3, nx_el=3, ny_el=2, tilts_deg=((0.0, 0.0), (4.0, -3.0)),
                   n_samples=samples, z0=0.5 * samples * C1.c / C1.fs - 40 * dz)
    rf = np.random.default_rng(1).standard_normal((3, 2, 6, samples)).astype(np.float32)
    iq = gpu_das(acq, dev(rf), interp).cpu().numpy()
    want = native.das_from_bb(acq, native.rf2iq(rf, acq.fc, acq.fs), interp)
    assert rel_l2(iq, want) < 1e-4
    assert np.array_equal(iq.any(axis=0), want.any(axis=0))
