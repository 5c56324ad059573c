"""Demodulation at the longest records that its on-chip staging holds."""
import numpy as np
import pytest

from fqscene import get_config
from helpers import dev, gpu_das, rel_l2
from oracle import native

pytestmark = pytest.mark.gpu

C1 = get_config('c1').acq


@pytest.mark.parametrize('samples', [5084, 5085, 5086, 5087])
@pytest.mark.parametrize('frames', [1, 7, 8, 15])   # blocks of 1, 7, 8 and 8 frames
def test_longest_records(gpu, samples, frames):
    """Tolerance as for the other beamforming tests (1e-4 relative L2)."""
    acq = C1.with_(nx=6, ny=5, nz=9, dz=4e-3, n_frames=frames, nx_el=2, ny_el=2, z0=20e-3, tilts_deg=((0.0, 0.0),),
                   n_samples=samples)
    rf = np.random.default_rng(samples).standard_normal((frames, 1, 4, samples)).astype(np.float32)
    iq = gpu_das(acq, dev(rf)).cpu().numpy()
    assert rel_l2(iq, native.das_from_bb(acq, native.rf2iq(rf, acq.fc, acq.fs), 0)) < 1e-4


@pytest.mark.parametrize('frames', [1, 8])
def test_longer_records_are_refused(gpu, frames):
    acq = C1.with_(nx=6, ny=5, nz=9, n_frames=frames, nx_el=2, ny_el=2, tilts_deg=((0.0, 0.0),), n_samples=5088)
    with pytest.raises(gpu.FqError) as e:
        gpu_das(acq, dev(np.zeros((frames, 1, 4, 5088), dtype=np.float32)))
    assert e.value.status == 1   # FQ_E_INVALID
