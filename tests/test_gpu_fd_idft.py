"""The inverse transform of the frequency-domain synthesis with 8, 4, 2 and 1 elements a workgroup
(chosen by the number of elements, transmits and frames of a launch), and bands past the length
that 8 elements' spectra fit on chip for.  Same tolerance as the other tests of this path."""
import math

import numpy as np
import pytest

from helpers import rel_l2
from test_gpu_fd import TOL, gpu_fd, oracle_fd, scatterers

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('elems', [(1, 1), (13, 5), (24, 16)])
@pytest.mark.parametrize('frames', [1, 2, 30])   # 3 transmits: 8 elements from 2731 elements x frames on
def test_elements_of_a_workgroup(gpu, elems, frames):
    rng = np.random.default_rng(frames)
    tilts = [(math.radians(a), math.radians(b)) for a, b in rng.uniform(-8, 8, (3, 2))]
    pos, amp = scatterers(3, rng, F=frames)
    got = gpu_fd(elems[0], elems[1], tilts, pos, amp, 401, block=20000)
    for f in (0, frames - 1):
        assert rel_l2(got[f], oracle_fd(elems[0], elems[1], tilts, pos[f], amp, 401)) < TOL


@pytest.mark.parametrize('samples', [2399, 2400, 5000])   # about 1024 frequencies, and 2160
def test_long_bands(gpu, samples):
    rng = np.random.default_rng(1)
    pos, amp = scatterers(2, rng)
    got = gpu_fd(3, 1, [(0.0, 0.0)], pos, amp, samples)[0]
    assert rel_l2(got, oracle_fd(3, 1, [(0.0, 0.0)], pos[0], amp, samples)) < TOL
