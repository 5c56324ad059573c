"""Frequency-domain synthesis of scatterers on and next to an element's axis, where the
directivity's direction cosines are zero, rounding errors or tiny of either sign.  Same tolerance
as the other tests of this path (1e-4)."""
import math

import numpy as np
import pytest

from helpers import dev, rel_l2
from oracle import pfield

pytestmark = pytest.mark.gpu

FC, FS, C = 7.8e6, 31.25e6, 1540.0
TOL = 1e-4
TILTS = [(math.radians(a), math.radians(b)) for a, b in ((0, 0), (5, 0), (0, -4), (3, 3))]


def check(n, pitch, n_tx, pos, T, n_sub=(1, 1), width=0.9, atten=0.0):
    import torch
    import paper_2509_05464_amd as fq
    probe = fq.make_probe(n[0], n[1], pitch, pitch, FC, FS, C)
    tx = fq.make_tx(TILTS[:n_tx])
    pulse = fq.make_pulse(2.0, 5.0, 1e-3)
    w = (width * pitch, width * pitch)
    fdp = fq.make_fd_params(w, n_sub, atten, 1e-7)
    pos = np.asarray(pos, dtype=np.float32)
    amp = np.linspace(1.0, 0.6, pos.shape[0], dtype=np.float32)
    ws = torch.empty(fq.fd_workspace_size(probe, tx, pulse, fdp, T, pos.shape[0]), dtype=torch.uint8, device='cuda')
    rf = torch.empty((1, n_tx, n[0] * n[1], T), dtype=torch.float32, device='cuda')
    fq.fd_synth(probe, tx, pulse, fdp, dev(pos[None]), dev(amp), rf, ws)
    want = pfield.fd_rf(n[0], n[1], pitch, FC, FS, C, TILTS[:n_tx], pos.astype(np.float64), amp.astype(np.float64), T,
                        elem_w=w, n_sub=n_sub, atten=atten)
    assert rel_l2(rf[0].cpu().numpy(), want) < TOL


@pytest.mark.parametrize('n', [3, 7, 11, 15])
@pytest.mark.parametrize('pitch', [0.1e-3, 0.11e-3, 0.15e-3, 0.2e-3, 0.22e-3, 0.3e-3])
@pytest.mark.parametrize('n_sub', [(1, 1), (3, 3)])
@pytest.mark.parametrize('n_tx', [1, 4])   # both legs in one workgroup, and apart
def test_scatterers_on_the_axis_of_an_odd_array(gpu, n, pitch, n_sub, n_tx):
    """The centre element's position is the rounding error of its coordinate (1e-20 m), so the
    direction cosines on the axis are about 1e-20 and not zero."""
    check((n, n), pitch, n_tx, [[0.0, 0.0, 5e-3], [0.0, 0.0, 8e-3], [0.0, 0.3e-3, 6e-3]], 360, n_sub)


@pytest.mark.parametrize('n_tx', [1, 4])
@pytest.mark.parametrize('far', [12.0, 30.0, 1e4, 1e8])
def test_attenuation_of_a_far_scatterer(gpu, n_tx, far):
    """A scatterer whose amplitude falls by 8 powers of two a frequency step and metre: from 16 m
    on one step passes FP32's range.  Nothing is left of its echo, and nothing of the others' is
    lost."""
    pos = [[0.1e-3, -0.2e-3, 5e-3], [0.0, 0.0, far], [-0.3e-3, 0.1e-3, 6e-3]]
    check((4, 3), 0.3e-3, n_tx, pos, 270, atten=5.0)
    check((4, 3), 0.3e-3, n_tx, pos, 270, width=0.0, atten=5.0)


@pytest.mark.parametrize('n_tx', [1, 4])
@pytest.mark.parametrize('width', [0.0, 0.9])
@pytest.mark.parametrize('z', [10e-3, 20e-3, 40e-3])
def test_band_from_zero_under_strong_attenuation(gpu, n_tx, width, z):
    """A record of one sample has a band of 22 frequencies from 0 on, 0.7 MHz apart: the amplitude
    falls by 12, 24 or 48 powers of two a step, and the lowest frequencies are all that is left."""
    check((3, 4), 0.3e-3, n_tx, [[0.2e-3, -0.1e-3, z]], 1, width=width, atten=99.0)
