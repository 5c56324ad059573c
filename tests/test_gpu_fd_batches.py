"""Frequency-domain synthesis over its launch shapes: every number of transmits a kernel is
compiled for and one that takes two groups, a band that ends inside a chunk, frames in one
batch or several, echo splits, scatterers in blocks.  Same tolerance as the other tests of
this path (1e-4, from 4 frequency steps and the phase anchors)."""
import math

import numpy as np
import pytest

from helpers import rel_l2
from test_gpu_fd import TOL, gpu_fd, oracle_fd, scatterers

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('n_tx', [1, 2, 3, 4, 5, 6, 7, 8, 9, 10])
@pytest.mark.parametrize('block', [None, 100000])
def test_transmit_counts_and_batches(gpu, n_tx, block):
    rng = np.random.default_rng(n_tx)
    tilts = [(math.radians(a), math.radians(b)) for a, b in rng.uniform(-8, 8, (n_tx, 2))]
    pos, amp = scatterers(70, rng, F=4)
    kw = dict(elem_w=(0.27e-3, 0.2e-3), n_sub=(2, 1), atten=0.7)
    got = gpu_fd(5, 3, tilts, pos, amp, 301, block=block, floor=1e-5, **kw)
    for f in (0, 3):
        want = oracle_fd(5, 3, tilts, pos[f], amp, 301, **kw)
        assert rel_l2(got[f], want) < TOL + 1e-4   # the band's floor cuts 1e-5 of the peak on both sides


@pytest.mark.parametrize('floor', [0.9, 0.3, 1e-3])
def test_short_bands_in_the_smallest_workspace(gpu, floor):
    """One to a few dozen frequencies, 300 scatterers in blocks of 256, nine transmits: the
    smallest workspace gives what a large one does, up to the order of FP32 sums."""
    rng = np.random.default_rng(8)
    tilts = [(math.radians(a), 0.0) for a in np.linspace(-8, 8, 9)]
    pos, amp = scatterers(300, rng, F=3)
    small = gpu_fd(4, 4, tilts, pos, amp, 300, elem_w=(0.2e-3, 0.2e-3), floor=floor, block=256)
    large = gpu_fd(4, 4, tilts, pos, amp, 300, elem_w=(0.2e-3, 0.2e-3), floor=floor, block=5000)
    assert rel_l2(small, large) < 1e-6


@pytest.mark.parametrize('elems', [(1, 1), (8, 8), (13, 5), (16, 20), (23, 22), (23, 23)])   # one leg pair up to 512
@pytest.mark.parametrize('n_tx', [1, 2, 3])
def test_both_legs_in_one_workgroup(gpu, elems, n_tx):
    """Element counts around the wavefront and the largest workgroup, 9 scatterers (one past a
    group of four twice) with one behind the array of infinite amplitude."""
    rng = np.random.default_rng(elems[0] + n_tx)
    tilts = [(math.radians(a), math.radians(b)) for a, b in rng.uniform(-8, 8, (n_tx, 2))]
    pos, amp = scatterers(9, rng, F=2)
    behind = np.concatenate([pos, np.full((2, 1, 3), -2e-3)], axis=1)
    got = gpu_fd(elems[0], elems[1], tilts, behind, np.concatenate([amp, [np.inf]]), 420, elem_w=(0.2e-3, 0.27e-3))
    for f in range(2):
        want = oracle_fd(elems[0], elems[1], tilts, pos[f], amp, 420, elem_w=(0.2e-3, 0.27e-3))
        assert rel_l2(got[f], want) < TOL
