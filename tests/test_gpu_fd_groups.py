"""The legs of the frequency-domain synthesis apart (more than 3 transmits or 512 elements) at the
edges of their shapes: elements that four wavefronts share unevenly on transmit, and echo
workgroups of four, two and one scatterer groups, with fewer scatterers than groups, a block
and one more, and scatterers in blocks.  Same tolerance as the other tests of this path."""
import math

import numpy as np
import pytest

from helpers import rel_l2
from test_gpu_fd import TOL, gpu_fd, oracle_fd, scatterers

pytestmark = pytest.mark.gpu

TILTS = [(math.radians(a), math.radians(b)) for a, b in np.random.default_rng(2).uniform(-8, 8, (9, 2))]


@pytest.mark.parametrize('elems', [(1, 1), (3, 1), (5, 1), (9, 7), (8, 8), (13, 5), (16, 8), (43, 3), (12, 16), (17, 16)])
@pytest.mark.parametrize('n_tx', [4, 9])
@pytest.mark.parametrize('n', [1, 3, 33])
def test_elements_and_scatterers(gpu, elems, n_tx, n):
    rng = np.random.default_rng(n)
    pos, amp = scatterers(n, rng)
    kw = dict(elem_w=(0.2e-3, 0.27e-3))
    got = gpu_fd(elems[0], elems[1], TILTS[:n_tx], pos, amp, 420, **kw)[0]
    assert rel_l2(got, oracle_fd(elems[0], elems[1], TILTS[:n_tx], pos[0], amp, 420, **kw)) < TOL


def test_scatterer_blocks_over_groups(gpu):
    """600 scatterers in blocks of 256 give what one block does, up to the order of FP32 sums."""
    pos, amp = scatterers(600, np.random.default_rng(3))
    part = gpu_fd(7, 7, TILTS[:5], pos, amp, 400, block=256)
    assert rel_l2(part, gpu_fd(7, 7, TILTS[:5], pos, amp, 400)) < 1e-6
