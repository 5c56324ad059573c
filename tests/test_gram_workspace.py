"""Sizes of the Gram matrix's workspace, which need no device."""
import pytest

import paper_2509_05464_amd as fq


@pytest.mark.parametrize('nt', [1, 20, 33, 100, 200, 400, 512])
def test_gram_workspace_covers_smaller_calls(nt):
    """A workspace of a larger call holds one partial sum per 2048 voxels of any smaller one,
    which is what the smaller call needs at least."""
    nb = -(-nt // 32)
    tile = nb * (nb + 1) // 2 * 32 * 32 * 16
    for nv in list(range(1, 4200, 173)) + [9000, 18432, 18500, 65536, 262144, 589824, 590000, 599186, 600000]:
        splits = -(-(-(-nv // 2048)) // 8) * 8
        assert fq.gram_workspace_size(nv, nt, 0) >= splits * tile
