"""How a beamforming call is split, on the host."""
import pytest

import paper_2509_05464_amd as fq


def shape(nx, ny, nz, frames, nx_el=32, spacing=1e-4):
    probe = fq.make_probe(nx_el, 2, 3e-4, 3e-4, 7.8e6, 31.25e6, 1540.0)
    grid = fq.make_grid(nx, ny, nz, 0.0, 0.0, 5e-3, spacing, spacing, spacing)
    return fq.das_launch_shape(probe, fq.make_tx([(0.0, 0.0)]), grid, frames, 512)


@pytest.mark.parametrize('frames', [8, 4400, 8400, 8800, 20000, 80000])
def test_long_recordings_of_a_plane_fit_a_launch(frames):
    """One plane of 1000 x 1000 voxels: workgroups of 1024 threads while all of a launch stay
    below 2^32 threads, else of 256."""
    fb, _, groups, _, tiles = shape(1000, 1000, 1, frames)
    threads = tiles * -(-frames // fb) * (256 if groups == 1 else 1024)
    assert threads < 2 ** 32 or (groups == 1 and tiles == 63 * 63)
    assert groups == (4 if frames <= 8400 else 1)


def test_frames_and_wide_windows():
    assert [shape(8, 8, 8, f)[0] for f in (1, 8, 9, 20, 24, 33)] == [1, 8, 5, 7, 8, 7]
    assert shape(40, 40, 24, 2, spacing=1.5e-3)[2:4] == (1, 1)
    with pytest.raises(fq.FqError):
        shape(40, 40, 24, 2, spacing=5e-3)


@pytest.mark.parametrize('nx_el,groups', [(1, 1), (8, 1), (32, 16)])
def test_few_elements_are_not_split(nx_el, groups):
    """Too few elements to pay for a split workgroup's setting up; 64 do."""
    assert shape(64, 48, 7, 33, nx_el=nx_el)[2] == groups
