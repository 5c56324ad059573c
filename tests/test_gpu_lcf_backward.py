"""Gradient of the learned filter at the sizes where the tiled backward pass can go wrong:
series shorter than a tile's taps, one frame more or less than a tile, the longest series,
fewer series than wavefronts and more than one round of them.

Tolerance: a BF16 rounding that falls the other way moves one activation or dz by 2^-8 of
itself in one of three layers; with few series nothing averages it out, so 3 * 2^-8."""
import numpy as np
import pytest

from helpers import dev, rel_l2
from oracle import lcf as olcf
from test_gpu_lcf import _series, _weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('T,n', [(1, 5), (5, 3), (31, 6), (32, 2), (33, 4), (64, 1030), (97, 9), (256, 5), (257, 3),
                                 (512, 2), (12, 4100)])
def test_gradient_at_tile_edges(gpu, T, n):
    import torch
    w, wb = _weights(11)
    mix, blood = _series(12, n, T)
    x, tgt = dev(np.ascontiguousarray(mix.T)), dev(np.ascontiguousarray(blood.T))
    wt, wbt = dev(w), dev(wb.view(np.int16))
    act = torch.full((gpu.lcf_act_size(n, T),), 0xff, dtype=torch.uint8, device='cuda')   # NaN where unwritten
    gpu.lcf_forward(wt, wbt, x, 1e-30, act.view(torch.int16), None, None)
    grad = torch.empty(gpu.LCF_N_PARAM, dtype=torch.float32, device='cuda')
    loss = torch.empty(1, dtype=torch.float32, device='cuda')
    gpu.lcf_backward(wt, wbt, x, tgt, act.view(torch.int16), grad, loss, 1e-30)
    xo, s = olcf.normalise(mix.astype(np.complex128))
    yt = np.stack([blood.real, blood.imag], axis=1) / s[:, None, None]
    l16, g16 = olcf.loss_and_grad(w.astype(np.float64), xo, yt, bf16=True)
    print('grad', rel_l2(grad.cpu().numpy(), g16), 'loss', loss.item() / l16 - 1)
    assert rel_l2(grad.cpu().numpy(), g16) < 3 * 2 ** -8
    assert abs(loss.item() / l16 - 1) < 3 * 2 ** -8
