"""Image quality over the shapes of its tiles: images of one to a few rows or columns of window
positions (as tall or wide tiles, or every position by itself), and tiles that the image does
not fill.  Tolerances as for the other tests of the metrics (FP64 sums in another order)."""
import numpy as np
import pytest

from oracle import metrics
from test_gpu_metrics import gpu_quality

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('shape', [(11, 12), (12, 11), (11, 358), (11, 360), (11, 2000), (13, 1000), (14, 1000), (16, 400),
                                   (70, 11), (1000, 11), (3841, 11), (1000, 14), (400, 16), (64, 70), (65, 71), (70, 69),
                                   (19, 300), (300, 19), (63, 200), (200, 69), (131, 143)])
def test_shapes(gpu, shape):
    rng = np.random.default_rng(shape[0] * 5000 + shape[1])
    a = rng.random(shape).astype(np.float32)
    b = np.clip(a + 0.2 * rng.standard_normal(shape), 0, 1).astype(np.float32)
    mse, psnr, ssim = gpu_quality(a, b)
    assert abs(mse - metrics.mse(a, b)) <= 1e-12 * metrics.mse(a, b)
    assert abs(psnr - metrics.psnr(a, b)) <= 1e-12 * abs(metrics.psnr(a, b))
    assert abs(ssim - metrics.ssim(a, b)) <= 1e-12
