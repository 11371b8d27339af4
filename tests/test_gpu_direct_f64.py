"""The float64 direct convolution where its launch changes form: one thread per
output or the matrix cores, 32 x 32, 64 x 64 or 128 x 32 outputs per workgroup,
aligned runs of four values or single ones, chunks of 32 values of the reduction
partly filled, and an infinite weight beside the image's edge.

The bound is the one of a float64 sum of R products in any order, R u sum |x w|
with u = 2^-53, with a factor of two for the reference's own sum.
"""
import numpy as np
import pytest
import torch

from gpu_helpers import to_dev
from oracle import conv as OC
from oracle import fp as OF
from paper_1905_05233_amd import workloads as WL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [
    (1, 6, 6, 2, 9), (1, 6, 6, 2, 8),          # K just over and at the one-thread form's
    (1, 8, 4, 4, 32), (1, 3, 11, 4, 33),       # 32 pixels; K one past 32
    (1, 5, 7, 7, 31), (1, 9, 9, 32, 64),       # odd C; R = 288, nine whole chunks
    (3, 51, 57, 5, 65),                        # 64 x 64 blocks, ragged in both
    (2, 97, 91, 12, 20),                       # 128 x 32 blocks
], ids=str)
def test_direct_f64_launch_forms(shape, dtype):
    from paper_1905_05233_amd.layer_ops import direct_conv_f64
    N, H, W, C, K = shape
    x, w = WL.draw_inputs(N, H, W, C, K, "uniform", seed=C + K)
    x, w = OF.to_dtype(x, dtype), OF.to_dtype(w, dtype)
    y = direct_conv_f64(to_dev(x, dtype), to_dev(w, dtype)).cpu().numpy()
    ref = OC.direct_f64(x, w)
    mag = OC.direct_f64(np.abs(x), np.abs(w))
    assert np.all(np.abs(y - ref) <= 2 * 2.0 ** -53 * (9 * C) * mag)


@pytest.mark.parametrize("C,K", [(4, 40), (3, 12)])
def test_direct_f64_taps_outside_the_image_do_not_meet_an_infinite_weight(C, K):
    from paper_1905_05233_amd.layer_ops import direct_conv_f64
    x = torch.ones((1, 9, 10, C), device="cuda")
    w = torch.full((K, 3, 3, C), 0.5, device="cuda")
    w[5, 0, 1, 1] = float("inf")               # the tap above the pixel
    y = direct_conv_f64(x, w)[0]
    assert bool(torch.isfinite(y[0]).all())    # the first row has no pixel above
    assert bool(torch.isinf(y[1:, :, 5]).all())
    other = [k for k in range(K) if k != 5]
    assert bool((y[1:-1, 1:-1][:, :, other] == 4.5 * C).all())
