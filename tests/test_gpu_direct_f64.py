"""The float64 direct convolution where its launch changes form: one thread per
output or the matrix cores, 32 x 32, 64 x 64 or 128 x 32 outputs per workgroup,
aligned runs of four values or single ones, chunks of 32 values of the reduction
partly filled, 3x3 and 1x3 kernels, and infinities and NaN beside the image's
edge.  Each shape names the form that it selects; tests/test_launch_split.py holds
the rule to it on the CPU.

The bound is the one of a float64 sum of R products in any order, R u sum |x w|
with u = 2^-53, with a factor of two for the reference's own sum.
"""
import numpy as np
import pytest
import torch

from gpu_helpers import TORCH, to_dev
from oracle import conv as OC
from oracle import fp as OF
from paper_1905_05233_amd import workloads as WL

pytestmark = pytest.mark.gpu

CUS = 256   # compute units of an MI355X: the rule counts blocks against them
SHAPES = [
    ((1, 6, 6, 2, 8), "one thread per output"),
    ((1, 6, 6, 2, 9), "32 x 32"),              # K just over the one-thread form's
    ((1, 8, 4, 4, 32), "32 x 32"),             # 32 pixels
    ((1, 3, 11, 4, 33), "32 x 32"),            # a pixel and a channel past 32
    ((1, 5, 7, 7, 31), "32 x 32"),             # odd C
    ((1, 9, 9, 32, 64), "32 x 32"),            # R = 288, nine whole chunks
    ((1, 64, 127, 4, 64), "32 x 32"),          # 127 blocks of 64 x 64
    ((1, 64, 128, 4, 64), "64 x 64"),          # 128 of them
    ((3, 51, 57, 5, 65), "64 x 64"),           # ragged in both, single values
    ((3, 51, 57, 12, 68), "64 x 64"),          # ragged in both, runs of four
    ((2, 56, 56, 128, 128), "64 x 64"),        # whole blocks, 36 chunks
    ((2, 97, 91, 12, 20), "128 x 32"),
    ((2, 97, 91, 13, 20), "128 x 32"),
]
SHAPES_1D = [
    ((2, 1, 90, 6, 12), "32 x 32"),
    ((2, 1, 90, 8, 40), "32 x 32"),
    ((5, 1, 1701, 8, 70), "64 x 64"),
    ((5, 1, 1701, 7, 70), "64 x 64"),
    ((4, 1, 4101, 12, 20), "128 x 32"),
    ((4, 1, 4101, 7, 20), "128 x 32"),
]
SPECIAL = [
    ((1, 9, 10, 4, 6), "one thread per output"),
    ((1, 9, 10, 4, 40), "32 x 32"),
    ((1, 9, 10, 3, 12), "32 x 32"),
    ((2, 65, 70, 4, 70), "64 x 64"),
    ((2, 65, 70, 3, 70), "64 x 64"),
    ((1, 130, 128, 4, 12), "128 x 32"),
    ((1, 130, 128, 3, 12), "128 x 32"),
]


@pytest.fixture(autouse=True)
def _whole_card():
    assert torch.cuda.get_device_properties(0).multi_processor_count == CUS


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("shape", [s for s, _ in SHAPES], ids=str)
def test_direct_f64_launch_forms(shape, dtype):
    from paper_1905_05233_amd.layer_ops import direct_conv_f64
    N, H, W, C, K = shape
    x, w = WL.draw_inputs(N, H, W, C, K, "uniform", seed=C + K)
    x, w = OF.to_dtype(x, dtype), OF.to_dtype(w, dtype)
    y = direct_conv_f64(to_dev(x, dtype), to_dev(w, dtype)).cpu().numpy()
    ref = OC.direct_f64(x, w)
    mag = OC.direct_f64(np.abs(x), np.abs(w))
    assert np.all(np.abs(y - ref) <= 2 * 2.0 ** -53 * (9 * C) * mag)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("shape", [s for s, _ in SHAPES_1D], ids=str)
def test_direct_f64_launch_forms_1d(shape, dtype):
    from paper_1905_05233_amd.layer_ops import direct_conv_f64
    N, _, L, C, K = shape
    x4, w4 = WL.draw_inputs(N, 1, L, C, K, "uniform", seed=C + K)
    x, w = OF.to_dtype(x4[:, 0], dtype), OF.to_dtype(w4[:, 1], dtype)
    y = direct_conv_f64(to_dev(x[:, None], dtype), to_dev(w[:, None], dtype)).cpu().numpy()[:, 0]
    ref = OC.direct1d_f64(x, w)
    mag = OC.direct1d_f64(np.abs(x), np.abs(w))
    assert np.all(np.abs(y - ref) <= 2 * 2.0 ** -53 * (3 * C) * mag)


@pytest.mark.parametrize("value", [float("inf"), float("nan")], ids=str)
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("shape", [s for s, _ in SPECIAL], ids=str)
def test_direct_f64_special_weight(shape, dtype, value):
    """Taps outside the image do not meet an infinite or NaN weight, and no
    other output channel does."""
    from paper_1905_05233_amd.layer_ops import direct_conv_f64
    N, H, W, C, K = shape
    x = torch.ones((N, H, W, C), device="cuda", dtype=TORCH[dtype])
    w = torch.full((K, 3, 3, C), 0.5, device="cuda", dtype=TORCH[dtype])
    w[5, 0, 1, 1] = value                      # the tap above the pixel
    want = direct_conv_f64(x, torch.full_like(w, 0.5))
    assert bool((want[:, 1:-1, 1:-1] == 4.5 * C).all())
    want[:, 1:, :, 5] = value                  # the first row has no pixel above
    assert torch.equal(torch.nan_to_num(direct_conv_f64(x, w), nan=-7.0), torch.nan_to_num(want, nan=-7.0))


@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")], ids=str)
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("shape", [s for s, _ in SPECIAL], ids=str)
def test_direct_f64_special_input(shape, dtype, value):
    """An infinite or NaN pixel reaches the outputs of its window and no others."""
    from paper_1905_05233_amd.layer_ops import direct_conv_f64
    N, H, W, C, K = shape
    x = torch.ones((N, H, W, C), device="cuda", dtype=TORCH[dtype])
    w = torch.full((K, 3, 3, C), 0.5, device="cuda", dtype=TORCH[dtype])
    want = direct_conv_f64(x, w)
    for h, v in ((0, 0), (H - 1, W - 1), (4, 5)):
        x[N - 1, h, v, C - 1] = value
        want[N - 1, max(0, h - 1):h + 2, max(0, v - 1):v + 2] = value
    assert torch.equal(torch.nan_to_num(direct_conv_f64(x, w), nan=-7.0), torch.nan_to_num(want, nan=-7.0))
