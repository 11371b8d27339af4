"""The input transform where its launch changes form: pairs of channels or
single ones, domain rows split over workgroups, the last workgroup partly
filled, batches whose input exceeds the 1 GiB that one launch addresses, and
single images beyond it.  V is compared bit for bit: with the oracle's at small
sizes, and at large ones with the V of a crop or of single images, whose tiles
see the same pixels.
"""
import numpy as np
import pytest
import torch

from gpu_helpers import TORCH, stages_on_device_layout, to_dev, to_np
from oracle import conv as OC
from oracle import fp as OF
from oracle import plan as OP
from paper_1905_05233_amd import workloads as WL

pytestmark = pytest.mark.gpu

F8 = ("0,-1,1,-1/2,2,1/2,-2,a^2+1,inf", 8)


@pytest.mark.parametrize("spec,m,dtype,shape", [
    (WL.F4_A2P1, 4, "bf16", (1, 4, 64, 16)),      # 16 tiles x 16 channels: one workgroup exactly
    (WL.F4_A2P1, 4, "f16", (1, 4, 68, 16)),       # one tile more
    (WL.F4_A2P1, 4, "bf16", (1, 128, 128, 64)),   # 256 workgroups of single channels
    (WL.F4_A2P1, 4, "bf16", (1, 128, 129, 64)),   # a tile column more: pairs
    (WL.F4_A2P1, 4, "f16", (1, 128, 132, 66)),    # pairs off the 16-byte chunk
    (WL.F2_LINEAR, 2, "bf16", (2, 50, 94, 29)),   # many threads, odd C: single channels, units behind
    (WL.F4_A2P1, 4, "bf16", (2, 13, 9, 15)),      # odd C: the last run past C
    (WL.F4_A2P1, 4, "f16", (2, 13, 9, 18)),       # C off the 16-byte chunk
    (WL.F4_A2P1, 4, "bf16", (3, 5, 7, 1)),        # one channel of eight
    (WL.F6_TWO_QUAD, 6, "f32", (1, 96, 96, 128)),  # 2^15 threads: rows split over four workgroups
    (WL.F6_TWO_QUAD, 6, "f32", (1, 96, 97, 128)),  # just above: not split
    (WL.F6_LINEAR, 6, "bf16", (1, 20, 20, 40)),   # split, 8 domain rows: two a group
    (F8[0], F8[1], "f16", (1, 30, 22, 23)),       # split, 11 domain rows: the last group has two
], ids=str)
def test_input_transform_launch_forms(spec, m, dtype, shape):
    from paper_1905_05233_amd.winograd import Plan
    N, H, W, C = shape
    x, w = WL.draw_inputs(N, H, W, C, 2, "halfnormal", seed=H + C)
    x, w = OF.to_dtype(x, dtype), OF.to_dtype(w, dtype)
    st = OC.winograd_emulated_stages(x, w, OP.build_plan(spec, n_o=m), dtype)
    Uo, Vo = stages_on_device_layout(st)
    p = Plan(spec, m=m, dtype=dtype)
    V = to_np(p.input_transform(to_dev(x, dtype)))
    assert np.array_equal(V[:, :, :C], Vo)
    assert not V[:, :, C:].any()
    U2, V2 = p.kernel_input_transform(to_dev(w, dtype), to_dev(x, dtype))
    assert np.array_equal(to_np(V2), V) and np.array_equal(to_np(U2)[:, :, :C], Uo)


def _random(shape, dtype, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda").to(TORCH[dtype])


@pytest.mark.parametrize("dtype,C", [("f32", 32), ("bf16", 64)])
def test_input_transform_batch_over_one_launch(dtype, C):
    """Five images of 288 MiB: three in the first launch, two in the second."""
    from paper_1905_05233_amd.winograd import Plan
    p = Plan(WL.F2_LINEAR, m=2, dtype=dtype)
    x = _random((5, 1536, 1536, C), dtype, 1)
    assert 3 * x[0].numel() * x.element_size() <= 1 << 30 < 4 * x[0].numel() * x.element_size()
    V = p.input_transform(x)
    per = 768 * 768
    for n in range(5):
        one = p.input_transform(x[n:n + 1].contiguous())
        assert torch.equal(V[:, n * per:(n + 1) * per], one), n


@pytest.mark.parametrize("dtype,C", [("f32", 8), ("bf16", 15)])
def test_input_transform_image_over_one_launch(dtype, C):
    """One image over 1 GiB: its first and last tile rows against a crop's."""
    from paper_1905_05233_amd.winograd import Plan
    p = Plan(WL.F2_LINEAR, m=2, dtype=dtype)
    H, W = 4100 + (4800 if dtype == "bf16" else 0), 8192
    x = _random((1, H, W, C), dtype, 2)
    assert x.numel() * x.element_size() > 1 << 30
    V = p.input_transform(x)
    tw = W // 2
    top = p.input_transform(x[:, :42].contiguous())           # tile rows 0 .. 19 see rows below 41
    assert torch.equal(V[:, :20 * tw], top[:, :20 * tw])
    end = p.input_transform(x[:, H - 42:].contiguous())       # the last 20 tile rows
    assert torch.equal(V[:, -20 * tw:], end[:, -20 * tw:])
