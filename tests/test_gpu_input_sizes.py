"""The input transform where its launch changes form: pairs of channels or
single ones, domain rows split over workgroups, the last workgroup partly
filled, batches whose input exceeds the 1 GiB that one launch addresses, single
images beyond it and single rows.  V is compared bit for bit: with the oracle's at small
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
F8A12 = ("0,-1,1,-1/2,2,a^2+1,a^2-2,inf", 8)
F10 = ("0,-1,1,-1/2,2,1/2,-2,-1/4,4,a^2+1,inf", 10)
F12 = ("0,-1,1,-1/2,2,1/2,-2,-1/4,4,1/4,-4,a^2+1,inf", 12)


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
    (F8[0], F8[1], "bf16", (2, 90, 88, 130)),     # 10x10 windows above 2^15 threads: not split
    (F8A12[0], F8A12[1], "f32", (2, 90, 88, 130)),  # alpha' = 12: split
    (F10[0], F10[1], "bf16", (2, 115, 110, 130)),  # 12x12, 13 domain rows: split, the last group has one
    (F12[0], F12[1], "bf16", (2, 136, 130, 130)),  # 14x14, 15 domain rows: two a group, the last has one
    (F12[0], F12[1], "f32", (2, 136, 130, 130)),   # four a group, the last has three
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


def _bits(t):
    return t.view(torch.int32 if t.element_size() == 4 else torch.int16)


def _special(x, seed):
    """A few infinities and NaN spread over x, some beside its edges."""
    flat = x.view(-1)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    at = torch.randint(0, flat.numel(), (4096,), generator=g, device="cuda")
    flat[at[:2048]] = float("inf")
    flat[at[2048:3072]] = float("-inf")
    flat[at[3072:]] = float("nan")
    x[:, 0, 0], x[:, -1, -1] = float("inf"), float("nan")


@pytest.mark.parametrize("spec,m,dtype,H,C", [
    (WL.F2_LINEAR, 2, "f32", 4100, 8),
    (WL.F2_LINEAR, 2, "bf16", 8900, 15),
    (WL.F4_A2P1, 4, "f16", 5003, 16),     # built-in coefficients, pairs, a partial last tile row
    (WL.F6_TWO_QUAD, 6, "bf16", 4999, 16),
], ids=str)
def test_input_transform_image_over_one_launch(spec, m, dtype, H, C):
    """One image over 1 GiB, infinities and NaN in it, against
    crops of it: all of V, the tiles at a crop's cut edges apart."""
    from paper_1905_05233_amd.winograd import Plan
    p = Plan(spec, m=m, dtype=dtype)
    W = 8192
    x = _random((1, H, W, C), dtype, 2)
    _special(x, 3)
    assert x.numel() * x.element_size() > 1 << 30
    w = _random((5, 3, 3, C), dtype, 4)
    U, V = p.kernel_input_transform(w, x)
    assert torch.equal(U, p.kernel_transform(w))
    assert torch.equal(_bits(p.input_transform(x)), _bits(V))
    th, tw, step = -(-H // m), -(-W // m), 600
    for r in range(0, th, step):
        r0, r1 = max(0, r - 1), min(th, r + step + 1)   # a tile row more on each side
        crop = p.input_transform(x[:, r0 * m:min(H, r1 * m)].contiguous())
        a, b = (r - r0) * tw, (min(th, r + step) - r0) * tw
        assert torch.equal(_bits(V[:, r * tw:r * tw + b - a]), _bits(crop[:, a:b])), r


@pytest.mark.parametrize("dtype,C", [("bf16", 16), ("f16", 15), ("f32", 8)])
def test_input_transform_row_over_one_launch(dtype, C):
    """Rows of pixels of which four exceed 1 GiB: 64-bit addresses."""
    from paper_1905_05233_amd.winograd import Plan
    p = Plan(WL.F2_LINEAR, m=2, dtype=dtype)
    W, m, n = 1 << 24, 2, 1 << 12
    x = _random((1, 3, W, C), dtype, 5)
    _special(x, 6)
    assert 4 * W * C * x.element_size() > 1 << 30
    w = _random((5, 3, 3, C), dtype, 7)
    U, V = p.kernel_input_transform(w, x)
    assert torch.equal(U, p.kernel_transform(w))
    tw = W // m
    for c0 in (0, W // 2, W - n):           # crops of n columns, their cut edges apart
        crop = p.input_transform(x[:, :, c0:c0 + n].contiguous())
        for ty in range(2):
            a, b = (0 if c0 == 0 else 1), n // m - (0 if c0 == W - n else 1)
            got = V[:, ty * tw + c0 // m + a:ty * tw + c0 // m + b]
            assert torch.equal(_bits(got), _bits(crop[:, ty * (n // m) + a:ty * (n // m) + b])), (c0, ty)
