"""conv2d of ReLU(x) with the ReLU applied as the input transform reads x:
the same bits as the ReLU kernel followed by conv2d, NaN, -0 and infinities
among the inputs, on each path and in chunks of the batch; plans without that
form refuse it."""
import pytest
import torch

from gpu_helpers import TORCH
from paper_1905_05233_amd import workloads as WL

pytestmark = pytest.mark.gpu


def _layer(shape, dtype, special):
    N, H, W, C, K = shape
    g = torch.Generator(device="cuda")
    g.manual_seed(C + K)
    x = torch.randn((N, H, W, C), generator=g, device="cuda")
    if special:
        flat = x.view(-1)
        flat[::37] = float("nan")
        flat[1::41] = -0.0
        flat[2::97] = float("-inf")
        flat[3::1009] = float("inf")
    w = torch.randn((K, 3, 3, C), generator=g, device="cuda") * 0.1
    return x.to(TORCH[dtype]), w.to(TORCH[dtype])


@pytest.mark.parametrize("special", [False, True], ids=["finite", "special"])
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("spec,m,path,shape", [
    (WL.F4_A2P1, 4, "auto", (2, 19, 22, 40, 24)),
    (WL.F4_A2P1, 4, "fused", (1, 21, 17, 33, 70)),       # odd C
    (WL.F2_LINEAR, 2, "separate", (1, 9, 8, 6, 5)),
    (WL.F6_TWO_QUAD, 6, "separate", (1, 20, 21, 12, 9)),  # rows split over workgroups
    (WL.F6_LINEAR, 6, "auto", (4, 60, 60, 64, 16)),
], ids=str)
def test_relu_input_same_bits(spec, m, path, shape, dtype, special):
    from paper_1905_05233_amd.layer_ops import relu_pool
    from paper_1905_05233_amd.winograd import Plan
    x, w = _layer(shape, dtype, special)
    p = Plan(spec, m=m, dtype=dtype, path=path)
    assert p.relu_input_supported(*shape)
    got = p.conv2d_relu_input(x, w)
    want = p.conv2d(relu_pool(x, False), w)
    assert torch.equal(torch.nan_to_num(got.float()), torch.nan_to_num(want.float()))
    assert torch.equal(torch.isnan(got), torch.isnan(want))


def test_relu_input_in_chunks():
    from paper_1905_05233_amd.layer_ops import relu_pool
    from paper_1905_05233_amd.winograd import Plan
    shape = (9, 224, 224, 64, 64)
    x, w = _layer(shape, "bf16", False)
    p = Plan(WL.F4_A2P1, m=4, dtype="bf16")
    assert p.conv_chunks(*shape)[0] == 2
    assert torch.equal(p.conv2d_relu_input(x, w), p.conv2d(relu_pool(x, False), w))


def test_relu_input_refused():
    from paper_1905_05233_amd._native import WinogradError
    from paper_1905_05233_amd.winograd import Plan
    x, w = _layer((1, 9, 9, 3, 40), "bf16", False)
    for p in (Plan(WL.F4_A2P1, m=4, dtype="bf16", generic_transforms=True),
              Plan(WL.F4_A2P1, m=4, dtype="bf16", path="fused_input")):
        assert not p.relu_input_supported(1, 9, 9, 3, 40)
        with pytest.raises(WinogradError, match="UNSUPPORTED"):
            p.conv2d_relu_input(x, w)


def test_stack_with_a_plan_exchanged_after_a_pass():
    """A layer's plan replaced by one without the ReLU form: the ReLU kernel runs before it."""
    from paper_1905_05233_amd.vgg import VggStack
    from paper_1905_05233_amd.winograd import Plan
    s = VggStack(dtype="bf16", plans=[WL.PlanSpec(WL.F4_A2P1, 4)] * 13)
    x = s.input(1)
    s.forward(x)
    s.layers[1]["plan"] = Plan(WL.F4_A2P1, m=4, dtype="bf16", generic_transforms=True)
    got = s.forward(x)
    want, _ = s.forward(x, keep=True)
    assert torch.equal(got, want)
