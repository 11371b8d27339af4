"""The 1D form where its launch changes: V, M and the output transform in one
kernel or in the separate ones, 64 tiles x 64 channels or 32 x 128 per
workgroup, rows of 4-byte runs or single 16-bit channels, ragged ends of every
kind, inputs over 1 GiB, infinities and NaN.  Against the oracle's 1D path
element by element within ``pair_bound_1d`` (the same U and V, another order of
the fp32 channel sums).
"""
import numpy as np
import pytest
import torch

from gpu_helpers import TORCH, pair_bound_1d
from oracle import conv as OC
from oracle import fp as OF
from oracle import plan as OP
from paper_1905_05233_amd import workloads as WL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("spec,m,shape", [
    (WL.F4_A2P1, 4, (1, 256, 8, 64)),        # 64 tiles exactly, one block of 64 channels
    (WL.F4_A2P1, 4, (1, 257, 8, 65)),        # one tile and one channel more: two blocks of 128 channels
    (WL.F4_A2P1, 4, (2, 131, 17, 30)),       # odd C: single 16-bit channels; K off four
    (WL.F4_A2P1, 4, (40, 130, 34, 66)),      # two chunks and a partial one, tiles crossing rows
    (WL.F2_LINEAR, 2, (3, 1, 3, 1)),         # one position a row
    (WL.F6_TWO_QUAD, 6, (60, 100, 48, 40)),  # ten points
    (WL.F4_LINEAR, 4, (1, 40, 200, 20)),     # long rows, one block: the separate kernels
], ids=str)
def test_conv1d_launch_forms(spec, m, shape, dtype):
    from paper_1905_05233_amd.winograd import Plan
    N, L, C, K = shape
    x4, w4 = WL.draw_inputs(N, 1, L, C, K, "uniform", seed=L + C)
    x, w = OF.to_dtype(x4[:, 0], dtype), OF.to_dtype(w4[:, 1], dtype)
    dev = [torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(TORCH[dtype]).cuda() for a in (x, w)]
    y = Plan(spec, m=m, dtype=dtype).conv1d(*dev).float().cpu().numpy().astype(np.float64)
    op = OP.build_plan(spec, n_o=m)
    st = OC.winograd1d_emulated_stages(x, w, op, dtype)
    assert np.all(np.abs(y - st["y"]) <= pair_bound_1d(st, op, dtype, y))


@pytest.mark.parametrize("dtype,C", [("bf16", 32), ("f16", 33), ("f32", 16)])
def test_conv1d_input_over_the_one_kernel_form(dtype, C):
    """Rows of over 1 GiB together go through the separate kernels: both ends of
    the first and last row against the oracle on crops."""
    from paper_1905_05233_amd.winograd import Plan
    N, L, K, m, n = 3, 6_000_001, 8, 4, 64
    g = torch.Generator(device="cuda")
    g.manual_seed(C)
    x = torch.randn((N, L, C), generator=g, device="cuda", dtype=TORCH[dtype])
    w = torch.randn((K, 3, C), generator=g, device="cuda", dtype=TORCH[dtype]) * 0.25
    assert x.numel() * x.element_size() > 1 << 30
    y = Plan(WL.F4_A2P1, m=m, dtype=dtype).conv1d(x, w)
    op = OP.build_plan(WL.F4_A2P1, n_o=m)
    wn = w.float().cpu().numpy()
    start = (L - n) // m * m                  # on the grid of tiles
    for row in (0, N - 1):
        for l0, l1 in ((0, n), (start, L)):
            xc = np.ascontiguousarray(x[row:row + 1, l0:l1].float().cpu().numpy())
            yc = y[row:row + 1, l0:l1].float().cpu().numpy().astype(np.float64)
            st = OC.winograd1d_emulated_stages(xc, wn, op, dtype)
            keep = slice(m, None) if l0 else slice(0, -m)   # the tile at the crop's cut edge apart
            err, bound = np.abs(yc - st["y"]), pair_bound_1d(st, op, dtype, yc)
            assert np.all(err[:, keep] <= bound[:, keep]), (row, l0)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("C,K", [(200, 20), (201, 70)])
def test_conv1d_special_values_in_both_forms(C, K, dtype):
    """Infinities and NaN in x: the same rows in a batch large enough for the one
    kernel, and a few at a time through the separate kernels, meet them in the
    same outputs; rows without any are the clean run's."""
    from paper_1905_05233_amd.winograd import Plan
    N, L = 1400, 41
    g = torch.Generator(device="cuda")
    g.manual_seed(C)
    x = torch.randn((N, L, C), generator=g, device="cuda").to(TORCH[dtype])
    w = (torch.randn((K, 3, C), generator=g, device="cuda") * 0.1).to(TORCH[dtype])
    p = Plan(WL.F4_A2P1, m=4, dtype=dtype)
    clean = p.conv1d(x, w)
    xs = x.clone()
    xs[3, 0, 0], xs[5, L - 1, C - 1], xs[9, 20, 7] = float("inf"), float("nan"), float("-inf")
    xs[N - 1, 17, C - 1], xs[N - 1, 18, 0] = float("inf"), float("inf")
    got = p.conv1d(xs, w)
    touched = [3, 5, 9, N - 1]
    rest = torch.ones(N, dtype=torch.bool, device="cuda")
    rest[touched] = False
    assert torch.equal(got[rest], clean[rest])
    for r in touched:
        few = p.conv1d(xs[r:r + 1].clone(), w)[0]
        one = got[r]
        assert not bool(torch.isfinite(one).all())
        assert torch.equal(torch.isnan(one), torch.isnan(few)), r
        assert torch.equal(torch.isinf(one), torch.isinf(few)), r
        inf = torch.isinf(one)
        assert torch.equal(one[inf], few[inf]), r
