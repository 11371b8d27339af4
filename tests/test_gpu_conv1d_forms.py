"""The 1D form where its launch changes: V, M and the output transform in one
kernel or in the separate ones, 64 tiles x 64 channels or 32 x 128 per
workgroup, rows of 4-byte runs or single 16-bit channels, ragged ends of every
kind.  Against the oracle's 1D path element by element within ``pair_bound_1d``
(the same U and V, another order of the fp32 channel sums).
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
