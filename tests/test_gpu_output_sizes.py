"""The output transform where its launch changes form: one workgroup per (tile,
64 channels) below 2^17 (tile, channel) pairs, one thread per (tile, channel,
row group) from there on, with K off every block and ragged tiles.  Against the
same M through the other form (fewer images at a time), bit for bit, and the
small one against the oracle's output transform elsewhere in these tests.
"""
import pytest
import torch

from paper_1905_05233_amd import workloads as WL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("spec,m,shape", [
    (WL.F2_LINEAR, 2, (8, 32, 32, 64)),          # 2^17 pairs exactly
    (WL.F4_A2P1, 4, (6, 75, 91, 121)),           # odd K, tiles past both edges
    (WL.F4_LINEAR, 4, (9, 61, 50, 96)),
    (WL.F6_TWO_QUAD, 6, (16, 50, 55, 130)),
    ("0,-1,1,-1/2,inf", 3, (10, 70, 71, 25)),    # odd tiles: groups of two rows and one
    ("0,-1,1,-1/2,2,1/2,-2,a^2+1,inf", 8, (20, 64, 60, 108)),
    ("0,a^2+1,inf", 2, (30, 57, 35, 250)),       # M of 382 MiB: one row group
], ids=str)
def test_output_transform_forms_agree(spec, m, shape, dtype):
    from paper_1905_05233_amd.winograd import Plan
    N, H, W, K = shape
    p = Plan(spec, m=m, dtype=dtype)
    g = p.geometry(N, H, W, 8, K)
    per = g["T"] // N
    assert g["T"] * K >= 1 << 17 > per * K
    gen = torch.Generator(device="cuda")
    gen.manual_seed(K)
    M = torch.randn((p.alpha ** 2, g["T"], g["Kp"]), generator=gen, device="cuda")
    y = p.output_transform(M, N, H, W, K)
    for n in range(N):
        one = p.output_transform(M[:, n * per:(n + 1) * per].contiguous(), 1, H, W, K)
        assert torch.equal(y[n:n + 1], one), n


def test_output_transform_over_one_launch():
    """33 images of 2^26 (tile, channel) pairs: the first launch ends inside the 32nd."""
    from paper_1905_05233_amd.winograd import Plan
    N, H, W, K = 33, 2048, 2048, 64
    p = Plan(WL.F2_LINEAR, m=2, dtype="f16")
    g = p.geometry(N, H, W, 8, K)
    per = g["T"] // N
    assert g["T"] * K > 1 << 31
    if torch.cuda.mem_get_info()[0] < 200 << 30:
        pytest.skip("needs 200 GiB of device memory")
    M = torch.empty((p.alpha ** 2, g["T"], g["Kp"]), device="cuda").uniform_(-1.0, 1.0)
    y = p.output_transform(M, N, H, W, K)
    for n in (0, 31, 32):
        one = p.output_transform(M[:, n * per:(n + 1) * per].contiguous(), 1, H, W, K)
        assert torch.equal(y[n:n + 1], one), n
    del M, y, one
    torch.cuda.empty_cache()
