"""The launches of layers too large for one, and the forms that the 1D and the
float64 convolution take: the host arithmetic of launch_split.hpp, compiled and run on
the CPU.  HIP takes fewer than 2^32 work-items (gridDim.x * blockDim.x) along x."""
import subprocess

import pytest

import test_gpu_direct_f64 as F64
from paper_1905_05233_amd import build_native as B

SRC = r"""
#include <cstdio>
#include <cstdlib>
#include "launch_split.hpp"
int main(int argc, char** argv) {
    if (argc == 8) {   // H, bytes of a row of pixels, tile rows, threads of a row of tiles, m, row groups, a word
        int64_t a[6];
        for (int i = 0; i < 6; ++i) a[i] = std::atoll(argv[1 + i]);
        const int groups = static_cast<int>(a[5]);
        const wg::InputSplit s = wg::input_split(a[0], a[1], a[2], a[3], static_cast<int>(a[4]), groups);
        const int64_t threads = std::max<int64_t>(s.images, 1) * s.rows * a[3];
        std::printf("%lld %lld\n", (long long)threads, (long long)(wg::input_blocks(threads, groups) * wg::kInBlock));
        std::printf("%lld %lld\n", (long long)s.images, (long long)s.rows);
        for (int64_t r0 = 0; s.rows && s.rows < a[2] && r0 < a[2]; r0 += s.rows) {
            const wg::InputBand b = wg::input_band(a[0], r0, std::min(s.rows, a[2] - r0), static_cast<int>(a[4]));
            std::printf("%lld %lld %lld\n", (long long)r0, (long long)b.first, (long long)b.end);
        }
        return 0;
    }
    if (argc == 9) {   // tiles, Cp, K, Kp, alpha', bytes of a value, two words
        int64_t a[6];
        for (int i = 0; i < 6; ++i) a[i] = std::atoll(argv[1 + i]);
        std::printf("%d\n", wg::conv1d_one_kernel_pays(a[0], a[1], a[2], a[3], static_cast<int>(a[4]), a[5]));
        return 0;
    }
    if (argc == 7) {   // pixels, C, K, taps, bytes of a value, compute units
        int64_t a[6];
        for (int i = 0; i < 6; ++i) a[i] = std::atoll(argv[1 + i]);
        std::printf("%d\n", wg::f64_form(a[0], a[1], a[2], static_cast<int>(a[3]), a[4], static_cast<int>(a[5])));
        return 0;
    }
    const int groups = std::atoi(argv[1]);
    for (int i = 2; i < argc; ++i) {   // row groups, then output channels, more than eight of them
        const int64_t K = std::atoll(argv[i]), per = wg::output_tiles_per_launch(K, groups);
        std::printf("%lld %lld %lld\n", (long long)per, (long long)(per * K),
                    (long long)(wg::output_blocks(per * K, groups) * wg::kOutBlock));
    }
}
"""


@pytest.fixture(scope="module")
def split(tmp_path_factory):
    d = tmp_path_factory.mktemp("split")
    (d / "split.cpp").write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-Wall", f"-I{B.CSRC}", str(d / "split.cpp"), "-o", str(d / "split")], check=True)
    return str(d / "split")


@pytest.mark.parametrize("groups", [1, 2])
def test_output_transform_launches_stay_within_the_grid(split, groups):
    ks = [1, 3, 64, 255, 256, 257, 512, 4096, 65537, 0x7fffff00]
    out = subprocess.run([split, str(groups)] + [str(k) for k in ks], capture_output=True, text=True, check=True).stdout
    for k, line in zip(ks, out.splitlines(), strict=True):
        per, pairs, items = map(int, line.split())
        assert per >= 1 and pairs < 2 ** 31, k       # ids of 31 bits
        assert pairs > 2 ** 31 - 256 - k, k          # and as many tiles as fit
        assert groups * pairs <= items < 2 ** 32, k


@pytest.mark.parametrize("m,groups", [(2, 1), (4, 1), (7, 1), (8, 4), (12, 4)])
@pytest.mark.parametrize("H,row", [(16, 1 << 20), (1024, 1 << 20), (1025, 1 << 20), (1 << 14, (1 << 17) + 2),
                                   (300, (1 << 26) - 6), (9, 1 << 28), (3, 1 << 29), (1, 1 << 30), (1, (1 << 30) + 4),
                                   (1 << 29, 2), (1 << 30, 2)])
def test_input_transform_launches_reach_every_row(split, H, row, m, groups):
    """Groups of images or bands of tile rows: the bytes and ids of each within
    32-bit reach, and every pixel that a band's tiles read among its rows."""
    th, thr = -(-H // m), 8 * max(1, row // 64)
    args = [split] + [str(v) for v in (H, row, th, thr, m, groups)] + ["input"]
    out = subprocess.run(args, capture_output=True, text=True, check=True).stdout
    (threads, items), (images, rows), *bands = [tuple(map(int, line.split())) for line in out.splitlines()]
    assert threads < 2 ** 31 and threads * groups <= items < 2 ** 32
    most = min(2 ** 31 - 1, (2 ** 32 - 1) // groups // 256 * 256)
    if H * row <= 1 << 30 and th * thr <= most:
        assert rows == th and images >= 1 and images * H * row <= 1 << 30
        assert (images + 1) * H * row > 1 << 30 or (images + 1) * th * thr > most
        return
    assert images == 1
    if rows == 0:
        assert (m + 2) * row > 1 << 30 or thr > most
        return
    assert rows < th and len(bands) == -(-th // rows)
    for r0, first, end in bands:
        r1 = min(th, r0 + rows)
        assert (end - first) * row <= 1 << 30 and (r1 - r0) * thr <= most
        assert first == max(0, r0 * m - 1) and end == min(H, r1 * m + 1)


@pytest.mark.parametrize("m,alpha,es,layer,one_kernel", [
    # N, L, C, K and both times in us, one kernel and separate
    (4, 7, 2, (16, 4096, 128, 128), True),     # 26, 87
    (4, 7, 4, (16, 4096, 64, 128), True),      # a fifth of the separate kernels' bytes
    (4, 7, 2, (3, 6542, 16, 16), True),        # 6, 16: one chunk
    (4, 7, 2, (1, 100, 512, 512), False),      # 40, 21: four blocks
    (4, 7, 2, (32, 512, 512, 512), True),      # 69, 89
    (6, 10, 4, (5, 8000, 128, 512), False),    # 173, 146
    (6, 10, 4, (16, 4096, 512, 512), False),   # 901, 633
    (6, 10, 2, (64, 300, 512, 1024), False),   # 258, 140
    (6, 10, 2, (32, 8000, 301, 77), True),     # 334, 388
    (4, 6, 4, (64, 300, 512, 512), False),     # 270, 200
    (2, 4, 4, (4, 8000, 256, 128), True),      # 0.67 of the separate kernels' time
    # the layers of the GPU tests of both forms
    (4, 7, 2, (1, 257, 8, 65), True), (4, 7, 4, (40, 130, 34, 66), True), (4, 6, 2, (1, 40, 200, 20), False),
    (6, 10, 2, (60, 100, 48, 40), True), (4, 7, 2, (1400, 41, 200, 20), True), (4, 7, 4, (1400, 41, 201, 70), True),
    (4, 7, 2, (1, 41, 200, 20), False), (4, 7, 4, (1, 41, 201, 70), False),
], ids=str)
def test_1d_form_of_a_layer(split, m, alpha, es, layer, one_kernel):
    N, L, C, K = layer
    args = [N * -(-L // m), -(-C // 8) * 8, K, -(-K // 8) * 8, alpha, es, "1d", "form"]
    out = subprocess.run([split] + [str(v) for v in args], capture_output=True, text=True, check=True).stdout
    assert bool(int(out)) == one_kernel


FORMS = ["one thread per output", "32 x 32", "64 x 64", "128 x 32"]


def test_float64_shapes_reach_every_form(split):
    """The shapes of the float64 tests select the forms that they name, and
    together every form, with aligned runs of four values and without."""
    seen = set()
    cases = [(9, s, f) for s, f in F64.SHAPES + F64.SPECIAL] + [(3, s, f) for s, f in F64.SHAPES_1D]
    for taps, (N, H, W, C, K), form in cases:
        for es in (2, 4):
            args = [N * H * W, C, K, taps, es, F64.CUS]
            out = subprocess.run([split] + [str(v) for v in args], capture_output=True, text=True, check=True).stdout
            assert FORMS[int(out)] == form, (taps, (N, H, W, C, K))
        seen.add((taps, form, C % 4 == 0))
    for taps in (9, 3):
        assert {(taps, f, v4) for f in FORMS[1:] for v4 in (True, False)} <= seen
    for form in FORMS[1:]:   # special values: every block shape
        assert form in [f for _, f in F64.SPECIAL]
