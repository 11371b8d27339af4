"""The launches of layers too large for one: the host arithmetic of
launch_split.hpp, compiled and run on the CPU.  HIP takes fewer than 2^32
work-items (gridDim.x * blockDim.x) along x."""
import subprocess

import pytest

from paper_1905_05233_amd import build_native as B

SRC = r"""
#include <cstdio>
#include <cstdlib>
#include "launch_split.hpp"
int main(int argc, char** argv) {
    for (int i = 1; i < argc; ++i) {
        const int64_t K = std::atoll(argv[i]), per = wg::output_tiles_per_launch(K);
        std::printf("%lld %lld %lld\n", (long long)per, (long long)(per * K),
                    (long long)(wg::output_blocks(per * K) * wg::kOutBlock));
    }
}
"""


@pytest.fixture(scope="module")
def split(tmp_path_factory):
    d = tmp_path_factory.mktemp("split")
    (d / "split.cpp").write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-Wall", f"-I{B.CSRC}", str(d / "split.cpp"), "-o", str(d / "split")], check=True)
    return str(d / "split")


def test_output_transform_launches_stay_within_the_grid(split):
    ks = [1, 3, 64, 255, 256, 257, 512, 4096, 65537, 0x7fffff00]
    out = subprocess.run([split] + [str(k) for k in ks], capture_output=True, text=True, check=True).stdout
    for k, line in zip(ks, out.splitlines(), strict=True):
        per, pairs, items = map(int, line.split())
        assert per >= 1 and pairs < 2 ** 31, k       # ids of 31 bits
        assert pairs > 2 ** 31 - 256 - k, k          # and as many tiles as fit
        assert 2 * pairs <= items < 2 ** 32, k       # two row groups
