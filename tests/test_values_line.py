"""Where V is transposed ahead of a bf16 launch: the library's rule at the calls that it was measured on, and the tests' copy of it."""
import os
import shutil
import subprocess

import pytest

import launch_rules
from paper_2507_09071_amd import build

DRIVER = r"""
#include <cstdio>
#include "tilemap_internal.h"
int main()
{
    long long d, steps, tiles;
    while (std::scanf("%lld %lld %lld", &d, &steps, &tiles) == 3) std::printf("%d\n", (int)bs::transposed_values((int32_t)d, steps, tiles));
}
"""
# head dimension, steps per tile, tiles; which side was faster by half a percent and more
COPY = [(128, 24.3, 148), (128, 26.0, 188), (128, 23.8, 60), (128, 27.3, 37), (128, 38.8, 2080), (128, 59.6, 2272), (128, 82.8, 1136),
        (64, 1.2, 88), (64, 2.46, 104), (64, 2.85, 144), (64, 3.11, 192), (64, 3.6, 148), (64, 4.64, 2336), (64, 8.75, 1280), (64, 30.1, 1280), (64, 12.5, 9088), (64, 20.3, 17056)]
IN_PLACE = [(128, 11.5, 192), (128, 15.1, 240), (128, 17.8, 296), (128, 9.66, 1216), (128, 12.4, 316), (128, 17.5, 4272), (128, 18.8, 4104), (128, 24.6, 2844), (128, 4.95, 16576),
            (64, 1.22, 2576), (64, 2.85, 576), (64, 3.1, 768), (64, 2.97, 3688), (64, 5.6, 4264), (64, 8.75, 5120), (64, 2.03, 11368)]


def library_says(tmp_path, calls):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    (tmp_path / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
                    str(tmp_path / "driver.cpp"), "-o", str(tmp_path / "driver")], check=True)
    done = subprocess.run([tmp_path / "driver"], input="".join("%d %d %d\n" % c for c in calls), capture_output=True, text=True, check=True)
    return [x == "1" for x in done.stdout.split()]


def test_the_faster_side_is_taken(tmp_path):
    calls = [(d, round(r * t), t) for d, r, t in COPY + IN_PLACE]
    assert library_says(tmp_path, calls) == [True] * len(COPY) + [False] * len(IN_PLACE)


def test_the_tests_know_the_rule(tmp_path):
    calls = [(d, steps, t) for d in (64, 128) for t in (1, 200, 256, 257, 2000, 4096, 4097, 50000) for x in (0, 4, 10, 22, 32) for steps in (x * t - 1, x * t, x * t + 1)
             if steps >= 0]
    assert library_says(tmp_path, calls) == [launch_rules.transposed_values(*c) for c in calls]
