"""The host builder and planner under the undefined-behaviour sanitizer: a driver of its own, compiled with the builder's source,
plans the units and shares of a few prompts."""
import os
import shutil
import subprocess

import pytest

from paper_2507_09071_amd import build

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "blindsight.h"

static void ok(int rc, const char *what) { if (rc != BS_OK) { std::fprintf(stderr, "%s: %d\n", what, rc); std::exit(2); } }

int main()
{
    for (int L : {1, 300, 5000, 40000})
        for (uint32_t flags : {0u, (uint32_t)BS_MAP_REGROUP_ROWS, (uint32_t)(BS_MAP_PACK_KEYS | BS_MAP_BIDIR_IMAGES)})
            for (int window : {0, 700})
                for (int q_begin : {0, L / 2, L - 1}) {
                    std::vector<bs_span> spans;
                    for (int p = 7; p + 900 < L; p += 913) spans.push_back({p, p + 900, p % 3});
                    const uint8_t classes[8] = {0, 1, 2, 3, 3, 2, 1, 0};
                    const int32_t offsets[3] = {0, 64, 899};
                    bs_tilemap *tm = nullptr;
                    ok(bs_build_tilemap_suffix(spans.data(), (int32_t)spans.size(), L, classes, 8, L < 5 ? 0 : 5, 128, 64, flags, offsets,
                                               3, window, q_begin, &tm), "build");
                    ok(bs_tilemap_pair_plan(tm, 4, nullptr, nullptr, nullptr), "pair plan");
                    for (int wgs : {256, 512, 7}) {
                        ok(bs_tilemap_share_plan(tm, 4, wgs, nullptr, nullptr, nullptr), "share plan");
                        ok(bs_tilemap_share_plan(tm, 0, wgs, nullptr, nullptr, nullptr), "share plan, fp32");
                    }
                    for (int c = 0; c < 4; ++c) ok(bs_tilemap_stats(tm, c, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr), "stats");
                    bs_tilemap_destroy(tm);
                }
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_no_undefined_behaviour(tmp_path):
    driver, exe = tmp_path / "driver.cpp", tmp_path / "driver"
    driver.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-static-libubsan",
                    "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, os.path.join(build.CSRC, "tilemap.cpp"), str(driver),
                    "-o", str(exe)], check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True)
    assert done.returncode == 0, done.stderr
