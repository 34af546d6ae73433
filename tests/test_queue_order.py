"""The order of the work units in the eight queues: a driver of its own, compiled with the builder's source, looks at plans of many units (two
bytes of every field) and few."""
import os
import shutil
import subprocess

import pytest

from paper_2507_09071_amd import build

DRIVER = r"""
#include <algorithm>
#include <cstdio>
#include <tuple>
#include "blindsight.h"
#include "tilemap_internal.h"

int main()
{
    for (int L : {700, 9000, 70000})
        for (int G : {1, 2, 7}) {
            std::vector<bs_span> spans;
            for (int p = 30; p + 500 < L; p += 530) spans.push_back({p, p + 500, 50});
            std::vector<uint8_t> classes(21 * G);
            for (size_t h = 0; h < classes.size(); ++h) classes[h] = (uint8_t)(h * 7 / 3 % 4);
            bs_tilemap *tm = nullptr;
            if (bs_build_tilemap_suffix(spans.data(), (int32_t)spans.size(), L, classes.data(), 21 * G, 5, 128, 64, BS_MAP_PACK_KEYS, nullptr, 0, L * 4 / 7, 0, &tm) != BS_OK) return 1;
            bs_plan_pairs(tm, G);
            const auto &plan = tm->pairs;
            const int n = (int)plan.items.size(), block = std::min(16, std::max(8, n / 2048));
            if (plan.queue_off[0] != 0 || plan.queue_off[8] != n) return 2;
            int at[8];
            std::copy(plan.queue_off, plan.queue_off + 8, at);
            std::tuple<int, int, int> last{-1, 0, 0};
            for (int p = 0; p < n; ++p) {   // as they were dealt: in a window by cost in steps of 8, KV head, rows
                const int q = p / block % 8;
                if (at[q] >= plan.queue_off[q + 1]) return 3;
                const bs::PairItem &it = plan.items[at[q]++];
                const std::tuple<int, int, int> now{100000 - it.n_tiles / 8, it.head_a / G, it.tile_a};
                if (now < last) { std::printf("L %d G %d unit %d\n", L, G, p); return 4; }
                last = now;
            }
            bs_tilemap_destroy(tm);
        }
    return 0;
}
"""


def test_units_in_order(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    (tmp_path / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
                    os.path.join(build.CSRC, "tilemap.cpp"), str(tmp_path / "driver.cpp"), "-o", str(tmp_path / "driver")], check=True)
    done = subprocess.run([tmp_path / "driver"], capture_output=True, text=True)
    assert done.returncode == 0, (done.returncode, done.stdout)
