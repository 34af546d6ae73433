"""Without a window the blocks of up to 2048 units are dealt to the eight queues there and back (of more, in turn): every unit once, in order, and with full turns
no queue has more steps than another by more than its heaviest block and the width of the cost buckets allow."""
import os
import shutil
import subprocess

import pytest

from paper_2507_09071_amd import build

DRIVER = r"""
#include <algorithm>
#include <cstdio>
#include <vector>
#include "blindsight.h"
#include "tilemap_internal.h"

int main()
{
    for (int L : {60, 700, 9000, 70000})
        for (int G : {1, 2, 7}) {
            std::vector<bs_span> spans;
            for (int p = 30; p + 500 < L; p += 530) spans.push_back({p, p + 500, 50});
            std::vector<uint8_t> classes(21 * G);
            for (size_t h = 0; h < classes.size(); ++h) classes[h] = (uint8_t)(h * 7 / 3 % 4);
            bs_tilemap *tm = nullptr;
            if (bs_build_tilemap_suffix(spans.data(), (int32_t)spans.size(), L, classes.data(), 21 * G, 5, 128, 64, BS_MAP_PACK_KEYS, nullptr, 0, 0, 0, &tm) != BS_OK) return 1;
            bs_plan_pairs(tm, G);
            const auto &plan = tm->pairs;
            const int n = (int)plan.items.size(), block = std::min(16, std::max(8, n / 2048));
            if (plan.queue_off[0] != 0 || plan.queue_off[8] != n) return 2;
            int at[8], heaviest = 0, last = 1 << 30;
            std::copy(plan.queue_off, plan.queue_off + 8, at);
            for (int p = 0; p < n; ++p) {
                const int round = p / block / 8, x = p / block % 8, q = n <= 2048 && (round & 1) ? 7 - x : x;
                if (at[q] >= plan.queue_off[q + 1]) return 3;
                const int tiles = plan.items[at[q]++].n_tiles;
                heaviest = std::max(heaviest, tiles);
                if (tiles > last + 32 * 32) { std::printf("L %d G %d unit %d\n", L, G, p); return 4; }   // (in buckets of some width)
                last = tiles;
            }
            for (int q = 0; q < 8; ++q)
                if (at[q] != plan.queue_off[q + 1]) return 5;
            // (full turns there and back; a unit may stand in front of a heavier one of its bucket)
            const int turns = n / block / 16;
            long most = 0, least = 1L << 60;
            for (int q = 0; q < 8; ++q) {
                long sum = 0;
                for (int i = 0; i < 2 * turns * block; ++i) sum += plan.items[plan.queue_off[q] + i].n_tiles;
                most = std::max(most, sum);
                least = std::min(least, sum);
            }
            if (n <= 2048 && turns > 0 && most - least > (long)block * heaviest + 2L * turns * block * 32 * 32) return 6;
            bs_tilemap_destroy(tm);
        }
    return 0;
}
"""


def test_blocks_there_and_back(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    (tmp_path / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
                    os.path.join(build.CSRC, "tilemap.cpp"), str(tmp_path / "driver.cpp"), "-o", str(tmp_path / "driver")], check=True)
    done = subprocess.run([tmp_path / "driver"], capture_output=True, text=True)
    assert done.returncode == 0, (done.returncode, done.stdout)
