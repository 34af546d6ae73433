"""Equal shares are cut from the units in the order that dealing the queues in turn gives, also where they are dealt there and back: the way the
queues are dealt changes neither which units are cut nor, with it, the rounding of the results."""
import os
import shutil
import subprocess

import pytest

from paper_2507_09071_amd import build

DRIVER = r"""
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <vector>
#include "blindsight.h"
#include "tilemap_internal.h"

template <class T>
static bool same(const std::vector<T> &a, const std::vector<T> &b)
{
    return a.size() == b.size() && (a.empty() || std::memcmp(a.data(), b.data(), a.size() * sizeof(T)) == 0);
}

int main()
{
    int shared = 0, moved = 0;
    for (int L : {700, 1337, 2500, 4000, 36864})
        for (int G : {1, 4, 7})
            for (int rows : {0, 517, 2048}) {
                if (rows >= L || (rows == 0 && L > 4000)) continue;
                std::vector<bs_span> spans;
                for (int p = 30; p + 500 < L; p += 530) spans.push_back({p, p + 500, 50});
                std::vector<uint8_t> classes(4 * G);
                for (size_t h = 0; h < classes.size(); ++h) classes[h] = (uint8_t)(h * 7 / 3 % 4);
                bs_tilemap *map[2] = {nullptr, nullptr};
                for (bs_tilemap *&tm : map)
                    if (bs_build_tilemap_suffix(spans.data(), (int32_t)spans.size(), L, classes.data(), 4 * G, 5, 128, 64, BS_MAP_PACK_KEYS, nullptr, 0, 0, rows ? L - rows : 0, &tm) != BS_OK) return 1;
                bs_plan_shares(map[0], G, 256);
                // the other map's queues as dealing in turn fills them
                bs_plan_pairs(map[1], G);
                bs::PairPlan &plan = map[1]->pairs;
                const int n = (int)plan.items.size(), block = 8;
                std::vector<bs::PairItem> sorted, queues[8], dealt;
                std::vector<int> at(plan.queue_off, plan.queue_off + 8);
                for (int p = 0; p < n; ++p) {
                    const int round = p / block / 8, x = p / block % 8;
                    sorted.push_back(plan.items[at[round & 1 ? 7 - x : x]++]);
                }
                for (int p = 0; p < n; ++p) queues[p / block % 8].push_back(sorted[p]);
                for (int q = 0; q < 8; ++q) {
                    plan.queue_off[q] = (int32_t)dealt.size();
                    dealt.insert(dealt.end(), queues[q].begin(), queues[q].end());
                }
                moved += !same(plan.items, dealt);
                plan.items.swap(dealt);
                plan.back_block = 0;
                bs_plan_shares(map[1], G, 256);
                const bs::SharePlan &a = map[0]->shares, &b = map[1]->shares;
                if (!same(a.parts, b.parts) || !same(a.ranges, b.ranges) || !same(a.share_off, b.share_off) || !same(a.cut, b.cut)) {
                    std::printf("L %d G %d rows %d\n", L, G, rows);
                    return 2;
                }
                shared += !a.cut.empty();
                for (bs_tilemap *tm : map) bs_tilemap_destroy(tm);
            }
    std::printf("%d with cut units, %d dealt in another order\n", shared, moved);
    return shared >= 10 && moved >= 10 ? 0 : 3;
}
"""


def test_shares_do_not_hang_on_how_the_queues_are_dealt(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    (tmp_path / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
                    os.path.join(build.CSRC, "tilemap.cpp"), str(tmp_path / "driver.cpp"), "-o", str(tmp_path / "driver")], check=True)
    done = subprocess.run([tmp_path / "driver"], capture_output=True, text=True)
    assert done.returncode == 0, (done.returncode, done.stdout)
