"""Without a window the blocks of up to 2048 units are dealt to the eight queues there and back (of more, in turn): every item once, in the order of
the cost buckets, and the heaviest queue of a launch is, in whole turns, less than half as far from the lightest as dealing in turn puts it."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2507_09071_amd import build

DRIVER = r"""
#include <algorithm>
#include <cstdio>
#include <tuple>
#include <vector>
#include "blindsight.h"
#include "tilemap_internal.h"

int main()
{
    int balanced = 0, place = 0;   // (what is wrong with the places is said when all launches are seen to be balanced)
    for (int L : {60, 700, 4000, 9000, 16000, 70000})
        for (int n_kv : {4, 8, 21})
            for (int G : {1, 2, 7})
                for (bool dense : {false, true}) {
                    std::vector<bs_span> spans;
                    for (int p = 30; p + 500 < L; p += 530) spans.push_back({p, p + 500, 50});
                    std::vector<uint8_t> classes(n_kv * G);
                    for (size_t h = 0; h < classes.size(); ++h) classes[h] = dense ? 0 : (uint8_t)(h * 7 / 3 % 4);
                    bs_tilemap *tm = nullptr;
                    if (bs_build_tilemap_suffix(spans.data(), (int32_t)spans.size(), L, classes.data(), n_kv * G, 5, 128, 64, BS_MAP_PACK_KEYS, nullptr, 0, 0, 0, &tm) != BS_OK) return 1;
                    // every item in one unit, with the lists of its class (the library's own check; long prompts take it a while)
                    int64_t n_units, tiles, skips;
                    if (L <= 9000 && bs_tilemap_pair_plan(tm, G, &n_units, &tiles, &skips) != BS_OK) return 2;
                    bs_plan_pairs(tm, G);
                    const auto &plan = tm->pairs;
                    const int n = (int)plan.items.size(), block = std::min(16, std::max(8, n / 2048));
                    if (plan.queue_off[0] != 0 || plan.queue_off[8] != n) return 2;

                    long total = 0;
                    for (const bs::PairItem &it : plan.items) total += it.n_tiles;
                    const long wide = 32L * std::max(1, n_kv / 4) * std::max(1, n_kv / 4), even = total / 256 / 64;
                    const int bucket = (int)std::max(1L, even < 32 ? even : std::min(wide, even) / 32 * 32);
                    const auto key = [&](const bs::PairItem &it) { return std::make_tuple(-(it.n_tiles / bucket), it.head_a / G, -it.n_tiles); };

                    // steps of the queues in whole turns there and back, and of those that dealing in turn would make
                    const int turns = n / block / 16;
                    std::vector<bs::PairItem> sorted = plan.items;
                    std::stable_sort(sorted.begin(), sorted.end(), [&](const bs::PairItem &a, const bs::PairItem &b) { return key(a) < key(b); });
                    long queue[8] = {0}, in_turn[8] = {0};
                    for (int q = 0; q < 8; ++q)
                        for (int i = plan.queue_off[q]; i < std::min(plan.queue_off[q] + 2 * turns * block, plan.queue_off[q + 1]); ++i) queue[q] += plan.items[i].n_tiles + 6;
                    for (int p = 0; p < 16 * turns * block; ++p) in_turn[p / block % 8] += sorted[p].n_tiles + 6;
                    const auto spread = [](const long *x) { return (double)*std::max_element(x, x + 8) / *std::min_element(x, x + 8) - 1; };
                    if (n <= 2048 && turns >= 2) {
                        ++balanced;
                        if (spread(in_turn) > 0.04 && spread(queue) > spread(in_turn) / 2) {
                            std::printf("L %d KV heads %d G %d dense %d: %.3f, in turn %.3f\n", L, n_kv, G, dense, spread(queue), spread(in_turn));
                            return 6;
                        }
                    }

                    int at[8];
                    std::copy(plan.queue_off, plan.queue_off + 8, at);
                    for (int p = 0; p < n; ++p) {
                        const int round = p / block / 8, x = p / block % 8, q = n <= 2048 && (round & 1) ? 7 - x : x;
                        if (at[q] >= plan.queue_off[q + 1]) { place = 3; break; }
                        if (key(plan.items[at[q]++]) != key(sorted[p])) { std::printf("L %d KV heads %d G %d dense %d unit %d\n", L, n_kv, G, dense, p); place = 4; break; }
                    }
                    bs_tilemap_destroy(tm);
                }
    return balanced < 20 ? 5 : place;
}
"""


def run_driver(tmp_path, builder):
    (tmp_path / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, str(builder), str(tmp_path / "driver.cpp"),
                    "-o", str(tmp_path / "driver")], check=True)
    return subprocess.run([tmp_path / "driver"], capture_output=True, text=True)


@pytest.fixture
def source():
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    return os.path.join(build.CSRC, "tilemap.cpp")


def test_blocks_there_and_back(tmp_path, source):
    done = run_driver(tmp_path, source)
    assert done.returncode == 0, (done.returncode, done.stdout)


def test_dealing_in_turn_is_noticed(tmp_path, source):
    text, n = re.subn(r"there_and_back = [^;]*;", "there_and_back = false;", open(source).read(), count=1)
    assert n == 1
    (tmp_path / "in_turn.cpp").write_text(text)
    done = run_driver(tmp_path, tmp_path / "in_turn.cpp")
    assert done.returncode == 6, (done.returncode, done.stdout)
