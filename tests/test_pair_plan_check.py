"""bs_tilemap_pair_plan checks the work units against the lists they come from: a driver of its own, compiled with the builder's
source, plants a mistake in a plan (which stays as long as the class vector does) and asks again."""
import os
import shutil
import subprocess

import pytest

from paper_2507_09071_amd import build

DRIVER = r"""
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include "blindsight.h"
#include "tilemap_internal.h"

static void expect(bool ok, const char *what) { if (!ok) { std::fprintf(stderr, "%s\n", what); std::exit(1); } }

int main(int, char **argv)
{
    std::vector<bs_span> spans;
    for (int p = 30; p + 256 < 9000; p += 276) spans.push_back({p, p + 256, 20});
    const uint8_t classes[4] = {3, 3, 2, 2};
    bs_tilemap *tm = nullptr;
    expect(bs_build_tilemap_ex(spans.data(), (int32_t)spans.size(), 9000, classes, 4, 5, 128, 64, BS_MAP_PACK_KEYS, &tm) == BS_OK, "build");
    expect(bs_tilemap_pair_plan(tm, 4, nullptr, nullptr, nullptr) == BS_OK, "plan");
    // a unit that walks compact tiles, then the prompt's, its list copied to the end so that it is nobody else's
    bs::PairPlan &plan = tm->pairs;
    bs::PairItem *unit = nullptr;
    for (bs::PairItem &it : plan.items)
        if (plan.ranges[it.list_begin].begin >= tm->N0 && plan.ranges[it.list_end - 1].begin < tm->N0) unit = &it;
    expect(unit != nullptr, "a unit of both kinds of tiles");
    std::vector<bs::PairRange> list(plan.ranges.begin() + unit->list_begin, plan.ranges.begin() + unit->list_end);
    const bs::PairRange first = list.front(), last = list.back();
    const auto tiles = [](const bs::PairRange &r) { return (r.end_states >> 4) - r.begin; };
    const auto prompt = std::find_if(list.begin(), list.end(), [&](const bs::PairRange &r) { return r.begin < tm->N0; });
    if (!std::strcmp(argv[1], "compact tiles twice")) {          // compact, prompt, compact
        list.push_back(first);
        unit->n_tiles += tiles(first);
    } else if (!std::strcmp(argv[1], "prompt tiles twice")) {    // compact, prompt, compact, prompt
        list.push_back(first);
        list.push_back(last);
        unit->n_tiles += tiles(first) + tiles(last);
    } else if (!std::strcmp(argv[1], "prompt tiles first")) {
        std::rotate(list.begin(), prompt, list.end());
    } else if (!std::strcmp(argv[1], "tile missing")) {
        unit->n_tiles -= tiles(last);
        list.pop_back();
    }
    unit->list_begin = (int32_t)plan.ranges.size();
    plan.ranges.insert(plan.ranges.end(), list.begin(), list.end());
    unit->list_end = (int32_t)plan.ranges.size();
    const bool right = !std::strcmp(argv[1], "as it was");
    expect((bs_tilemap_pair_plan(tm, 4, nullptr, nullptr, nullptr) == BS_OK) == right, "the check");
    bs_tilemap_destroy(tm);
    return 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("pair_plan")
    (d / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
                    os.path.join(build.CSRC, "tilemap.cpp"), str(d / "driver.cpp"), "-o", str(d / "driver")], check=True)
    return str(d / "driver")


@pytest.mark.parametrize("what", ["as it was", "compact tiles twice", "prompt tiles twice", "prompt tiles first", "tile missing"])
def test_planted_mistake(driver, what):
    done = subprocess.run([driver, what], capture_output=True, text=True)
    assert done.returncode == 0, done.stderr
