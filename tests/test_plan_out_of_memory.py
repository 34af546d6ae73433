"""A plan that ran out of memory half-way leaves nothing behind: a driver of its own, compiled with the builder's source, lets the
allocation behind k others fail, for every k, and plans again.  The plans that a call uses are then those of a map that never failed."""
import os
import shutil
import subprocess

import pytest

from paper_2507_09071_amd import build

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include "blindsight.h"
#include "tilemap_internal.h"

static long fail_after = -1;   // of the allocations from now on, the one behind that many fails
void *operator new(std::size_t n)
{
    if (fail_after >= 0 && fail_after-- == 0) throw std::bad_alloc();
    if (void *p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }

static void expect(bool ok, const char *what, long k) { if (!ok) { std::fprintf(stderr, "%s (allocation %ld failed)\n", what, k); std::exit(1); } }
template <typename T>
static bool same(const std::vector<T> &a, const std::vector<T> &b)
{
    return a.size() == b.size() && (a.empty() || std::memcmp(a.data(), b.data(), a.size() * sizeof(T)) == 0);
}

static const uint8_t kSparse[8] = {3, 2, 1, 3, 3, 3, 2, 2}, kDense[8] = {0, 0, 0, 0, 3, 2, 1, 0};
static int plan(bs_tilemap *tm, int G) { return bs_tilemap_share_plan(tm, G, 256, nullptr, nullptr, nullptr); }

static bs_tilemap *map(const char *what)   // up to the plan that fails
{
    std::vector<bs_span> spans;
    for (int p = 30; p + 256 < 9000; p += 276) spans.push_back({p, p + 256, 20});
    bs_tilemap *tm = nullptr;
    expect(bs_build_tilemap_ex(spans.data(), (int32_t)spans.size(), 9000, kSparse, 8, 5, 128, 64, BS_MAP_PACK_KEYS, &tm) == BS_OK, "build", -1);
    if (std::strcmp(what, "first plan")) expect(plan(tm, 4) == BS_OK, "plan before", -1);
    if (!std::strcmp(what, "all Dense for the first time")) expect(bs_tilemap_rebind(tm, kDense, 8) == BS_OK, "rebind", -1);
    return tm;
}

int main(int, char **argv)
{
    const int fails_at = !std::strcmp(argv[1], "other group size") ? 8 : (!std::strcmp(argv[1], "one head a unit") ? 0 : 4);
    bs_tilemap *right = map(argv[1]);
    expect(plan(right, 4) == BS_OK, "plan", -1);
    expect(right->stacked.text.n_tiles > 0, "stacked tiles", -1);
    for (long k = 0;; ++k) {
        bs_tilemap *tm = map(argv[1]);
        fail_after = k;
        const int rc = plan(tm, fails_at);
        const bool failed = fail_after < 0;
        fail_after = -1;
        expect(rc == BS_OK || (failed && rc == BS_ENOMEM), "what the call says", k);   // (a sort does without its buffer)
        expect(plan(tm, 4) == BS_OK && bs_tilemap_pair_plan(tm, 4, nullptr, nullptr, nullptr) == BS_OK, "plan again", k);
        expect(same(tm->pairs.items, right->pairs.items) && same(tm->pairs.ranges, right->pairs.ranges), "units", k);
        expect(same(tm->shares.parts, right->shares.parts) && same(tm->shares.ranges, right->shares.ranges) &&
               same(tm->shares.share_off, right->shares.share_off) && same(tm->shares.cut, right->shares.cut) &&
               !std::memcmp(tm->shares.queue_off, right->shares.queue_off, sizeof right->shares.queue_off), "shares", k);
        bs_tilemap_destroy(tm);
        if (!failed) break;
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("plan_out_of_memory")
    (d / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
                    os.path.join(build.CSRC, "tilemap.cpp"), str(d / "driver.cpp"), "-o", str(d / "driver")], check=True)
    return str(d / "driver")


@pytest.mark.parametrize("what", ["first plan", "all Dense for the first time", "other group size", "one head a unit"])
def test_allocation_fails(driver, what):
    done = subprocess.run([driver, what], capture_output=True, text=True)
    assert done.returncode == 0, done.stderr
