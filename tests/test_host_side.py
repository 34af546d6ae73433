"""What the library's host side does when a launch fails and when several threads call it, with a stand-in for the HIP runtime (host_runtime.cpp) that runs no kernel:
no GPU is involved."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2507_09071_amd as bs
from paper_2507_09071_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
DRIVER = r"""
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <thread>
#include <vector>
#include "blindsight.h"
#include "host_runtime.h"

static void expect(bool ok, const char *what) { if (!ok) { std::fprintf(stderr, "%s\n", what); std::exit(1); } }

static const bs_span kSpans[3] = {{40, 540, 20}, {552, 852, 20}, {900, 1500, 20}};
static const uint8_t kClasses[4] = {0, 1, 2, 3};
alignas(16) static char kData[16];   // no kernel runs, so nothing is read or written

static bs_tilemap *map(uint32_t flags = BS_MAP_PACK_KEYS)
{
    bs_tilemap *tm = nullptr;
    expect(bs_build_tilemap_ex(kSpans, 3, 1600, kClasses, 4, 8, 128, 64, flags, &tm) == BS_OK, "build");
    return tm;
}

static int call(bs_tilemap *tm, int dtype = BS_BF16)
{
    return bs_attn_prefill(kData, kData, kData, kData, tm, dtype, 4, 2, 128, 0.1f, nullptr);
}

// The units of a run over tiles that the run before packed come with a kernel of their own: the second copy, behind the prompt's.
static void copy_of_units()
{
    uint8_t types[4] = {9, 9, 9, 9};
    double nmse[12];
    host_fail_launch("copy_from_host", 1);
    const int rc = bs_characterize_prompt(kData, kData, kData, kSpans, 3, 1600, 8, BS_BF16, 4, 2, 128, 0.1f, 0.1, BS_MAP_PACK_KEYS, nullptr, 0,
                                          0, types, nmse, nullptr);
    expect(rc == BS_EHIP, "a run whose work units did not arrive is reported");
    expect(std::strstr(bs_last_error(), "an error") != nullptr, "with the runtime's words");
    for (uint8_t t : types) expect(t == 9, "no head type");
    expect(host_launches("attn_prefill_bf16") == 1, "and not launched");
}

// The pre-pass brings the tiles and the work units that the attention kernel reads.
static void pre_pass()
{
    bs_tilemap *tm = map();
    host_fail_launch("pack_kv_tiles", 0);
    expect(call(tm) == BS_EHIP, "a call without its pre-pass is reported");
    expect(host_launches("attn_prefill_bf16") == 0 && host_launches("merge_cut_items") == 0, "nothing is launched behind it");
    const int64_t copied = host_copied_bytes();
    expect(call(tm) == BS_OK && host_launches("attn_prefill_bf16") == 1, "the next call runs");
    expect(host_copied_bytes() > copied, "and brings the units again");
    expect(call(tm) == BS_OK, "once more");
    const int64_t bound = host_copied_bytes();
    expect(bs_tilemap_prepare(tm, BS_BF16, 2, nullptr) == BS_OK && host_copied_bytes() == bound, "which are then bound");
    host_fail_launch("pack_kv_tiles", 0);
    expect(bs_attn_prefill_static(kData, kData, kData, kData, tm, 4, 2, 128, 0.1f, nullptr) == BS_EHIP, "the static entry as well");
    expect(host_launches("attn_prefill_bf16") == 2, "nothing is launched behind it");
    bs_tilemap_destroy(tm);
}

// An error that somebody else's call left behind says nothing about a launch: a pinned buffer is not handed on while a kernel reads it.
static void last_error()
{
    bs_tilemap *tm = map(0);
    expect(call(tm, BS_F32) == BS_OK, "call");
    const uint8_t other[4] = {3, 2, 1, 0};
    expect(bs_tilemap_rebind(tm, other, 4) == BS_OK, "rebind");
    const int copies = host_launches("copy_from_host"), events = host_event_records();
    host_set_last_error(1);
    (void)call(tm, BS_F32);
    expect(host_launches("copy_from_host") == copies + 1, "the units are copied");
    expect(host_event_records() > events, "and an event behind the copy says when their buffer is free");
    bs_tilemap_destroy(tm);
}

// First calls of as many threads as there are pinned buffers, or more, each with a map of its own: all are inside an upload at once.
static void threads(int n, int dtype)
{
    host_malloc_takes(20);
    std::vector<int> rc(n, 1);
    std::vector<std::thread> ts;
    std::atomic<int> ready{0};
    for (int i = 0; i < n; ++i)
        ts.emplace_back([&, i] {
            bs_tilemap *tm = map();
            ++ready;
            while (ready < n) std::this_thread::yield();
            rc[i] = call(tm, dtype);
            if (rc[i] != BS_OK) std::fprintf(stderr, "%d: %s\n", rc[i], bs_last_error());
            bs_tilemap_destroy(tm);
        });
    for (std::thread &t : ts) t.join();
    for (int r : rc) expect(r == BS_OK, "a thread's call");
}

// A call that gets no workspace has its units copied all the same: the map's last use is behind that copy.
static void no_workspace()
{
    bs_tilemap *tm = map();
    host_fail_malloc(2);   // its prompt part and work units, then the workspace
    const int events = host_event_records();
    expect(call(tm) == BS_ENOMEM, "no workspace");
    expect(host_launches("attn_prefill_bf16") == 0, "nothing launched");
    // the span table's buffer, the prompt part, the units' buffer, the units
    expect(host_event_records() == events + 4, "events behind both uploads");
    expect(call(tm) == BS_OK && host_launches("attn_prefill_bf16") == 1, "the next call runs");
    bs_tilemap_destroy(tm);
}

// The same in fp32, for a map whose prompt part is made, and in a preparation.
static void no_workspace_f32()
{
    bs_tilemap *tm = map(0);
    host_fail_malloc(2);
    expect(call(tm, BS_F32) == BS_ENOMEM, "no workspace");
    const uint8_t other[4] = {3, 2, 1, 0};
    expect(bs_tilemap_rebind(tm, other, 4) == BS_OK, "rebind");
    host_fail_malloc(1);
    int events = host_event_records();
    expect(call(tm, BS_F32) == BS_ENOMEM, "no workspace after a rebind");
    expect(host_event_records() == events + 2, "events behind the units");   // their buffer's, the map's
    expect(call(tm, BS_F32) == BS_OK, "the next call runs");
    bs_tilemap *tm2 = map(0);
    host_fail_malloc(1);   // (the block of the units before the rebind is free)
    events = host_event_records();
    expect(bs_tilemap_prepare(tm2, BS_F32, 2, nullptr) == BS_ENOMEM, "no workspace to prepare");
    expect(host_event_records() == events + 4, "events behind both uploads of a preparation");
    bs_tilemap_destroy(tm2);
    bs_tilemap_destroy(tm);
}

int main(int argc, char **argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "copy of the units") copy_of_units();
    else if (what == "pre-pass") pre_pass();
    else if (what == "last error") last_error();
    else if (what == "eight threads, fp32") threads(8, BS_F32);
    else if (what == "eight threads, bf16") threads(8, BS_BF16);
    else if (what == "twelve threads, bf16") threads(12, BS_BF16);
    else if (what == "no workspace") no_workspace();
    else if (what == "no workspace, fp32") no_workspace_f32();
    else return 2;
    return 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("host_side")
    bs.load_library()
    lib = bs.library_path()
    needs = open(lib, "rb").read()
    soname = re.search(rb"libamdhip64\.so\.\d+", needs).group().decode()
    versions = sorted({v.decode() for v in re.findall(rb"\0(hip_\d+\.\d+)\0", needs)})
    (d / "versions").write_text("".join(v + " { global: *; };\n" for v in versions))
    (d / "driver.cpp").write_text(DRIVER)
    rocm = os.path.dirname(os.path.dirname(shutil.which(build.hipcc()) or "/opt/rocm/bin/hipcc"))
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"), "-I", HERE,
                    os.path.join(HERE, "host_runtime.cpp"), f"-Wl,-soname,{soname}", f"-Wl,--version-script={d / 'versions'}",
                    "-o", str(d / soname)], check=True)
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", os.path.join(build.ROOT, "include"), "-I", HERE, str(d / "driver.cpp"), lib,
                    str(d / soname), f"-Wl,-rpath,{d}", "-Wl,--disable-new-dtags", "-Wl,--allow-shlib-undefined", "-o", str(d / "driver")], check=True)
    return str(d / "driver")


@pytest.mark.parametrize("what", ["copy of the units", "pre-pass", "last error", "eight threads, fp32", "eight threads, bf16", "twelve threads, bf16", "no workspace", "no workspace, fp32"])
def test_host_side(driver, what):
    done = subprocess.run([driver, what], capture_output=True, text=True, timeout=60)
    assert done.returncode == 0, done.stderr
