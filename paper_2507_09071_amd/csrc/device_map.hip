// Device memory for tile maps: block cache, pinned staging, upload of the two parts of a map.
//
// A serving loop builds a tile map per prompt and binds it to one class vector per layer.
// hipMalloc / hipFree per map would cost more than the pre-pass kernels and hipFree would drain
// the device, so the blocks a destroyed map held go back to a small per-process cache instead,
// tagged with an event recorded on the stream that last used them; the next owner's stream waits
// for that event before touching the block.  Host-to-device copies are assembled in place in a
// ring of pinned buffers and copied by a kernel on the caller's stream, so nothing here blocks the host or
// drains the device once the cache is warm.  Cached blocks and pinned buffers are kept until the
// process ends.
#include "device_map.h"

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

namespace bs {

thread_local char g_last_error[256] = "";

int fail_hip(hipError_t e, const char *what)
{
    snprintf(g_last_error, sizeof g_last_error, "%s: %s (%d)", what, hipGetErrorString(e), (int)e);
    (void)hipGetLastError();
    return e == hipErrorOutOfMemory ? BS_ENOMEM : BS_EHIP;
}

int fail_msg(int code, const char *what)
{
    snprintf(g_last_error, sizeof g_last_error, "%s", what);
    return code;
}

namespace {

struct CachedBlock {
    int device;
    void *ptr;
    size_t cap;
    std::shared_ptr<EventHolder> released;   // last use of the block by its previous owner (may be null: never used)
};
struct StagingBuffer {
    void *host = nullptr;
    size_t cap = 0;
    hipEvent_t done = nullptr;   // the copy out of this buffer
    bool queued = false;         // a copy out of this buffer has been queued (done is recorded)
    bool in_use = false;         // a host thread is filling it
};
constexpr size_t kCacheMaxBlocks = 24;
constexpr int kStagingBuffers = 8;
std::mutex g_mem_mutex;
// never destroyed: at process exit the HIP runtime may already be gone
std::vector<CachedBlock> &g_cache = *new std::vector<CachedBlock>();
StagingBuffer g_staging[kStagingBuffers];
int g_staging_next = 0;
std::vector<void *> &g_outgrown = *new std::vector<void *>();   // pinned buffers replaced by larger ones

constexpr size_t kGranule = (size_t)1 << 20;
size_t round_up(size_t x, size_t g) { return (x + g - 1) / g * g; }

}  // namespace

hipError_t pool_acquire(int device, size_t bytes, hipStream_t st, void **out, size_t *cap_out)
{
    const size_t want = round_up(std::max<size_t>(bytes, 1), kGranule);
    {
        std::lock_guard<std::mutex> lock(g_mem_mutex);
        size_t best = g_cache.size();
        for (size_t i = 0; i < g_cache.size(); ++i)
            if (g_cache[i].device == device && g_cache[i].cap >= want && g_cache[i].cap <= 2 * want &&
                (best == g_cache.size() || g_cache[i].cap < g_cache[best].cap))
                best = i;
        if (best < g_cache.size()) {
            const CachedBlock b = g_cache[best];
            g_cache.erase(g_cache.begin() + best);
            const hipError_t e = b.released ? hipStreamWaitEvent(st, b.released->ev, 0) : hipSuccess;
            if (e != hipSuccess) { (void)hipFree(b.ptr); return e; }
            *out = b.ptr; *cap_out = b.cap;
            return hipSuccess;
        }
    }
    hipError_t e = hipMalloc(out, want);
    if (e == hipSuccess) *cap_out = want;
    return e;
}

void pool_release(int device, void *ptr, size_t cap, const std::shared_ptr<EventHolder> &last_use)
{
    if (!ptr) return;
    void *drop = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_mem_mutex);
        g_cache.push_back({device, ptr, cap, last_use});
        if (g_cache.size() > kCacheMaxBlocks) {   // drop the oldest block
            drop = g_cache.front().ptr;
            g_cache.erase(g_cache.begin());
        }
    }
    if (drop) (void)hipFree(drop);   // waits for the block's users; outside the lock
}

hipError_t staging_begin(size_t bytes, Staging *out)
{
    StagingBuffer *sb = nullptr;
    int slot = -1;
    hipEvent_t wait_for = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_mem_mutex);
        for (int i = 0; i < kStagingBuffers && !sb; ++i) {
            const int c = (g_staging_next + i) % kStagingBuffers;
            if (!g_staging[c].in_use) { sb = &g_staging[c]; slot = c; }
        }
        if (!sb) return hipErrorNotReady;   // more than kStagingBuffers host threads inside an upload
        g_staging_next = (slot + 1) % kStagingBuffers;
        sb->in_use = true;
        if (sb->queued) wait_for = sb->done;
    }
    // the copy that last read this buffer must be over (it was queued several uploads ago); the
    // wait happens outside the lock, the buffer is reserved by in_use
    hipError_t e = wait_for ? hipEventSynchronize(wait_for) : hipSuccess;
    if (e == hipSuccess && sb->cap < bytes) {
        // Grow in powers of two and keep the outgrown buffer (hipHostFree drains the device, which
        // would stall the caller behind every kernel it has queued): the buffers a slot has outgrown
        // add up to less than the one it holds.
        size_t cap = kGranule;
        while (cap < bytes) cap *= 2;
        void *grown = nullptr;
        e = hipHostMalloc(&grown, cap, hipHostMallocDefault);
        if (e == hipSuccess) {
            if (sb->host) {
                std::lock_guard<std::mutex> lock(g_mem_mutex);
                g_outgrown.push_back(sb->host);
            }
            sb->host = grown;
            sb->cap = cap;
        }
    }
    if (e == hipSuccess && !sb->done) {
        e = hipEventCreateWithFlags(&sb->done, hipEventDisableTiming);
        if (e != hipSuccess) sb->done = nullptr;
    }
    if (e != hipSuccess) {
        std::lock_guard<std::mutex> lock(g_mem_mutex);
        sb->in_use = false;
        return e;
    }
    out->host = sb->host;
    out->slot = slot;
    return hipSuccess;
}

// The copy is a kernel that reads the pinned buffer over the bus.  hipMemcpyAsync hands copies of more than some
// 16 KB to a DMA engine, and handing the stream over to it and back leaves the GPU idle for 25-60 us per copy (every
// layer of a model has one); a kernel follows its neighbours at once and takes 3 us for a short prompt's work units.
__global__ __launch_bounds__(256) void copy_from_host(const uint4 *__restrict__ src, uint4 *__restrict__ dst, size_t n)
{
    const size_t stride = (size_t)gridDim.x * 256;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) dst[i] = src[i];
}

hipError_t staging_commit(const Staging &s, void *dst, size_t bytes, hipStream_t st)
{
    StagingBuffer &sb = g_staging[s.slot];
    const size_t n = (bytes + 15) / 16;   // both blocks are longer than that: their sizes are multiples of 1 MiB
    hipError_t e = hipSuccess;
    if (n) {
        hipLaunchKernelGGL(copy_from_host, dim3((unsigned)std::min<size_t>((n + 255) / 256, 1024)), dim3(256), 0, st,
                           static_cast<const uint4 *>(sb.host), static_cast<uint4 *>(dst), n);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipEventRecord(sb.done, st);
    std::lock_guard<std::mutex> lock(g_mem_mutex);
    sb.queued = (e == hipSuccess);
    sb.in_use = false;
    return e;
}

void staging_abandon(const Staging &s)
{
    if (s.slot < 0) return;
    std::lock_guard<std::mutex> lock(g_mem_mutex);
    g_staging[s.slot].in_use = false;
}

void free_device_map(DeviceMap *d)
{
    if (!d) return;
    int cur = -1;
    (void)hipGetDevice(&cur);
    if (d->device >= 0 && cur != d->device) (void)hipSetDevice(d->device);
    pool_release(d->device, d->blob, d->blob_cap, d->last_use);
    pool_release(d->device, d->bind_blob, d->bind_cap, d->last_use);
    pool_release(d->device, d->vt_buf, d->vt_bytes, d->last_use);
    if (cur >= 0 && cur != d->device) (void)hipSetDevice(cur);
    delete d;
}

int order_after_last_use(DeviceMap *d, hipStream_t st)
{
    if (d->last_stream == st) return BS_OK;
    // the buffers of the map were last written or read on another stream: order this call after that
    const hipError_t e = hipStreamWaitEvent(st, d->last_use->ev, 0);
    if (e != hipSuccess) return fail_hip(e, "hipStreamWaitEvent");
    d->last_stream = st;
    return BS_OK;
}

namespace {
size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
}

int ensure_device_map(bs_tilemap *tm, hipStream_t st)
{
    if (!tm) return BS_EINVAL;
    if (tm->dev) return BS_OK;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail_hip(e, "hipGetDevice");
    DeviceMap *d = new (std::nothrow) DeviceMap();
    std::shared_ptr<EventHolder> holder;
    try {
        holder = std::make_shared<EventHolder>();
    } catch (const std::bad_alloc &) {
    }
    if (!d || !holder) { delete d; return BS_ENOMEM; }
    e = hipEventCreateWithFlags(&holder->ev, hipEventDisableTiming);
    if (e != hipSuccess) { delete d; return fail_hip(e, "hipEventCreate"); }
    d->device = dev;
    d->last_stream = st;
    d->last_use = holder;
    tm->dev = d;
    tm->dev_free = free_device_map;
    return BS_OK;
}

int upload_prompt_part(bs_tilemap *tm, hipStream_t st)
{
    if (!tm) return BS_EINVAL;
    if (tm->dev && tm->dev->blob) return BS_OK;
    if (tm->bn > 64) return BS_EUNSUPPORTED;  // the per-tile key bit masks are 64 wide
    int rc = ensure_device_map(tm, st);
    if (rc != BS_OK) return rc;
    DeviceMap *d = tm->dev;
    if ((rc = order_after_last_use(d, st)) != BS_OK) return rc;
    const int dev = d->device;
    hipError_t e;

    const int64_t M1 = (int64_t)tm->M + 1;
    int64_t total_ranges = 0;
    for (int c = 0; c < 4; ++c) total_ranges += (int64_t)tm->cls[c].ranges.size();
    if (total_ranges >= INT32_MAX) return BS_EUNSUPPORTED;
    const size_t G1 = tm->spans.size() + 1;

    const size_t off_code = 0;
    const size_t off_rows = align256(off_code + (size_t)tm->L * 4);
    const size_t off_keys = align256(off_rows + tm->row_order.size() * 4);
    const size_t off_fbefore = align256(off_keys + tm->key_order.size() * 4);
    const size_t off_sfree = align256(off_fbefore + std::max<size_t>(tm->free_before.size(), 1) * 4);
    const size_t off_tbits = align256(off_sfree + std::max<size_t>(tm->span_free_range.size(), 2) * 4);
    const size_t off_sbits = align256(off_tbits + (size_t)tm->N * 8);
    const size_t off_spans = align256(off_sbits + (size_t)tm->N * 8);
    const size_t off_rowptr = align256(off_spans + G1 * 8);
    const size_t off_ranges = align256(off_rowptr + (size_t)(4 * M1) * 4);
    const size_t bytes = align256(off_ranges + (size_t)std::max<int64_t>(total_ranges, 1) * 8);

    Staging sg;
    e = staging_begin(bytes, &sg);
    if (e != hipSuccess) return fail_hip(e, "pinned staging buffer");
    unsigned char *host = static_cast<unsigned char *>(sg.host);
    std::memcpy(host + off_code, tm->code.data(), (size_t)tm->L * 4);
    std::memcpy(host + off_rows, tm->row_order.data(), tm->row_order.size() * 4);
    std::memcpy(host + off_keys, tm->key_order.data(), tm->key_order.size() * 4);
    if (!tm->free_before.empty()) std::memcpy(host + off_fbefore, tm->free_before.data(), tm->free_before.size() * 4);
    if (!tm->span_free_range.empty())
        std::memcpy(host + off_sfree, tm->span_free_range.data(), tm->span_free_range.size() * 4);
    else
        std::memset(host + off_sfree, 0, 8);
    std::memcpy(host + off_tbits, tm->text_bits.data(), (size_t)tm->N * 8);
    std::memcpy(host + off_sbits, tm->sink_bits.data(), (size_t)tm->N * 8);
    int2 *sp = reinterpret_cast<int2 *>(host + off_spans);
    sp[0] = make_int2(0, 0);
    for (size_t g = 0; g < tm->spans.size(); ++g) sp[g + 1] = make_int2(tm->spans[g].start, tm->spans[g].end);
    int32_t *rp = reinterpret_cast<int32_t *>(host + off_rowptr);
    int2 *rg = reinterpret_cast<int2 *>(host + off_ranges);
    int64_t base = 0;
    for (int c = 0; c < 4; ++c) {
        const ClassLists &cl = tm->cls[c];
        for (int64_t m = 0; m < M1; ++m) rp[c * M1 + m] = (int32_t)(base + cl.row_ptr[m]);
        static_assert(sizeof(TileRange) == sizeof(int2), "range lists are copied as they are");
        if (!cl.ranges.empty()) std::memcpy(rg + base, cl.ranges.data(), cl.ranges.size() * sizeof(TileRange));
        base += (int64_t)cl.ranges.size();
    }

    void *blob = nullptr;
    size_t blob_cap = 0;
    e = pool_acquire(dev, bytes, st, &blob, &blob_cap);
    if (e != hipSuccess) {
        staging_abandon(sg);
        return fail_hip(e, "hipMalloc(tile map)");
    }
    e = staging_commit(sg, blob, bytes, st);
    if (e == hipSuccess) e = hipEventRecord(d->last_use->ev, st);
    if (e != hipSuccess) {
        (void)hipFree(blob);
        return fail_hip(e, "hipMemcpyAsync(tile map)");
    }
    unsigned char *b = static_cast<unsigned char *>(blob);
    d->blob = blob;
    d->blob_cap = blob_cap;
    d->code = reinterpret_cast<const uint32_t *>(b + off_code);
    d->row_order = reinterpret_cast<const int32_t *>(b + off_rows);
    d->key_order = reinterpret_cast<const int32_t *>(b + off_keys);
    d->free_before = reinterpret_cast<const int32_t *>(b + off_fbefore);
    d->span_free = reinterpret_cast<const int2 *>(b + off_sfree);
    d->text_bits = reinterpret_cast<const uint64_t *>(b + off_tbits);
    d->sink_bits = reinterpret_cast<const uint64_t *>(b + off_sbits);
    d->span_range = reinterpret_cast<const int2 *>(b + off_spans);
    d->row_ptr = reinterpret_cast<const int32_t *>(b + off_rowptr);
    d->ranges = reinterpret_cast<const int2 *>(b + off_ranges);
    return BS_OK;
}

int upload_binding(bs_tilemap *tm, int32_t kind, int32_t gqa_group, int32_t n_wgs, hipStream_t st)
{
    DeviceMap *d = tm->dev;
    if (!d) return BS_EINVAL;
    if (kind == kBindSolo) gqa_group = 0;   // its units do not depend on it
    if (d->bind_kind == kind && d->bind_G == gqa_group && d->bind_wgs == n_wgs && d->bind_epoch == tm->class_epoch) return BS_OK;
    try {
        bs_plan_shares(tm, gqa_group, n_wgs);   // and the pair or solo plan it is made from
    } catch (const std::bad_alloc &) {
        return BS_ENOMEM;
    }
    const PairPlan &plan = kind == kBindPairPlan ? tm->pairs : tm->solo;
    if (plan.ranges.size() >= (size_t)INT32_MAX) return BS_EUNSUPPORTED;
    const SharePlan &shares = tm->shares;
    const bool shared = !shares.share_off.empty();
    // the parts of the block, one after the other: units, their ranges, queue offsets [9] and counters [8 at + 64 B]; then
    // equal shares: parts, their ranges, share offsets, queue offsets, cut items
    size_t bytes = 0;
    auto section = [&](size_t n) { const size_t at = bytes; bytes = align256(bytes + n); return at; };
    const size_t off_a = section(plan.items.size() * sizeof(PairItem));
    const size_t off_b = section(std::max<size_t>(plan.ranges.size(), 1) * sizeof(PairRange));
    const size_t off_q = section(256);
    const size_t off_si = section(shares.parts.size() * sizeof(PairItem));
    const size_t off_sr = section(shares.ranges.size() * sizeof(PairRange));
    const size_t off_so = section(shares.share_off.size() * 4);
    const size_t off_sq = section(sizeof shares.queue_off);
    const size_t off_sc = section(shares.cut.size() * sizeof(CutItem));

    Staging sg;
    hipError_t e = staging_begin(bytes, &sg);
    if (e != hipSuccess) return fail_hip(e, "pinned staging buffer");
    unsigned char *host = static_cast<unsigned char *>(sg.host);
    static_assert(sizeof(PairItem) == 2 * sizeof(int4) && sizeof(PairRange) == sizeof(int2) && sizeof(CutItem) == sizeof(int4), "copied as they are");
    auto put = [&](size_t at, const auto &v) { if (!v.empty()) std::memcpy(host + at, v.data(), v.size() * sizeof(v[0])); };
    put(off_a, plan.items);
    put(off_b, plan.ranges);
    std::memset(host + off_q, 0, 256);
    std::memcpy(host + off_q, plan.queue_off, sizeof plan.queue_off);
    put(off_si, shares.parts);
    put(off_sr, shares.ranges);
    put(off_so, shares.share_off);
    std::memcpy(host + off_sq, shares.queue_off, sizeof shares.queue_off);
    put(off_sc, shares.cut);
    // a fresh block every time: kernels of an earlier binding may still be reading the old one,
    // which goes back to the cache behind the map's last-use event
    void *blob = nullptr;
    size_t cap = 0;
    e = pool_acquire(d->device, bytes, st, &blob, &cap);
    if (e != hipSuccess) {
        staging_abandon(sg);
        return fail_hip(e, "hipMalloc(work units)");
    }
    e = staging_commit(sg, blob, bytes, st);
    if (e != hipSuccess) {
        (void)hipFree(blob);
        return fail_hip(e, "copy of the work units");
    }
    if (d->bind_blob) {
        // the event object is shared with the cached block, and recorded again by later launches
        // of this map: the block then simply waits a little longer than it has to
        pool_release(d->device, d->bind_blob, d->bind_cap, d->last_use);
    }
    unsigned char *b = static_cast<unsigned char *>(blob);
    d->bind_blob = blob;
    d->bind_cap = cap;
    d->bind_kind = kind;
    d->bind_G = gqa_group;
    d->bind_wgs = n_wgs;
    d->bind_epoch = tm->class_epoch;
    d->pair_items = reinterpret_cast<const int4 *>(b + off_a);
    d->pair_ranges = reinterpret_cast<const int2 *>(b + off_b);
    d->n_pairs = (int32_t)plan.items.size();
    d->queue_off = reinterpret_cast<const int32_t *>(b + off_q);
    d->queue_ctr = reinterpret_cast<int32_t *>(b + off_q + 64);
    d->share_items = reinterpret_cast<const int4 *>(b + off_si);
    d->share_ranges = reinterpret_cast<const int2 *>(b + off_sr);
    d->share_off = reinterpret_cast<const int32_t *>(b + off_so);
    d->share_queue_off = reinterpret_cast<const int32_t *>(b + off_sq);
    d->cut_items = reinterpret_cast<const int4 *>(b + off_sc);
    d->n_shares = shared ? (int32_t)shares.share_off.size() - 1 : 0;
    d->n_cut = (int32_t)shares.cut.size();
    d->n_slots = shares.n_slots;
    return BS_OK;
}

}  // namespace bs
