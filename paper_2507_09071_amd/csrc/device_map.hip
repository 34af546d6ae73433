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
#include <condition_variable>
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
// The events order kernels of one device after each other, or tell the host that a kernel has read a pinned buffer: nobody
// looks at memory that a kernel wrote from outside the device on their word, so they need no system-wide fence.  With one
// the next kernel on the stream starts some 3 us later, twice or three times a call: of passes back to back, six decoded
// layers take 135 us (145), 517 rows behind 36K keys 730 (743).
constexpr unsigned kEventFlags = hipEventDisableTiming | hipEventDisableSystemFence;
constexpr size_t kCacheMaxBlocks = 24;
constexpr int kStagingBuffers = 8;
std::mutex g_mem_mutex;
// never destroyed: at process exit the HIP runtime may already be gone
std::vector<CachedBlock> &g_cache = *new std::vector<CachedBlock>();
StagingBuffer g_staging[kStagingBuffers];
int g_staging_next = 0;
std::condition_variable g_staging_freed;   // a buffer is not in use any more
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
        // With more than kStagingBuffers host threads inside an upload the next one waits for its turn.  A thread holds one
        // buffer at a time, until the kernel that reads it is queued, so a buffer comes free.
        std::unique_lock<std::mutex> lock(g_mem_mutex);
        g_staging_freed.wait(lock, [&] {
            for (int i = 0; i < kStagingBuffers && !sb; ++i) {
                const int c = (g_staging_next + i) % kStagingBuffers;
                if (!g_staging[c].in_use) { sb = &g_staging[c]; slot = c; }
            }
            return sb != nullptr;
        });
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
        e = hipEventCreateWithFlags(&sb->done, kEventFlags);
        if (e != hipSuccess) sb->done = nullptr;
    }
    if (e != hipSuccess) {
        staging_abandon({nullptr, slot});
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

hipError_t staging_queued(const Staging &s, hipStream_t st)
{
    StagingBuffer &sb = g_staging[s.slot];
    const hipError_t e = hipEventRecord(sb.done, st);
    std::lock_guard<std::mutex> lock(g_mem_mutex);
    sb.queued = (e == hipSuccess);
    sb.in_use = false;
    g_staging_freed.notify_one();
    return e;
}

hipError_t copy_pending(PendingCopy *copy, hipStream_t st)
{
    if (copy->n == 0) return hipSuccess;
    const hipError_t e = launch_kernel(copy_from_host, dim3((unsigned)std::min<size_t>((copy->n + 255) / 256, 1024)), dim3(256), 0, st,
                                       copy->src, copy->dst, copy->n);
    copy->n = 0;
    if (e == hipSuccess) return staging_queued(copy->staging, st);
    staging_abandon(copy->staging);
    return e;
}

hipError_t staging_commit(const Staging &s, void *dst, size_t bytes, hipStream_t st)
{
    // (whole pieces of 16 bytes: the sizes of both blocks are multiples of 1 MiB)
    PendingCopy copy{s, static_cast<const uint4 *>(s.host), static_cast<uint4 *>(dst), (bytes + 15) / 16};
    if (copy.n == 0) staging_abandon(s);
    return copy_pending(&copy, st);
}

void staging_abandon(const Staging &s)
{
    if (s.slot < 0) return;
    std::lock_guard<std::mutex> lock(g_mem_mutex);
    g_staging[s.slot].in_use = false;
    g_staging_freed.notify_one();
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
    for (const auto &b : d->outgrown) pool_release(d->device, b.first, b.second, d->last_use);
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

struct ExpandArgs {
    const SpanInfo *spans;     // n_spans + 1, the last one a sentinel that starts at L
    const int32_t *offsets;
    int32_t n_offsets, n_spans, L, N0, text_tile0, n_tiles, M, n_free, q_begin, window, sink_len;
    int32_t bidir, regrouped, n_img_rows, m_img;
    int32_t text0;             // text tokens before q_begin
    int4 *rows;
    int32_t *compact_keys;
    uint64_t *text_bits, *sink_bits;
    int32_t n_workgroups;      // behind these, workgroups that bring the work units from a pinned buffer
    const uint4 *copy_src;
    uint4 *copy_dst;
    size_t n_copy;
};

// Number of the first n table entries for which `before` holds (it holds for a prefix of them).
template <typename F>
__device__ inline int32_t partition(int32_t n, F before)
{
    int32_t lo = 0;
    while (n > 0) {
        const int32_t half = n >> 1;
        if (before(lo + half)) { lo += half + 1; n -= half + 1; } else n = half;
    }
    return lo;
}
}

// The device arrays of a map from its span table: what each query row may see, the keys of the compact tiles, the key bit
// masks.  One wave per 64 row slots / key tile; a lane finds its image by bisection.  (Filled on the host and uploaded,
// these arrays were 0.4 ms of host time and 1 MB on a 40K-token prompt, 5 ms and 10 MB at 300K; the kernel takes a few
// microseconds, and a kernel that works on a query tile finds all it has to know about a row in one record.)
__global__ __launch_bounds__(256) void expand_map(const ExpandArgs a)
{
    if ((int32_t)blockIdx.x >= a.n_workgroups) {
        const size_t stride = (size_t)(gridDim.x - a.n_workgroups) * 256;
        for (size_t i = (size_t)(blockIdx.x - a.n_workgroups) * 256 + threadIdx.x; i < a.n_copy; i += stride) a.copy_dst[i] = a.copy_src[i];
        return;
    }
    const int lane = threadIdx.x & 63;
    const int32_t wave = (int32_t)(blockIdx.x * 4 + (threadIdx.x >> 6));
    const SpanInfo *sp = a.spans;
    auto offsets_below = [&](int32_t x) { return partition(a.n_offsets, [&](int32_t i) { return a.offsets[i] < x; }); };
    auto sinks_in = [&](const SpanInfo &s, int32_t x) {   // sink tokens among the first x of an image
        const int32_t p = min(x, s.prefix);
        return p + offsets_below(x) - offsets_below(p);
    };
    auto span_at = [&](int32_t t) { return partition(a.n_spans, [&](int32_t g) { return sp[g].end <= t; }); };

    if (wave < 2 * a.M) {   // ---- 64 row slots
        const int32_t slot = wave * 64 + lane, m = slot >> 7, j = slot & 127;
        int32_t pos = -1;
        if (!a.regrouped) {
            pos = a.q_begin + slot;
            if (pos >= a.L) pos = -1;
        } else if (m < a.m_img) {
            if (slot < a.n_img_rows) {   // image token number (those before q_begin) + slot
                const int32_t x = a.q_begin - a.text0 + slot;
                const int32_t g = partition(a.n_spans, [&](int32_t i) { return sp[i].start - sp[i].text_before <= x; }) - 1;
                pos = sp[g].start + (x - (sp[g].start - sp[g].text_before));
            }
        } else {
            const int32_t x = a.text0 + (m - a.m_img) * 128 + j;   // text token number x
            if (x < sp[a.n_spans].text_before) {
                const int32_t g = partition(a.n_spans + 1, [&](int32_t i) { return sp[i].text_before <= x; });
                pos = sp[g].start - (sp[g].text_before - x);
            }
        }
        RowRecord r{a.L, 0, 0, 0, 0, 0, 0, 0};   // no row
        if (pos >= 0) {
            r.pos = pos;
            const SpanInfo s = sp[span_at(pos)];
            if (s.start <= pos) {   // (the sentinel starts at L)
                r.img_lo = s.start;
                r.img_hi = s.end;
                if (a.n_tiles > a.N0) {   // the free keys up to the last one the row sees; the text keys before its image
                    r.free_before = s.free_before;
                    r.free_hi = s.free_before + sinks_in(s, (a.bidir ? s.end : pos + 1) - s.start);
                    r.text_hi = s.text_before;
                    if (a.window > 0) {   // those before the first one it sees (see QueryView)
                        const int32_t first = a.bidir ? min(max(0, pos - a.window + 1), s.start) : max(0, pos - a.window + 1);
                        const SpanInfo f = sp[span_at(first)];
                        const int32_t x = first - f.start;
                        r.free_lo = f.free_before + (x > 0 ? sinks_in(f, x) : x);
                        r.text_lo = f.text_before + min(x, 0);
                    }
                }
            }
        }
        int4 *out = a.rows + 2 * (size_t)slot;
        out[0] = make_int4(r.pos, r.img_lo, r.img_hi, r.free_lo);
        out[1] = make_int4(r.free_hi, r.free_before, r.text_lo, r.text_hi);
        return;
    }
    const int32_t n = wave - 2 * a.M;   // ---- a key tile
    if (n >= a.n_tiles) return;
    bool text = false, sink = false;
    if (n < a.N0) {
        const int32_t t = n * 64 + lane;
        if (t < a.L) {
            const SpanInfo s = sp[span_at(t)];
            text = s.start > t;
            const int32_t o = t - s.start;
            sink = text ? t < a.sink_len : (o < s.prefix || offsets_below(o + 1) > offsets_below(o));
        }
    } else {
        const int32_t slot = (n - (n < a.text_tile0 ? a.N0 : a.text_tile0)) * 64 + lane;
        int32_t pos = -1;
        if (n >= a.text_tile0) {   // text token number `slot`
            if (slot < sp[a.n_spans].text_before) {
                const int32_t g = partition(a.n_spans + 1, [&](int32_t i) { return sp[i].text_before <= slot; });
                pos = sp[g].start - (sp[g].text_before - slot);
                text = true;
                sink = pos < a.sink_len;
            }
        } else if (slot < a.n_free) {   // free token number `slot`: a sink of the last image that begins before it, or text behind that
            const int32_t g = partition(a.n_spans, [&](int32_t i) { return sp[i].free_before <= slot; }) - 1;
            if (g < 0) {
                pos = slot;
                text = true;
            } else {
                const SpanInfo s = sp[g];
                const int32_t x = slot - s.free_before, sinks = sinks_in(s, s.end - s.start);
                text = x >= sinks;
                if (text) pos = s.end + (x - sinks);
                else if (x < s.prefix) pos = s.start + x;
                else pos = s.start + a.offsets[offsets_below(s.prefix) + (x - s.prefix)];
            }
            sink = text ? pos < a.sink_len : true;
        }
        a.compact_keys[(n - a.N0) * 64 + lane] = pos;
    }
    const uint64_t tb = __ballot(text), sb = __ballot(sink);
    if (lane == 0) {
        a.text_bits[n] = tb;
        a.sink_bits[n] = sb;
    }
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
    e = hipEventCreateWithFlags(&holder->ev, kEventFlags);
    if (e != hipSuccess) { delete d; return fail_hip(e, "hipEventCreate"); }
    d->device = dev;
    d->last_stream = st;
    d->last_use = holder;
    tm->dev = d;
    tm->dev_free = free_device_map;
    return BS_OK;
}

int upload_prompt_part(bs_tilemap *tm, hipStream_t st, PendingCopy *units, const std::function<int()> &stage)
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

    // the span table and the sink offsets go up, the rest is made from them
    const PromptGeometry &P = tm->geo;
    size_t bytes = 0;
    auto section = [&](size_t n) { const size_t at = bytes; bytes = align256(bytes + n); return at; };
    const size_t off_spans = section(P.spans.size() * sizeof(SpanInfo));
    const size_t off_offsets = section(std::max<size_t>(P.offsets.size(), 1) * 4);
    const size_t up_bytes = bytes;
    const bool device_tiles = tm->bm == 128 && tm->bn == 64;   // the kernels' tile sizes: other maps have no device arrays
    const size_t off_rows = section(device_tiles ? (size_t)tm->M * 128 * sizeof(RowRecord) : 0);
    const size_t off_keys = section((size_t)(tm->n_tiles - tm->N0) * 64 * 4);
    const size_t off_tbits = section((size_t)tm->n_tiles * 8);
    const size_t off_sbits = section((size_t)tm->n_tiles * 8);

    Staging sg;
    e = staging_begin(up_bytes, &sg);
    if (e != hipSuccess) return fail_hip(e, "pinned staging buffer");
    unsigned char *host = static_cast<unsigned char *>(sg.host);
    std::memcpy(host + off_spans, P.spans.data(), P.spans.size() * sizeof(SpanInfo));
    if (!P.offsets.empty()) std::memcpy(host + off_offsets, P.offsets.data(), P.offsets.size() * 4);

    void *blob = nullptr;
    size_t blob_cap = 0;
    e = pool_acquire(dev, bytes, st, &blob, &blob_cap);
    if (e != hipSuccess) {
        staging_abandon(sg);
        return fail_hip(e, "hipMalloc(tile map)");
    }
    e = staging_commit(sg, blob, up_bytes, st);
    if (e == hipSuccess && stage && (rc = stage()) != BS_OK) {
        (void)hipFree(blob);
        return rc;
    }
    unsigned char *b = static_cast<unsigned char *>(blob);
    if (e == hipSuccess && device_tiles) {
        ExpandArgs a{};
        a.spans = reinterpret_cast<const SpanInfo *>(b + off_spans);
        a.offsets = reinterpret_cast<const int32_t *>(b + off_offsets);
        a.n_offsets = (int32_t)P.offsets.size();
        a.n_spans = P.n_spans; a.L = tm->L; a.N0 = tm->N0; a.text_tile0 = tm->text_tile0; a.n_tiles = tm->n_tiles; a.M = tm->M;
        a.n_free = P.n_free(tm->L);
        a.q_begin = tm->q_begin; a.window = tm->window; a.sink_len = P.sink_len;
        a.bidir = tm->bidir; a.regrouped = P.regrouped;
        a.n_img_rows = P.n_img_rows; a.m_img = P.m_img;
        a.text0 = P.n_text(tm->q_begin);
        a.rows = reinterpret_cast<int4 *>(b + off_rows);
        a.compact_keys = reinterpret_cast<int32_t *>(b + off_keys);
        a.text_bits = reinterpret_cast<uint64_t *>(b + off_tbits);
        a.sink_bits = reinterpret_cast<uint64_t *>(b + off_sbits);
        const int64_t waves = 2 * (int64_t)tm->M + tm->n_tiles;
        a.n_workgroups = (int32_t)((waves + 3) / 4);
        int32_t copy_wgs = 0;
        if (units && units->n > 0) {
            a.copy_src = units->src; a.copy_dst = units->dst; a.n_copy = units->n;
            copy_wgs = (int32_t)std::min<size_t>((units->n + 255) / 256, 1024);
        }
        e = launch_kernel(expand_map, dim3((unsigned)(a.n_workgroups + copy_wgs)), dim3(256), 0, st, a);
        if (e == hipSuccess && copy_wgs > 0) {
            units->n = 0;
            e = staging_queued(units->staging, st);
        }
    }
    if (e == hipSuccess) e = hipEventRecord(d->last_use->ev, st);
    if (e != hipSuccess) {
        (void)hipFree(blob);
        return fail_hip(e, "tile map upload");
    }
    d->blob = blob;
    d->blob_cap = blob_cap;
    d->rows = reinterpret_cast<const int4 *>(b + off_rows);
    d->compact_keys = reinterpret_cast<const int32_t *>(b + off_keys);
    d->text_bits = reinterpret_cast<const uint64_t *>(b + off_tbits);
    d->sink_bits = reinterpret_cast<const uint64_t *>(b + off_sbits);
    return BS_OK;
}

int upload_binding(bs_tilemap *tm, int32_t kind, int32_t gqa_group, int32_t n_wgs, int32_t n_wgs_too, hipStream_t st, PendingCopy *later)
{
    DeviceMap *d = tm->dev;
    if (!d) return BS_EINVAL;
    if (kind == kBindSolo) gqa_group = 0;   // its units do not depend on it
    if (d->bind_kind == kind && d->bind_G == gqa_group && d->bind_epoch == tm->class_epoch && d->shares_for(n_wgs) &&
        (n_wgs_too == 0 || d->shares_for(n_wgs_too))) return BS_OK;
    SharePlan too;   // the plan for n_wgs_too
    try {
        if (n_wgs_too != 0) {
            bs_plan_shares(tm, gqa_group, n_wgs_too);
            too = tm->shares;
        }
        bs_plan_shares(tm, gqa_group, n_wgs);   // and the pair or solo plan it is made from
    } catch (const std::bad_alloc &) {
        return BS_ENOMEM;
    }
    const PairPlan &plan = kind == kBindPairPlan ? tm->pairs : tm->solo;
    if (plan.ranges.size() >= (size_t)INT32_MAX) return BS_EUNSUPPORTED;
    const SharePlan *const share_plans[2] = {&tm->shares, &too};
    // the parts of the block, one after the other: units, their ranges, queue offsets [9], counters [8 at + 64 B] and the rows of
    // stacked tiles [at + 128 B]; then
    // equal shares: parts, their ranges, share offsets, queue offsets, cut items
    size_t bytes = 0;
    auto section = [&](size_t n) { const size_t at = bytes; bytes = align256(bytes + n); return at; };
    const bool records = kind == kBindPairPlan;
    const size_t unit_bytes = records ? sizeof(UnitRecord) : sizeof(PairItem);
    const size_t off_a = section(plan.items.size() * unit_bytes);
    const size_t off_b = section(std::max<size_t>(plan.ranges.size(), 1) * sizeof(PairRange));
    const size_t off_q = section(256);
    size_t off_s[2][5];
    for (int i = 0; i < 2; ++i) {
        const SharePlan &s = *share_plans[i];
        off_s[i][0] = section(s.parts.size() * unit_bytes);
        off_s[i][1] = section(s.ranges.size() * sizeof(PairRange));
        off_s[i][2] = section(s.share_off.size() * 4);
        off_s[i][3] = section(s.share_off.empty() ? 0 : sizeof s.queue_off);
        off_s[i][4] = section(s.cut.size() * sizeof(CutItem));
    }

    Staging sg;
    hipError_t e = staging_begin(bytes, &sg);
    if (e != hipSuccess) return fail_hip(e, "pinned staging buffer");
    unsigned char *host = static_cast<unsigned char *>(sg.host);
    static_assert(sizeof(PairItem) == 2 * sizeof(int4) && sizeof(PairRange) == sizeof(int2) && sizeof(CutItem) == sizeof(int4), "copied as they are");
    auto put = [&](size_t at, const auto &v) { if (!v.empty()) std::memcpy(host + at, v.data(), v.size() * sizeof(v[0])); };
    auto put_units = [&](size_t at, const std::vector<PairItem> &items, const std::vector<PairRange> &ranges) {
        if (!records) return put(at, items);
        UnitRecord *to = reinterpret_cast<UnitRecord *>(host + at);   // (written once, in order: the pinned buffer is not read)
        for (const PairItem &it : items) {
            UnitRecord r{it.head_a, it.tile_a, it.head_b, it.tile_b, it.n_tiles, it.classes, it.head_a / gqa_group, it.list_end, {}, 0, 0, 0, 0};
            int32_t p = it.list_begin, code = 0, end = 0;   // the run, the tile in it
            if (p < it.list_end) {
                end = ranges[p].end_states;
                code = (ranges[p].begin << 4) | (end & 15);
            }
            for (int32_t i = 0; i < 4; ++i) {   // (as TileWalker<2> goes)
                r.tile[i] = code;
                if (i == 3) break;
                if (code + 16 < end) {
                    code += 16;
                } else if (p + 1 < it.list_end) {
                    end = ranges[++p].end_states;
                    code = (ranges[p].begin << 4) | (end & 15);
                } else {
                    code &= ~15;
                    end = code + 16;
                }
            }
            r.run_end = end;
            r.next = p + 2;
            if (p + 1 < it.list_end) {
                r.next_begin = ranges[p + 1].begin;
                r.next_end_states = ranges[p + 1].end_states;
            }
            *to++ = r;
        }
    };
    put_units(off_a, plan.items, plan.ranges);
    put(off_b, plan.ranges);
    std::memset(host + off_q, 0, 256);
    std::memcpy(host + off_q, plan.queue_off, sizeof plan.queue_off);
    const StackedRows stacked = {tm->M, tm->stacked.text.n_tiles, tm->geo.n_text_rows(), tm->geo.n_other_rows(), tm->geo.m_img * 128};
    std::memcpy(host + off_q + 128, &stacked, sizeof stacked);
    for (int i = 0; i < 2; ++i) {
        const SharePlan &s = *share_plans[i];
        put_units(off_s[i][0], s.parts, s.ranges);
        put(off_s[i][1], s.ranges);
        put(off_s[i][2], s.share_off);
        if (!s.share_off.empty()) std::memcpy(host + off_s[i][3], s.queue_off, sizeof s.queue_off);
        put(off_s[i][4], s.cut);
    }
    // a fresh block every time: kernels of an earlier binding may still be reading the old one,
    // which goes back to the cache behind the map's last-use event
    void *blob = nullptr;
    size_t cap = 0;
    e = pool_acquire(d->device, bytes, st, &blob, &cap);
    if (e != hipSuccess) {
        staging_abandon(sg);
        return fail_hip(e, "hipMalloc(work units)");
    }
    if (later) {
        *later = {sg, static_cast<const uint4 *>(sg.host), static_cast<uint4 *>(blob), (bytes + 15) / 16};
    } else if ((e = staging_commit(sg, blob, bytes, st)) != hipSuccess) {
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
    d->bind_epoch = tm->class_epoch;
    d->pair_items = records ? nullptr : reinterpret_cast<const int4 *>(b + off_a);
    d->units = records ? reinterpret_cast<const UnitRecord *>(b + off_a) : nullptr;
    d->pair_ranges = reinterpret_cast<const int2 *>(b + off_b);
    d->n_pairs = (int32_t)plan.items.size();
    d->n_steps = 0;
    for (const PairItem &it : plan.items) d->n_steps += it.n_tiles;
    d->queue_off = reinterpret_cast<const int32_t *>(b + off_q);
    d->queue_ctr = reinterpret_cast<int32_t *>(b + off_q + 64);
    d->stacked = reinterpret_cast<const StackedRows *>(b + off_q + 128);
    for (int i = 0; i < 2; ++i) {
        const SharePlan &s = *share_plans[i];
        ShareSet &to = d->shares[i];
        to.n_wgs = i == 0 ? n_wgs : n_wgs_too;
        to.n_shares = s.share_off.empty() ? 0 : (int32_t)s.share_off.size() - 1;
        to.n_cut = (int32_t)s.cut.size();
        to.n_slots = s.n_slots;
        to.items = records ? nullptr : reinterpret_cast<const int4 *>(b + off_s[i][0]);
        to.units = records ? reinterpret_cast<const UnitRecord *>(b + off_s[i][0]) : nullptr;
        to.ranges = reinterpret_cast<const int2 *>(b + off_s[i][1]);
        to.off = reinterpret_cast<const int32_t *>(b + off_s[i][2]);
        to.queue_off = reinterpret_cast<const int32_t *>(b + off_s[i][3]);
        to.cut_items = reinterpret_cast<const int4 *>(b + off_s[i][4]);
    }
    return BS_OK;
}

}  // namespace bs
