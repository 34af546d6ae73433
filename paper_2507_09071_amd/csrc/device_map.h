// Device-side copy of a tile map and the memory plumbing around it (internal to the library).
//
// A map has two parts on the device.  The PROMPT part depends on the span table and the map
// options only (what each query row may see, key order, key bit masks): a kernel makes it from the span
// table, once per map, and it serves every layer of the model.  The BINDING part depends on the class
// vector the map is bound to (and, for the bf16 kernel, on the GQA group size): the work units.  bs_tilemap_rebind only invalidates the binding part.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <functional>
#include <memory>
#include <tuple>
#include <utility>
#include <vector>

#include "tilemap_internal.h"

namespace bs {

// Detail of the last failure on this thread, for bs_last_error().
extern thread_local char g_last_error[256];

// Records `what` and the HIP error string, clears HIP's sticky error, returns BS_ENOMEM or BS_EHIP.
int fail_hip(hipError_t e, const char *what);
// Records a plain message for bs_last_error() and returns `code`.
int fail_msg(int code, const char *what);

// Queues a kernel and returns the status of that launch alone; hipGetLastError may tell of a call before, of anybody's on the thread.
template <typename... P, typename... A>
hipError_t launch_kernel(void (*kernel)(P...), dim3 grid, dim3 block, size_t lds_bytes, hipStream_t st, const A &...args)
{
    std::tuple<P...> values(args...);
    const hipError_t e = std::apply([&](auto &...v) {
        void *pointers[] = {const_cast<void *>(static_cast<const void *>(&v))...};
        return hipLaunchKernel(reinterpret_cast<const void *>(kernel), grid, block, pointers, lds_bytes, st);
    }, values);
    if (e != hipSuccess) (void)hipGetLastError();   // reported here
    return e;
}

// An event that dies with its last owner (a map, or cached blocks that wait to be reused).
struct EventHolder {
    hipEvent_t ev = nullptr;
    ~EventHolder() { if (ev) (void)hipEventDestroy(ev); }
};

enum BindingKind : int32_t { kBindNone = 0, kBindSolo = 1, kBindPairPlan = 2 };

// A query-tile slot: two int4.  pos = L: a slot without a row.  The slots of compact tiles that a row sees, apart from those
// of its own image: free keys [free_lo, free_before), with the own image's sinks [free_lo, free_hi), text keys [text_lo, text_hi).
struct RowRecord {
    int32_t pos;                  // position of the row; L: no row
    int32_t img_lo, img_hi;       // own image; empty for a text row
    int32_t free_lo, free_hi, free_before;
    int32_t text_lo, text_hi;
};

// Equal shares of the bound units for `n_wgs` workgroups, instead of the queues.
struct ShareSet {
    int32_t n_wgs = 0;                    // 0: not made
    int32_t n_shares = 0;                 // 0: not worth it
    int32_t n_cut = 0, n_slots = 0;
    const int4 *items = nullptr;          // the parts (fp32), ...
    const UnitRecord *units = nullptr;    // ... or (bf16) their records
    const int2 *ranges = nullptr;
    const int32_t *off = nullptr;         // ... [n_shares + 1] the parts of each workgroup, ...
    const int32_t *queue_off = nullptr;   // ... [9] the parts for whoever is done first, ...
    const int4 *cut_items = nullptr;      // ... [n_cut] the items whose results come in parts
};

struct DeviceMap {
    int device = -1;
    // ---- prompt part: one block, uploaded once
    void *blob = nullptr;
    size_t blob_cap = 0;
    const int4 *rows = nullptr;           // [M * 128][2] what the query in each query-tile slot may see (RowRecord)
    const int32_t *compact_keys = nullptr;   // [(n_tiles - N0) * 64] position of each compact slot, -1 = none
    const uint64_t *text_bits = nullptr;  // [n_tiles] text keys of each key tile
    const uint64_t *sink_bits = nullptr;  // [n_tiles] sink keys of each key tile
    // ---- binding part: one block, uploaded again after a rebind / for another kind or group size
    void *bind_blob = nullptr;
    size_t bind_cap = 0;
    int32_t bind_kind = kBindNone;
    int32_t bind_G = 0;
    uint64_t bind_epoch = 0;              // class_epoch of the map the binding was made for
    const int4 *pair_items = nullptr;     // fp32: work units, two int4 each
    const UnitRecord *units = nullptr;    // bf16: their records
    const int2 *pair_ranges = nullptr;
    int32_t n_pairs = 0;
    const int32_t *queue_off = nullptr;   // [9] the units of XCD x are pair_items[queue_off[x] .. queue_off[x + 1])
    ShareSet shares[2];                   // the second for an fp32 map that was prepared, whose head dimension is not known yet
    uint64_t rows_epoch = 0;              // class_epoch and group size of the last call that the few-row kernel took: it needs
    int32_t rows_G = 0;                   // no units, and prepares the map for the static entry as the upload of units does
    int64_t n_steps = 0;                  // key-tile steps of the work units
    const StackedRows *stacked = nullptr; // which rows the stacked tiles among the units hold (bf16)
    int32_t *queue_ctr = nullptr;         // [8] next unit of each queue; cleared by the pre-pass of every call
    // ---- bf16 workspace: packed K tiles, then V^T tiles or packed V tiles (room for all of V^T either way), or partial results, of the last call
    void *vt_buf = nullptr;
    size_t vt_bytes = 0;
    // Workspaces that a larger one took the place of, kept as long as the map: a call of it that was captured into a graph
    // still writes its partial results there when the graph is replayed.
    std::vector<std::pair<void *, size_t>> outgrown;
    hipStream_t last_stream = nullptr;    // stream of the most recent upload / launch (compared, never used)
    std::shared_ptr<EventHolder> last_use;   // recorded after the most recent upload / launch

    const ShareSet *shares_for(int32_t n_wgs) const   // null: not made for so many workgroups
    {
        for (const ShareSet &s : shares)
            if (s.n_wgs == n_wgs) return &s;
        return nullptr;
    }
};

// A device block of at least `bytes`, safe to use in work queued on `st` after this call.  Blocks
// come from a per-process cache of blocks that destroyed maps gave back (no hipMalloc / hipFree in
// a steady serving loop); the stream waits for the previous owner's last use.
hipError_t pool_acquire(int device, size_t bytes, hipStream_t st, void **out, size_t *cap_out);
// Hand a block back; `last_use` is the event after which nobody reads or writes it any more.
void pool_release(int device, void *ptr, size_t cap, const std::shared_ptr<EventHolder> &last_use);

// Host-to-device copies without blocking the host on the device: the caller fills a pinned buffer
// in place (staging_begin), the copy is queued on the caller's stream (staging_commit).
struct Staging {
    void *host = nullptr;
    int slot = -1;
};
hipError_t staging_begin(size_t bytes, Staging *out);
hipError_t staging_commit(const Staging &s, void *dst, size_t bytes, hipStream_t st);
void staging_abandon(const Staging &s);

// A copy that is left to a kernel which the caller launches anyway: `n` pieces of 16 bytes from the pinned buffer.  The caller
// launches that kernel and calls staging_queued, or has the copy done on its own (copy_pending).
struct PendingCopy {
    Staging staging;
    const uint4 *src = nullptr;
    uint4 *dst = nullptr;
    size_t n = 0;                  // 0: nothing to do
};
hipError_t staging_queued(const Staging &s, hipStream_t st);   // the kernel that reads the buffer is on the stream
hipError_t copy_pending(PendingCopy *copy, hipStream_t st);    // a kernel of its own; no-op if there is nothing to do

// The map's device side without any upload: the device it lives on, its last-use event (once per map).
int ensure_device_map(bs_tilemap *tm, hipStream_t st);
// Make the prompt part (once per map) / upload the binding part (when stale) on `st`; no host-side wait.
// `stage` (may be empty), if the prompt part is made now: leaves a copy in *units that goes with the kernel that makes it.  Called
// when the span table's pinned buffer has been handed on: a thread holds one at a time, or eight threads could wait for each other.
int upload_prompt_part(bs_tilemap *tm, hipStream_t st, PendingCopy *units = nullptr, const std::function<int()> &stage = nullptr);
// The shares are cut for n_wgs workgroups, and for n_wgs_too if that is not 0.
// `later` (may be null): leaves the copy to the caller.
int upload_binding(bs_tilemap *tm, int32_t kind, int32_t gqa_group, int32_t n_wgs, int32_t n_wgs_too, hipStream_t st, PendingCopy *later);
// Order work queued on `st` after the map's previous use if that was on another stream.
int order_after_last_use(DeviceMap *d, hipStream_t st);

void free_device_map(DeviceMap *d);

// bs_attn_prefill_ex for a caller that runs several bindings of one map over the same K and V: *kv_packed says in that
// the map's workspace holds the packed tiles of this K and V (its previous call was this one's predecessor), out
// that it holds them now.
int attn_prefill(const void *q, const void *k, const void *v, void *out, bs_tilemap *tm, int32_t dtype, int32_t n_q_heads,
                 int32_t gqa_group, int32_t head_dim, float scale, void *stream, void *ev_main_start, void *ev_main_stop,
                 bool *kv_packed);

}  // namespace bs
