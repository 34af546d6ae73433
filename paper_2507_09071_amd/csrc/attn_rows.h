// Attention of a few query rows against a long KV cache (internal to the library).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tilemap_internal.h"

namespace bs {

struct DeviceMap;

// How a call with few query rows is laid out over the chip (see attn_rows.hip).
struct RowsPlan {
    bool use = false;       // the few-row kernel takes the call
    bool need_bits = false; // some row needs the per-tile text / sink bit masks (the map's device copy)
    bool check = false;     // rows may be handed keys that their tile lists skip (see merge_rows_checked)
    int32_t groups = 1;     // row groups per KV head
    int32_t row_blocks = 1; // 32-row blocks of a group (1 or 2)
    int32_t parts = 1;      // key ranges per (KV head, row group)
    int32_t k0 = 0, k1 = 0; // blocks of 32 keys that the rows see between them
    size_t workspace = 0;   // bytes of partial results (0: one part and no check, results go straight to `out`)
};

// dtype / head_dim / gqa_group as in bs_attn_prefill, already checked; n_cus: compute units of the device.
RowsPlan plan_rows(const bs_tilemap *tm, int32_t dtype, int32_t gqa_group, int32_t head_dim, int32_t n_cus);
// Enqueues the kernels of the plan; `d` is looked at only if plan.need_bits.
void launch_rows(const RowsPlan &plan, const void *q, const void *k, const void *v, void *out, const bs_tilemap *tm,
                 const DeviceMap *d, void *workspace, int32_t gqa_group, int32_t head_dim, float scale, hipStream_t st);
// Raises the kernels' dynamic-LDS limits on the current device.
hipError_t rows_device_setup();

}  // namespace bs
