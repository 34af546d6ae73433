// Merging the partial results of cut work units (internal to the library).
#pragma once
#include <type_traits>

#include "attn_common.h"

namespace bs {

// Results of one item (128 rows) of a part of a cut unit: the output accumulators in register order (wave, channel
// block, quad, lane), then reference point and row sum of every row.  A slot holds the ITEMS items of a part.
template <int D>
constexpr int kCutItemFloats = kBlockM * D + 2 * kBlockM;

template <int D>
__device__ inline void store_cut_item(float *item, const floatx16 (&o)[D / 32], float m_run, float l_tot, int wave, int lane)
{
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            floatx4 w;
#pragma unroll
            for (int r = 0; r < 4; ++r) w[r] = o[db][4 * g + r];
            *reinterpret_cast<floatx4 *>(item + (((wave * (D / 32) + db) * 4 + g) * 64 + lane) * 4) = w;   // 1 KB per instruction
        }
    if (lane < 32) *reinterpret_cast<float2 *>(item + kBlockM * D + (wave * 32 + lane) * 2) = make_float2(m_run, l_tot);
}

// Merges the parts of the cut items: one wave per (cut item, 32 rows, 32 channels), so that some hundred cut items
// keep a thousand waves reading; bf16 rows leave through LDS as 16-byte pieces.
template <int D, int ITEMS, typename OUT>
__global__ __launch_bounds__(64) void merge_cut_items(KernelArgs a, const int4 *__restrict__ cut_items,
                                                      const int4 *__restrict__ map_rows, const StackedRows *__restrict__ stacked,
                                                      const float *__restrict__ cut_results)
{
    constexpr int NDB = D / 32, kStageRow = 64 + 16;   // 32 channels, then the row's position
    __shared__ __align__(16) unsigned char stage[32 * kStageRow];
    const int4 it = cut_items[blockIdx.x];
    const int head = it.x, m = it.y, n_parts = it.w >> 1, item = it.w & 1, wave = blockIdx.y, db = blockIdx.z;
    const int lane = threadIdx.x, hl = lane >> 5, col = lane & 31;
    const int R = a.L - a.q_begin;
    const float *slot = cut_results + ((size_t)it.z * ITEMS + item) * kCutItemFloats<D>;
    const float2 *ml = reinterpret_cast<const float2 *>(slot + kBlockM * D) + wave * 32 + col;
    const floatx4 *src = reinterpret_cast<const floatx4 *>(slot) + (wave * NDB + db) * 256 + lane;
    constexpr size_t kNext = (size_t)ITEMS * kCutItemFloats<D>;
    auto out_row = [&] {   // where the lane's row goes; -1: nowhere
        const RowRef ref = row_of(stacked, stacked && m >= stacked->first_tile, a.G, head, m, wave * 32 + col);
        const int pos = map_rows[2 * ref.record].x;
        return ref.there && pos < a.L ? ref.head * R + (pos - a.q_begin) : -1;
    };
    if constexpr (std::is_same<OUT, __bf16>::value) if (hl == 0) *reinterpret_cast<int32_t *>(stage + col * kStageRow + 64) = out_row();

    // one pass over the parts, with the reference point moving as in the attention loop
    float mx = -INFINITY, l = 0.f;
    floatx4 acc[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) acc[g] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int p = 0; p < n_parts; ++p) {
        const float2 x = ml[p * (kNext / 2)];
        floatx4 y[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) y[g] = src[p * (kNext / 4) + g * 64];
        const float m_new = fmaxf(mx, x.x);
        const float old = mx == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((mx - m_new) * a.scale_log2e);
        const float f = x.x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((x.x - m_new) * a.scale_log2e);
        mx = m_new;
        l = fmaf(l, old, x.y * f);
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[g][r] = fmaf(acc[g][r], old, y[g][r] * f);
    }
    const float inv = l > 0.f ? 1.f / l : 0.f;
    if constexpr (!std::is_same<OUT, __bf16>::value) {
        const int to = out_row();
        if (to >= 0)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *reinterpret_cast<floatx4 *>(static_cast<float *>(a.out) + (size_t)to * D + 32 * db + 8 * g + 4 * hl) = acc[g] * inv;
        return;
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        bf16x4 w;
#pragma unroll
        for (int r = 0; r < 4; ++r) w[r] = (__bf16)(acc[g][r] * inv);
        *reinterpret_cast<bf16x4 *>(stage + col * kStageRow + (8 * g + 4 * hl) * 2) = w;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int r = 16 * j + (lane >> 2), chunk = lane & 3;
        const uint4 piece = *reinterpret_cast<const uint4 *>(stage + r * kStageRow + chunk * 16);
        const int32_t to = *reinterpret_cast<const int32_t *>(stage + r * kStageRow + 64);
        if (to >= 0) *reinterpret_cast<uint4 *>(reinterpret_cast<__bf16 *>(a.out) + (size_t)to * D + 32 * db + chunk * 8) = piece;
    }
}

}  // namespace bs
