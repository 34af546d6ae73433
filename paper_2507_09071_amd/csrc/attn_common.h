// Device helpers shared by the attention kernels (internal to the library).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tilemap_internal.h"

namespace bs {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kBlockM = 128, kBlockN = 64;

__device__ inline float max_across_halves(float x)
{
    // r[0] = (x.lo, x.lo), r[1] = (x.hi, x.hi): both halves see both values
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

__device__ inline float sum_across_halves(float x)
{
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// What a launch of either prefill kernel is about.  The read-only tile-map arrays go as separate __restrict__ kernel
// parameters, so that loads with wave-uniform addresses go through the scalar cache (they then never wait on the
// vector memory counter that tracks the LDS-direct loads in flight).
struct KernelArgs {
    const void *q, *k, *v;
    void *out;
    int32_t L, G;
    float scale_log2e;  // scale * log2(e): softmax runs in the exp2 domain
    int32_t n_prompt_tiles;   // key tiles that are the prompt in position order; compact tiles of free keys follow, ...
    int32_t text_tile0;       // ... and from here on compact tiles of text keys (n_tiles: none)
    int32_t n_tiles;
    int32_t first_tile;       // a tile that is there for a list without any
    int32_t window, bidir;
    int32_t q_begin;          // q / out hold the query positions q_begin .. L - 1, row r = position q_begin + r
};

// What the lane's query may see (paper Sec. 3.2), in a form that is cheap to apply per tile: intervals of positions and of
// compact slots.  With compact tiles (see the tile-map builder) an image query of a sparse class reads the free keys --
// text and sink keys -- from there and only own-image keys from the prompt's tiles, so that every allowed pair is
// counted once; such queries, text queries and those of Dense heads see one interval of a tile, whatever its keys are, and
// a mask of it is all there is to form (15 instead of 55 vector instructions on a tile with a partial mask: 32 heads of d = 64 at
// 9K tokens 982 -> 967 us for three layers).
struct QueryView {
    int32_t lo, hi;             // positions seen: all up to the query, or those of the own image
    int32_t free_lo, free_hi;   // positions of which the free keys are seen, too (image query of a sparse class, no compact tiles)
    int32_t slot_lo, slot_hi;   // slots seen of the compact tiles that the class walks
    // From the row's record in the map's device copy (two int4, see RowRecord).
    __device__ void init(const int4 &r0, const int4 &r1, int cls, bool compact, const KernelArgs &a)
    {
        // (values first, then choices: a choice of fields would put the records into scratch memory)
        const int pos = r0.x, img_lo = r0.y, img_hi = r0.z, row_free_lo = r0.w, row_free_hi = r1.x, free_before = r1.y, text_lo = r1.z, text_hi = r1.w;
        const bool image = img_hi > img_lo, sees_all = !image || cls == BS_DENSE, own = (cls & 2) != 0;
        // an image query that sees its whole image behaves, for every class, like the image's last query under the causal
        // mask; its image stays visible beyond a window
        const bool whole = image && a.bidir;
        int first = a.window > 0 ? max(0, pos - a.window + 1) : 0;
        first = whole ? min(first, img_lo) : first;
        const int end = whole ? img_hi : pos + 1;
        lo = sees_all ? first : (own ? max(first, img_lo) : 0);
        hi = sees_all || own ? end : 0;
        const bool pattern = !sees_all && !compact;
        free_lo = pattern ? first : 0;
        free_hi = pattern ? end : 0;
        const bool text_slots = cls == BS_INTRA && a.text_tile0 < a.n_tiles;
        const int slot_end = text_slots ? text_hi : (cls == BS_SINK ? row_free_hi : free_before);   // (the own image's are not counted again)
        slot_lo = text_slots ? text_lo : row_free_lo;
        slot_hi = sees_all || !compact ? 0 : slot_end;
    }
};

// Bits [lo, hi) of 64; either may lie outside.
__device__ inline uint64_t bits_between(int lo, int hi)
{
    lo = min(max(lo, 0), 64);
    hi = min(max(hi, 0), 64);
    const uint64_t mask = (~0ull << (lo & 63)) & (~0ull >> ((64 - hi) & 63));   // (lo = 64 or hi = 0: an empty interval)
    return lo < hi ? mask : 0ull;
}

// Bit b set <=> the key in slot b of key tile n is allowed for this lane's query.  item_class: see PairItem::classes;
// tbits / sbits: text keys and sink keys of the tile.
__device__ inline uint64_t allowed_keys(const QueryView &qv, int item_class, uint64_t tbits, uint64_t sbits, int n, const KernelArgs &a)
{
    if (n < a.n_prompt_tiles) {
        const int n0 = n * kBlockN;
        uint64_t allowed = bits_between(qv.lo - n0, qv.hi - n0);
        if (item_class == BS_SINK || item_class == BS_INTRA || item_class == BS_INTRA_SINK)   // (sparse, no compact tiles)
            allowed |= (tbits | ((item_class & 1) ? sbits : 0ull)) & bits_between(qv.free_lo - n0, qv.free_hi - n0);
        return allowed;
    }
    // compact tile: slots are free keys, or text keys, in position order
    const int s0 = (n - (n < a.text_tile0 ? a.n_prompt_tiles : a.text_tile0)) * kBlockN;
    return ((item_class & 1) || n >= a.text_tile0 ? ~0ull : tbits) & bits_between(qv.slot_lo - s0, qv.slot_hi - s0);   // Intra-Image: text keys only
}

// A load from memory that no kernel in flight writes, at a wave-uniform address: through the scalar cache, whatever the
// compiler can prove (a vector load is waited for together with the LDS-direct loads in flight).
template <typename T, typename U>
__device__ inline T scalar_load(const U *p)
{
    static_assert(sizeof(T) == sizeof(U), "");
    return *(const __attribute__((address_space(4))) T *)(uintptr_t)p;
}
typedef int intx2 __attribute__((ext_vector_type(2)));
typedef int intx4 __attribute__((ext_vector_type(4)));

// The row in slot j of query tile m of `head`: its record, its head, whether there is one (the record of a head's own tile says
// so as well).  A stacked tile holds the rows of a group's heads, `head` being the first of them.
struct RowRef { int32_t record, head; bool there; };
__device__ inline RowRef row_of(const StackedRows *rows, bool stacked, int G, int head, int m, int j)
{
    if (!stacked) return {m * kBlockM + j, head, true};
    const intx4 r = scalar_load<intx4>(reinterpret_cast<const intx4 *>(rows));   // first_tile, n_text_tiles, n_text_rows, n_other_rows
    const bool text = m - r.x < r.y;
    const int s = (m - r.x - (text ? 0 : r.y)) * kBlockM + j, t = s / G, n = text ? r.z : r.w;
    return {(text ? scalar_load<int>(&rows->text_slot0) : 0) + min(t, n - 1), head + s - t * G, t < n};
}

// Walks the merged key-tile list of a work unit from its record on (bf16).  The run behind the present one is there before it
// is needed: a walk that asked for it at its turn would wait for the scalar cache, and with it for the operand reads in flight.
// Behind its last tile the walker stays on it (see PairWalker); with more than one tile a step both items skip it there.
template <int KT>
struct TileWalker {
    const int2 *__restrict__ rg;
    int cur, end;                     // the tile, with its states; where its run ends
    int next_begin, next_end;         // the next run, if p <= p_end
    int p, p_end;
    __device__ void next()
    {
        const int t = cur + 16;
        if (t != end) {
            cur = t;
        } else if (p <= p_end) {
            cur = (next_begin << 4) | (next_end & 15);
            end = next_end;
            const intx2 r = scalar_load<intx2>(rg + min(p, p_end - 1));
            next_begin = r.x;
            next_end = r.y;
            ++p;
        } else if (KT > 1) {
            cur &= ~15;
            end = cur + 16;
        }
    }
};

// The same from the list alone, a run at a time (fp32).
struct PairWalker {
    const int2 *__restrict__ rg;
    int p, p_end, n, n_end, states;
    __device__ void load()
    {
        if (p < p_end) {
            const intx2 r = scalar_load<intx2>(rg + __builtin_amdgcn_readfirstlane(p));
            n = __builtin_amdgcn_readfirstlane(r.x);
            n_end = __builtin_amdgcn_readfirstlane(r.y) >> 4;
            states = __builtin_amdgcn_readfirstlane(r.y) & 15;
        }
    }
    __device__ void init(const int2 *__restrict__ ranges, int begin, int end, int first_tile)
    {
        rg = ranges;
        n = first_tile; n_end = 0; states = 0;
        p = __builtin_amdgcn_readfirstlane(begin);
        p_end = __builtin_amdgcn_readfirstlane(end);
        load();
    }
    __device__ bool valid() const { return p < p_end; }
    // Behind its last tile the walker stays on it: what is fetched ahead there is never used, but it has to be a tile that
    // was written (a NaN times a probability of zero is a NaN), and one that is still in the caches.
    __device__ void next()
    {
        if (n + 1 < n_end) ++n;
        else if (++p < p_end) load();
        else p = p_end;
    }
    __device__ int state(int grp) const { return grp ? (states & 3) : (states >> 2); }  // 0 skip 1 partial 2 full
};

}  // namespace bs
