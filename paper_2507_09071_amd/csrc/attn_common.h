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
    int32_t n_prompt_tiles;   // key tiles that are the prompt in position order (compact tiles follow)
    int32_t packed, intra_compact;
    int32_t q_begin;          // q / out hold the query positions q_begin .. L - 1, row r = position q_begin + r
};
// What the lane's query may see (paper Sec. 3.2), in a form that is cheap to apply per tile.
// With packed keys (see the tile-map builder) an image query of a sparse class reads the free
// keys -- text and sink keys -- from compact tiles and only own-image keys from the prompt's
// tiles, so that every allowed pair is counted once.
struct QueryView {
    int32_t row;       // last visible position: the query's own (causal), the end of its image (bidirectional images)
    int32_t first;     // first visible position: 0, or the start of the query's sliding window
    int32_t own_lo;    // own image [own_lo, own_hi) if the class attends inside images, else empty
    int32_t own_hi;
    int32_t free_bound;  // packed: free keys at positions <= i (the visible compact slots are [0, free_bound))
    int32_t cfree_lo;    // packed, Intra-Image+Sink: compact slots of the free keys inside the own image
    int32_t cfree_hi;
    bool sees_all;     // text query or Dense head: every earlier key
    bool own_only;     // packed: in the prompt's tiles only own-image keys count for this query
    // From the row's record in the map's device copy (two int4, see RowRecord).
    __device__ void init(const int4 &r0, const int4 &r1, int cls, bool packed, bool intra_compact)
    {
        first = r0.y;
        row = r0.z;
        const bool image = r1.x > r0.w;
        sees_all = !image || cls == BS_DENSE;
        own_lo = own_hi = 0;
        free_bound = cfree_lo = cfree_hi = 0;
        own_only = false;
        if (!sees_all && (cls & 2)) { own_lo = r0.w; own_hi = r1.x; }
        if (packed && !sees_all && (cls != BS_INTRA || intra_compact)) {
            free_bound = r1.y;
            own_only = true;
            if (cls == BS_INTRA_SINK) { cfree_lo = r1.z; cfree_hi = r1.w; }
        }
    }
};

__device__ inline uint64_t bits_below(int x)  // bits [0, x), x in [0, 64]
{
    return x >= 64 ? ~0ull : ((1ull << x) - 1ull);
}
__device__ inline uint64_t bits_between(int lo, int hi)  // bits [lo, hi) clipped to [0, 64)
{
    return bits_below(min(max(hi, 0), 64)) & ~bits_below(min(max(lo, 0), 64));
}

// Bit b set <=> the key in slot b of key tile n is allowed for this lane's query.  tbits / sbits:
// text keys and sink keys of the tile; n_prompt: number of key tiles that are the prompt in
// position order (the tiles after them are compact tiles of free keys).
__device__ inline uint64_t allowed_keys(const QueryView &qv, int cls, uint64_t tbits, uint64_t sbits, int n, int n_prompt)
{
    if (n < n_prompt) {
        const int n0 = n * kBlockN;
        const uint64_t base = qv.sees_all ? ~0ull : (qv.own_only ? 0ull : (tbits | ((cls & 1) ? sbits : 0ull)));
        const uint64_t own = bits_between(qv.own_lo - n0, qv.own_hi - n0);
        return (base | own) & bits_between(qv.first - n0, qv.row - n0 + 1);   // keys first .. row
    }
    // compact tile: slots are free keys in position order, visible up to the row's bound
    const int s0 = (n - n_prompt) * kBlockN;
    const uint64_t base = qv.sees_all ? 0ull : ((cls & 1) ? ~0ull : tbits);   // Intra-Image: text keys only
    const uint64_t excl = bits_between(qv.cfree_lo - s0, qv.cfree_hi - s0);   // counted with the own image
    return base & ~excl & bits_below(min(max(qv.free_bound - s0, 0), 64));
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

// Walks the merged key-tile list of a work unit: runs of [begin, end) with a state per item.
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
    __device__ void init(const int2 *__restrict__ ranges, int begin, int end)
    {
        rg = ranges;
        n = 0; n_end = 0; states = 0;
        p = __builtin_amdgcn_readfirstlane(begin);
        p_end = __builtin_amdgcn_readfirstlane(end);
        load();
    }
    __device__ bool valid() const { return p < p_end; }
    __device__ void next()
    {
        if (++n == n_end) { ++p; load(); }
    }
    __device__ int state(int grp) const { return grp ? (states & 3) : (states >> 2); }  // 0 skip 1 partial 2 full
};

}  // namespace bs
