// Few query rows against a long KV cache: a decoding step (one row per head) or a handful of draft tokens.
//
// The 128-row query tiles of the prefill kernel are the wrong shape here.  The work is reading K and V once,
// so the bound is HBM, and what the prefill path does around it (a packed copy of V, a K and V tile per two heads, units
// cut over the chip and merged) costs a multiple of the read.  Measured, one row: 28 heads over 39.5K keys of
// 4 KV heads (81 MB) 103 us there, 21.0 us a call here, two kernels (by time stamps, keys from HBM, medians of 36 launches: the waves request
// their first keys at 0.9 us, their last ones have arrived at 13.1 us on average, 6.6 TB/s, and at 15.1 for the last of the 1024 waves, 5.7;
// the first kernel ends at 15.8, the merge runs from 16.9 to 18.8; a kernel that only reads takes 15.3 us for so little); 32 heads over 302K keys of 16 KV heads (2.5 GB) 1060 us there, 412 + 4 us here (6.0
// TB/s; a kernel that only reads reaches 6.2).  How:
//  * the query rows of ALL heads of a GQA group are stacked (head-major) into blocks of 32 rows, the free
//    dimension of a 32x32x16 MFMA, so K and V of a KV head are read once for the whole group;
//  * the keys are split over the chip: grid (parts, KV heads, row groups), about one workgroup per CU; its
//    four waves take every fourth block of 32 keys and run on their own: no barrier in the loop;
//  * K and V blocks go global -> LDS straight from the caller's arrays with 16-byte LDS-direct loads, whole
//    rows at a time, two blocks deep: 32-64 KB in flight per wave, which is what covers the latency of HBM.
//    The 16-byte chunks of a row are exchanged (XOR with the row) so that column reads are free of conflicts;
//  * V^T comes out of LDS through the transposing 64-bit read; scores and softmax are as in the prefill kernel;
//  * the four waves merge through LDS, the parts through a second, small kernel.
// Masks: the rows see keys of the prompt in position order, every allowed pair once; a mask word is formed per
// row and block from the row's bounds, its image and (image rows of sparse heads only) the text / sink bits.  The values of
// every key are multiplied, masked ones by zero: where a tile list would have skipped some, the merge looks for results
// that are not finite (merge_rows_checked).
#include "attn_rows.h"

#include <algorithm>
#include <climits>
#include <type_traits>
#include <cmath>

#include "attn_common.h"
#include "device_map.h"

namespace bs {

constexpr int kRowsWaves = 4, kRowsThreads = 64 * kRowsWaves, kRowsKeys = 32;
constexpr int kRowsMaxRows = 32, kRowsMaxHeads = 512;

// What one query row sees, whatever the head's class: keys first .. last, and for an image row its image.
struct RowBounds {
    int32_t first, last;
    int32_t img_lo, img_hi;   // own image, empty for a text row
};

struct RowsArgs {
    const void *q, *k, *v;
    void *out;
    float *part_o;       // [KV head][row group][part][row][D]
    float2 *part_ml;     // [KV head][row group][part][row]: reference point and row sum of a part
    const uint64_t *text_bits, *sink_bits;
    int32_t L, R, G;
    int32_t k0, blocks_each, blocks_more;   // a part has blocks_each key blocks, the first blocks_more parts one more
    float scale_log2e;
    RowBounds rows[kRowsMaxRows];
    uint32_t classes[kRowsMaxHeads / 16];   // two bits per head
};

template <int D>
struct RowsTraits {
    static constexpr int kRowBytes = D * 2;
    static constexpr int kBlock = kRowsKeys * kRowBytes;    // one block of K or V
    static constexpr int kLoads = kBlock / 1024;            // LDS-direct instructions per block
    static constexpr int kWave = 4 * kBlock;                // two stages of K and V
    static constexpr int kRing = kRowsWaves * kWave;
    static constexpr int kQuery = kRing + kRowsWaves * 64 * 8;   // the query rows, at most 64
    static constexpr int kLds = kQuery + 64 * kRowBytes;
    static constexpr int kPerCu = D == 64 ? 2 : 1;          // workgroups per CU
    // exchange of the 16-byte chunks of row r: rows that share their banks get different chunks
    __device__ static int swizzle(int r) { return D == 128 ? r & 15 : (r >> 1) & 7; }
};

__device__ inline uint32_t mask_below(int x)   // bits [0, x) of 32
{
    return x >= 32 ? ~0u : (x <= 0 ? 0u : (1u << x) - 1u);
}

template <int D, int NRB>
__global__ __launch_bounds__(kRowsThreads, NRB == 1 || D == 64 ? 2 : 1) void attn_rows_bf16(const RowsArgs a)
{
    using TR = RowsTraits<D>;
    constexpr int NT = D / 16, NDB = D / 32, ROWB = TR::kRowBytes, BLK = TR::kBlock, NI = TR::kLoads;
    extern __shared__ __align__(1024) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63, hl = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int part = blockIdx.x, kvh = blockIdx.y, grp = blockIdx.z, n_parts = gridDim.x;
    const int S = a.G * a.R;   // stacked rows of a KV head

    // ---- key blocks of this wave
    const int b_begin = part * a.blocks_each + min(part, a.blocks_more);
    const int b_end = b_begin + a.blocks_each + (part < a.blocks_more ? 1 : 0);
    const int n_steps = b_end - b_begin > wave ? (b_end - b_begin - wave + kRowsWaves - 1) / kRowsWaves : 0;
    const char *kh = static_cast<const char *>(a.k) + (size_t)kvh * a.L * ROWB;
    const char *vh = static_cast<const char *>(a.v) + (size_t)kvh * a.L * ROWB;
    auto block_of = [&](int i) { return a.k0 + b_begin + wave + kRowsWaves * i; };

    // LDS-direct loads of a block: instruction j moves 1 KB, i.e. 1024 / ROWB whole rows; a lane picks the chunk
    // of its row that belongs at its place.
    typedef __attribute__((address_space(3))) void *lds_ptr;
    const uint32_t ring = (uint32_t)(uintptr_t)(lds_ptr)lds + wave * TR::kWave;
    uint32_t voff[NI];
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        const int r = j * (1024 / ROWB) + lane / (ROWB / 16), p = lane % (ROWB / 16);
        voff[j] = r * ROWB + ((p ^ TR::swizzle(r)) << 4);
    }
    auto issue = [&](const char *base, int blk, uint32_t dst) __attribute__((always_inline)) {
        const char *src = base + (size_t)blk * BLK;
        const int rows_left = a.L - blk * kRowsKeys;
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            uint32_t off = voff[j];
            if (rows_left < kRowsKeys) {   // the last block of the cache: rows past its end repeat the last one (masked)
                const int r = j * (1024 / ROWB) + lane / (ROWB / 16);
                off = off % ROWB + min(r, rows_left - 1) * ROWB;
            }
            asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                         :
                         : "v"(off), "s"(src), "s"(dst + j * 1024)
                         : "memory", "m0");
        }
    };
    // The first keys are requested before anything else, so that memory is busy while the rows' bounds and the query rows come
    // (one row of 28 heads over 39.5K keys, a pass of six layers: 136.6 -> 132.7 us).  Not with more rows: what they see comes through
    // vector loads, which would be waited for together with the LDS-direct loads.
    const auto request_first_keys = [&]() __attribute__((always_inline)) {
        if (n_steps > 0) issue(kh, block_of(0), ring);
    };
    if (a.R == 1) request_first_keys();

    // ---- what the rows of this lane see (column `col` of every row block; a slot without a row works on a copy of the
    // last one, never stored).  A vector load here would be waited for together with the LDS-direct loads, which the
    // compiler does not know, so what a decoding step needs comes through scalar loads, and the rest is here before
    // the first of them goes out.
    constexpr int ROWS = NRB * 32;
    int first[NRB], last[NRB], own_lo[NRB], own_hi[NRB];
    bool sees_all[NRB], sinks[NRB];
    auto view = [&](int rb, RowBounds b, int cls) __attribute__((always_inline)) {
        first[rb] = b.first;
        last[rb] = b.last;
        sees_all[rb] = cls == BS_DENSE || b.img_hi == b.img_lo;
        sinks[rb] = cls & 1;
        own_lo[rb] = (cls & 2) ? b.img_lo : 0;
        own_hi[rb] = (cls & 2) ? b.img_hi : 0;
    };
    if (a.R == 1) {
        const int head0 = kvh * a.G + grp * ROWS, word0 = head0 >> 4;   // the classes of ROWS heads: ROWS / 16 + 1 words
        uint32_t words[ROWS / 16 + 1];
#pragma unroll
        for (int i = 0; i < ROWS / 16 + 1; ++i) words[i] = __builtin_amdgcn_readfirstlane(a.classes[min(word0 + i, kRowsMaxHeads / 16 - 1)]);
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) {
            const int head = kvh * a.G + min((grp * NRB + rb) * 32 + col, S - 1);
            uint32_t w = words[0];
#pragma unroll
            for (int i = 1; i < ROWS / 16 + 1; ++i) w = (head >> 4) - word0 == i ? words[i] : w;
            view(rb, a.rows[0], (w >> (2 * (head & 15))) & 3);
        }
    } else {
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) {
            const int s = min((grp * NRB + rb) * 32 + col, S - 1), g = s / a.R, head = kvh * a.G + g;
            view(rb, a.rows[s - g * a.R], (a.classes[head >> 4] >> (2 * (head & 15))) & 3);
            int all = sees_all[rb], snk = sinks[rb];
            asm volatile("" : "+v"(first[rb]), "+v"(last[rb]), "+v"(own_lo[rb]), "+v"(own_hi[rb]), "+v"(all), "+v"(snk));
            sees_all[rb] = all;
            sinks[rb] = snk;
        }
    }
    bool all_see_all = true;
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) all_see_all = all_see_all && __all(sees_all[rb]);

    if (a.R != 1) request_first_keys();

    floatx16 o[NRB][NDB];
    float m_run[NRB], l_run[NRB];
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) {
        m_run[rb] = -INFINITY;
        l_run[rb] = 0.f;
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) o[rb][db][i] = 0.f;
    }

    // at most `kNewer` blocks issued after the one that is waited for
    auto wait_loads = [&](auto newer) __attribute__((always_inline)) {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(decltype(newer)::value * NI) : "memory");
    };
    auto reads_done = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); };
    using N0 = std::integral_constant<int, 0>;
    using N1 = std::integral_constant<int, 1>;
    using N2 = std::integral_constant<int, 2>;
    using N3 = std::integral_constant<int, 3>;

    const uint32_t k_read = wave * TR::kWave + col * ROWB + ((hl ^ TR::swizzle(col)) << 4);
    uint32_t v_read[2];
    {
        const int i = lane & 15, half = (lane >> 4) & 1;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int r = 8 * h + 4 * hl + (i >> 2);
            v_read[h] = wave * TR::kWave + BLK + r * ROWB + (((2 * half + ((i >> 1) & 1)) ^ TR::swizzle(r)) << 4) + (i & 1) * 8;
        }
    }

    // The query rows go to LDS (all waves work on the same ones) in the layout of a K block, with the first blocks of
    // keys on the way: stacked rows of a KV head lie one behind the other.
    {
        const char *qh = static_cast<const char *>(a.q) + (size_t)kvh * S * ROWB;
        constexpr int kPerWave = ROWS * ROWB / 1024 / kRowsWaves;
#pragma unroll
        for (int j = 0; j < kPerWave; ++j) {
            const int i = wave * kPerWave + j, r = i * (1024 / ROWB) + lane / (ROWB / 16), p = lane % (ROWB / 16);
            const uint32_t off = min(grp * ROWS + r, S - 1) * ROWB + ((p ^ TR::swizzle(r & 31)) << 4);
            const uint32_t dst = (uint32_t)(uintptr_t)(lds_ptr)lds + TR::kQuery + i * 1024;
            asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(qh), "s"(dst) : "memory", "m0");
        }
    }
    if (n_steps > 0) issue(vh, block_of(0), ring + BLK);
    if (n_steps > 1) {
        issue(kh, block_of(1), ring + 2 * BLK);
        issue(vh, block_of(1), ring + 3 * BLK);
    }
    if (n_steps > 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * NI) : "memory");   // the query rows (and the first keys)
    else if (n_steps > 0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NI) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    bf16x8 q[NRB][NT];
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
        for (int t = 0; t < NT; ++t)
            q[rb][t] = *reinterpret_cast<const bf16x8 *>(lds + TR::kQuery + rb * 32 * ROWB + ((col * ROWB + ((hl ^ TR::swizzle(col)) << 4)) ^ (t << 5)));

    for (int i = 0; i < n_steps; ++i) {
        const int stage = (i & 1) * 2 * BLK;
        const int blk = block_of(i);
        const bool more = i + 1 < n_steps, more2 = i + 2 < n_steps;

        // ---- S^T = K Q^T
        if (more) wait_loads(N3{}); else wait_loads(N1{});
        floatx16 s[NRB];
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
            for (int e = 0; e < 16; ++e) s[rb][e] = 0.f;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const bf16x8 f = *reinterpret_cast<const bf16x8 *>(lds + ((k_read + stage) ^ (t << 5)));
#pragma unroll
            for (int rb = 0; rb < NRB; ++rb) s[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, q[rb][t], s[rb], 0, 0, 0);
        }
        reads_done();
        if (more2) issue(kh, block_of(i + 2), ring + stage);

        // ---- mask and online softmax (lane: 16 keys 8 (e / 4) + 4 hl + e % 4 of one row per block)
        bf16x8 p[NRB][2];
        const int n0 = blk * kRowsKeys;
        uint32_t tb = 0, sb = 0;
        if (!all_see_all) {
            // scalar loads: a vector load would be waited for together with the LDS-direct loads in flight
            typedef const __attribute__((address_space(4))) uint32_t *scalar_words;
            tb = ((scalar_words)(uintptr_t)a.text_bits)[blk];
            sb = ((scalar_words)(uintptr_t)a.sink_bits)[blk];
        }
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) {
            uint32_t allowed = ~0u;
            if (!sees_all[rb])
                allowed = tb | (sinks[rb] ? sb : 0u) | (mask_below(own_hi[rb] - n0) & ~mask_below(own_lo[rb] - n0));
            allowed &= mask_below(last[rb] + 1 - n0) & ~mask_below(first[rb] - n0);
            if (!__all(allowed == ~0u)) {
                const uint32_t w = allowed >> (4 * hl);
#pragma unroll
                for (int e = 0; e < 16; ++e) s[rb][e] = (w & (1u << (8 * (e / 4) + e % 4))) ? s[rb][e] : -INFINITY;
            }
            float mx = s[rb][0];
#pragma unroll
            for (int e = 1; e < 16; ++e) mx = fmaxf(mx, s[rb][e]);
            mx = max_across_halves(mx);
            // the reference point moves only when the block's maximum exceeds it by 2^8 (any reference gives the
            // same quotient), so the accumulators are rescaled a few times per row and not once per block
            const float c = a.scale_log2e;
            const bool grow = fmaf(mx, c, -(m_run[rb] * c)) > 8.f;
            const float m_new = grow ? mx : m_run[rb];
            const float off = m_new == -INFINITY ? 0.f : -(m_new * c);   // no key so far: p = 0
            const float alpha = grow ? __builtin_amdgcn_exp2f(fmaf(m_run[rb], c, off)) : 1.f;
            float sum = 0.f;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float pv = __builtin_amdgcn_exp2f(fmaf(s[rb][e], c, off));
                sum += pv;
                p[rb][e >> 3][e & 7] = (__bf16)pv;
            }
            l_run[rb] = fmaf(l_run[rb], alpha, sum);
            m_run[rb] = m_new;
            if (__any(alpha != 1.f)) {
#pragma unroll
                for (int db = 0; db < NDB; ++db)
#pragma unroll
                    for (int e = 0; e < 16; ++e) o[rb][db][e] *= alpha;
            }
        }

        // ---- O^T += V^T P^T
        if (more2) wait_loads(N3{}); else if (more) wait_loads(N2{}); else wait_loads(N0{});
        typedef __attribute__((address_space(3))) bf16x4 *lds_bf16x4;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int db = 0; db < NDB; ++db) {
                bf16x8 f;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const bf16x4 x = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
                        (lds_bf16x4)(lds + ((v_read[h] + stage + t * 16 * ROWB) ^ (db << 6))));
#pragma unroll
                    for (int e = 0; e < 4; ++e) f[4 * h + e] = x[e];
                }
#pragma unroll
                for (int rb = 0; rb < NRB; ++rb)
                    o[rb][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, p[rb][t], o[rb][db], 0, 0, 0);
            }
        reads_done();
        if (more2) issue(vh, block_of(i + 2), ring + stage + BLK);
    }

    // ---- merge of the four waves, through LDS: each leaves its rows in its own part of the ring, which nobody else reads, so that
    // one barrier is enough (one row of 28 heads over 39.5K keys, a pass of six layers: 133.6 -> 130.6 us, 17 rows of 40 heads over 7.4K, three
    // layers: 69.1 -> 63.9; three barriers before, and the rows scaled between them)
    constexpr int CH4 = D / 4;
    float2 *ml = reinterpret_cast<float2 *>(lds + TR::kRing);   // [wave][row]
    const int n_rows = min(ROWS, S - grp * ROWS);
    float4 *stage = reinterpret_cast<float4 *>(lds);            // [wave][row][chunks of 4 channels, exchanged]
    constexpr int kStageWave = TR::kWave / 16;
    static_assert(ROWS * CH4 <= kStageWave, "a wave's rows in its part of the ring");
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) {
        const int row = rb * 32 + col;
        const float l = sum_across_halves(l_run[rb]);
        if (hl == 0) ml[wave * ROWS + row] = make_float2(m_run[rb], l);
        if (row < n_rows)
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    stage[wave * kStageWave + row * CH4 + ((db * 8 + 2 * g + hl) ^ (col & (CH4 - 1)))] =
                        make_float4(o[rb][db][4 * g], o[rb][db][4 * g + 1], o[rb][db][4 * g + 2], o[rb][db][4 * g + 3]);
    }
    __syncthreads();
    const size_t slot = ((size_t)(kvh * gridDim.z + grp) * n_parts + part) * ROWS;
    for (int idx = tid; idx < n_rows * CH4; idx += kRowsThreads) {
        const int row = idx / CH4, ch = idx % CH4;
        float2 x[kRowsWaves];
        float4 y[kRowsWaves];
#pragma unroll
        for (int w = 0; w < kRowsWaves; ++w) {
            x[w] = ml[w * ROWS + row];
            y[w] = stage[w * kStageWave + row * CH4 + (ch ^ (row & 31 & (CH4 - 1)))];
        }
        const float m = fmaxf(fmaxf(x[0].x, x[1].x), fmaxf(x[2].x, x[3].x));
        float l = 0.f;
        float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int w = 0; w < kRowsWaves; ++w) {
            const float f = x[w].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((x[w].x - m) * a.scale_log2e);
            l = fmaf(x[w].y, f, l);
            sum.x = fmaf(y[w].x, f, sum.x); sum.y = fmaf(y[w].y, f, sum.y); sum.z = fmaf(y[w].z, f, sum.z); sum.w = fmaf(y[w].w, f, sum.w);
        }
        if (a.part_o == nullptr) {   // one part, and nothing to check
            const float inv = l > 0.f ? 1.f / l : 0.f;
            bf16x4 w;
            w[0] = (__bf16)(sum.x * inv); w[1] = (__bf16)(sum.y * inv); w[2] = (__bf16)(sum.z * inv); w[3] = (__bf16)(sum.w * inv);
            *reinterpret_cast<bf16x4 *>(static_cast<__bf16 *>(a.out) + ((size_t)kvh * S + grp * ROWS + row) * D + 4 * ch) = w;
        } else {
            *reinterpret_cast<float4 *>(a.part_o + (slot + row) * D + 4 * ch) = sum;
            if (ch == 0) a.part_ml[slot + row] = make_float2(m, l);
        }
    }
}

// Merges the parts of a stacked row (blockIdx.x) of a KV head (blockIdx.y): one workgroup; its threads are D / 4 channel quads times the parts in flight.  The
// result is in the first D / 4 threads.
template <int D>
struct MergeLds {
    static constexpr int CH4 = D / 4, LANES = 256 / CH4;   // parts handled side by side
    float4 acc[LANES][CH4];
    float m_wave[4], l_wave[4];
};

// Adds (takes the larger of) what the lanes of a wave hold that have a channel quad in common.
template <int D>
__device__ inline float sum_over_parts(float x)
{
    if constexpr (D == 64) x += __shfl_xor(x, 16, 64);
    return sum_across_halves(x);
}
template <int D>
__device__ inline float max_over_parts(float x)
{
    if constexpr (D == 64) x = fmaxf(x, __shfl_xor(x, 16, 64));
    return max_across_halves(x);
}

template <int D>
__device__ __forceinline__ bf16x4 merge_parts(MergeLds<D> &lds, const float *__restrict__ part_o, const float2 *__restrict__ part_ml,
                                     int groups, int rows_per_group, int n_parts, float scale_log2e)
{
    constexpr int CH4 = MergeLds<D>::CH4, LANES = MergeLds<D>::LANES;
    const int grp = blockIdx.x / (unsigned)rows_per_group, row = blockIdx.x % (unsigned)rows_per_group;
    const size_t base = (size_t)(blockIdx.y * groups + grp) * n_parts * rows_per_group + row;
    const int tid = threadIdx.x;

    // A lane merges its parts to the reference point that they have in common, up to 64 (128) or 128 (256) parts of a row requested together
    // at D = 128 (64); then the lanes of a wave do so, then the waves: a decoding step waits for memory once here, and for one
    // barrier.  With two, exchanges over all lanes for what the lanes of a part agree on, and the parts behind the first 64 in turn:
    // one row of 28 heads over 39.5K keys, 64 parts, a pass of six layers 128.8 us, 126.1 so; two rows of 16 heads over 81K keys, 128
    // parts, two layers 46.9 and 41.4.  (Rows and KV heads are a grid of two dimensions: dividing by the group and the number of
    // rows took 0.3 us a call.)
    const int ch = tid % CH4, p0 = tid / CH4;
    float m = -INFINITY, l = 0.f;
    float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
    // (all: every lane has N parts from `first` on.  A lane behind the last part holds a copy of it, which is replaced: times zero, an
    // infinity in it would be a NaN.  Values, not a branch on whether the part is there: its loads would go behind it.  Replacing them also
    // where all are there: 64 parts 125.7 -> 126.2 us, 128 parts 41.2 -> 42.3.)
    auto merge_some = [&](int first, auto n, auto all) __attribute__((always_inline)) {
        constexpr int N = decltype(n)::value;
        const auto there = [&](int i) { return decltype(all)::value || first + i * LANES < n_parts; };
        float2 x[N];
        float4 y[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const size_t at = base + (size_t)(there(i) ? first + i * LANES : n_parts - 1) * rows_per_group;
            x[i] = part_ml[at];
            y[i] = *reinterpret_cast<const float4 *>(part_o + at * D + 4 * ch);
        }
        const float m_old = m;
#pragma unroll
        for (int i = 0; i < N; ++i) m = fmaxf(m, x[i].x);
        const float old = m_old == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m_old - m) * scale_log2e);
        l *= old;
        sum.x *= old; sum.y *= old; sum.z *= old; sum.w *= old;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const float f = x[i].x == -INFINITY || !there(i) ? 0.f : __builtin_amdgcn_exp2f((x[i].x - m) * scale_log2e);
            l = fmaf(x[i].y, f, l);
            sum.x = fmaf(there(i) ? y[i].x : 0.f, f, sum.x); sum.y = fmaf(there(i) ? y[i].y : 0.f, f, sum.y);
            sum.z = fmaf(there(i) ? y[i].z : 0.f, f, sum.z); sum.w = fmaf(there(i) ? y[i].w : 0.f, f, sum.w);
        }
    };
    using N8 = std::integral_constant<int, 8>;
    using N16 = std::integral_constant<int, 16>;
    if (n_parts == 8 * LANES) {
        merge_some(p0, N8{}, std::true_type{});
    } else if (n_parts < 8 * LANES) {
        merge_some(p0, N8{}, std::false_type{});
    } else {
        int begin = 0;
        for (; begin + 16 * LANES <= n_parts; begin += 16 * LANES) merge_some(begin + p0, N16{}, std::true_type{});
        if (begin < n_parts) merge_some(begin + p0, N16{}, std::false_type{});
    }
    const float m_wave = max_over_parts<D>(m);
    const float f = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m - m_wave) * scale_log2e);
    l = sum_over_parts<D>(l * f);
    sum.x = sum_over_parts<D>(sum.x * f); sum.y = sum_over_parts<D>(sum.y * f); sum.z = sum_over_parts<D>(sum.z * f); sum.w = sum_over_parts<D>(sum.w * f);
    if ((tid & 63) < CH4) lds.acc[tid >> 6][ch] = sum;
    if ((tid & 63) == 0) { lds.m_wave[tid >> 6] = m_wave; lds.l_wave[tid >> 6] = l; }
    __syncthreads();
    bf16x4 w;
    w[0] = w[1] = w[2] = w[3] = (__bf16)0.f;
    if (tid < CH4) {
        const float m_all = fmaxf(fmaxf(lds.m_wave[0], lds.m_wave[1]), fmaxf(lds.m_wave[2], lds.m_wave[3]));
        float l_tot = 0.f;
        float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int i = 0; i < 4; ++i) {   // waves
            const float f = lds.m_wave[i] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((lds.m_wave[i] - m_all) * scale_log2e);
            const float4 y = lds.acc[i][tid];
            l_tot = fmaf(lds.l_wave[i], f, l_tot);
            t.x = fmaf(y.x, f, t.x); t.y = fmaf(y.y, f, t.y); t.z = fmaf(y.z, f, t.z); t.w = fmaf(y.w, f, t.w);
        }
        const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
        w[0] = (__bf16)(t.x * inv); w[1] = (__bf16)(t.y * inv); w[2] = (__bf16)(t.z * inv); w[3] = (__bf16)(t.w * inv);
    }
    return w;
}

template <int D>
__global__ __launch_bounds__(256) void merge_rows(const float *__restrict__ part_o, const float2 *__restrict__ part_ml,
                                                  __bf16 *__restrict__ out, int groups, int rows_per_group,
                                                  int n_parts, float scale_log2e)
{
    __shared__ MergeLds<D> lds;
    const bf16x4 w = merge_parts<D>(lds, part_o, part_ml, groups, rows_per_group, n_parts, scale_log2e);
    if (threadIdx.x < D / 4) *reinterpret_cast<bf16x4 *>(out + ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * D + 4 * threadIdx.x) = w;
}

// The same where rows are handed keys that their head's tile lists skip (see plan_rows).  The attention kernel multiplies
// the values of such a key by a probability of zero, and an infinity or a NaN there is a NaN in the result.  A row whose
// result is not finite is computed again here, a key at a time, from the keys that it sees and nothing else: rare, so
// what counts is that the usual row pays one vote for it (20 rows under 28 heads behind 1K / 39.5K keys: 18.4 / 51.6 us,
// unchecked 18.1 / 51.0; up to 128 keys, one part, take this launch on top: 12.9 -> 17.9, the prefill kernel 20.6).
template <int D>
__global__ __launch_bounds__(256) void merge_rows_checked(const RowsArgs a, int groups, int rows_per_group, int n_parts)
{
    constexpr int CH4 = MergeLds<D>::CH4, LANES = MergeLds<D>::LANES;
    __shared__ MergeLds<D> lds;
    __shared__ float p_key[256];   // probabilities of 256 keys, negative: not seen
    const int tid = threadIdx.x;
    bf16x4 w = merge_parts<D>(lds, a.part_o, a.part_ml, groups, rows_per_group, n_parts, a.scale_log2e);
    const size_t out_row = (size_t)blockIdx.y * gridDim.x + blockIdx.x;   // rows of a head one behind the other
    bool bad = false;
#pragma unroll
    for (int e = 0; e < 4; ++e) bad = bad || !(fabsf((float)w[e]) < INFINITY);
    if (__syncthreads_or(bad)) {
        const int head = blockIdx.y * a.G + blockIdx.x / a.R;
        const RowBounds b = a.rows[blockIdx.x % a.R];
        const int cls = (a.classes[head >> 4] >> (2 * (head & 15))) & 3;
        const bool sees_all = cls == BS_DENSE || b.img_hi == b.img_lo;
        const __bf16 *q = static_cast<const __bf16 *>(a.q) + out_row * D;
        const __bf16 *k = static_cast<const __bf16 *>(a.k) + (size_t)(head / a.G) * a.L * D;
        const __bf16 *v = static_cast<const __bf16 *>(a.v) + (size_t)(head / a.G) * a.L * D;
        const int ch = tid % CH4;
        float m = -INFINITY, l = 0.f;
        float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int n0 = b.first; n0 <= b.last; n0 += 256) {
            const int n = n0 + tid;
            bool seen = n <= b.last;
            if (seen && !sees_all) {
                const bool own = (cls & 2) && n >= b.img_lo && n < b.img_hi;
                const uint64_t free_keys = a.text_bits[n >> 6] | ((cls & 1) ? a.sink_bits[n >> 6] : 0ull);
                seen = own || ((free_keys >> (n & 63)) & 1);
            }
            float s = -INFINITY;
            if (seen) {
                s = 0.f;
                for (int c = 0; c < D; c += 8) {
                    const bf16x8 x = *reinterpret_cast<const bf16x8 *>(q + c), y = *reinterpret_cast<const bf16x8 *>(k + (size_t)n * D + c);
#pragma unroll
                    for (int e = 0; e < 8; ++e) s = fmaf((float)x[e], (float)y[e], s);
                }
            }
            float m_new = s;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) m_new = fmaxf(m_new, __shfl_xor(m_new, off, 64));
            if ((tid & 63) == 0) lds.m_wave[tid >> 6] = m_new;
            __syncthreads();   // (and the probabilities of the last 256 keys have been read)
            m_new = fmaxf(fmaxf(fmaxf(lds.m_wave[0], lds.m_wave[1]), fmaxf(lds.m_wave[2], lds.m_wave[3])), m);
            const float ref = m_new == -INFINITY ? 0.f : m_new;   // no key so far, or none with a number for a score
            p_key[tid] = seen ? __builtin_amdgcn_exp2f((s - ref) * a.scale_log2e) : -1.f;
            const float alpha = __builtin_amdgcn_exp2f((m - ref) * a.scale_log2e);
            m = m_new;
            l *= alpha;
            sum.x *= alpha; sum.y *= alpha; sum.z *= alpha; sum.w *= alpha;
            __syncthreads();
            for (int i = tid / CH4; i < 256; i += LANES) {
                const float p = p_key[i];
                if (p < 0.f) continue;
                const bf16x4 y = *reinterpret_cast<const bf16x4 *>(v + (size_t)(n0 + i) * D + 4 * ch);
                l += p;
                sum.x = fmaf(p, (float)y[0], sum.x); sum.y = fmaf(p, (float)y[1], sum.y);
                sum.z = fmaf(p, (float)y[2], sum.z); sum.w = fmaf(p, (float)y[3], sum.w);
            }
        }
        __syncthreads();
        lds.acc[tid / CH4][ch] = sum;
        if (ch == 0) p_key[tid / CH4] = l;   // the channel lanes of a key hold the same sum
        __syncthreads();
        if (tid < CH4) {
            float4 t = lds.acc[0][tid];
            float l_tot = p_key[0];
            for (int i = 1; i < LANES; ++i) {
                const float4 y = lds.acc[i][tid];
                t.x += y.x; t.y += y.y; t.z += y.z; t.w += y.w;
                l_tot += p_key[i];
            }
            const float inv = l_tot > 0.f ? 1.f / l_tot : (l_tot == 0.f ? 0.f : l_tot);   // (a NaN stays one)
            w[0] = (__bf16)(t.x * inv); w[1] = (__bf16)(t.y * inv); w[2] = (__bf16)(t.z * inv); w[3] = (__bf16)(t.w * inv);
        }
    }
    if (tid < CH4) *reinterpret_cast<bf16x4 *>(static_cast<__bf16 *>(a.out) + out_row * D + 4 * tid) = w;
}

RowsPlan plan_rows(const bs_tilemap *tm, int32_t dtype, int32_t gqa_group, int32_t head_dim, int32_t n_cus)
{
    RowsPlan p;
    const int32_t L = tm->L, R = L - tm->q_begin, n_kv = tm->n_q_heads / gqa_group;
    if (dtype != BS_BF16 || R > kRowsMaxRows || tm->n_q_heads > kRowsMaxHeads) return p;
    if (n_kv > 65535 || (int64_t)L * head_dim * 2 >= INT32_MAX) return p;
    // Up to 32 rows: with 28 / 4 heads and 32 rows a call takes 19 / 26 / 54 / 141 us at 1K / 8K / 39.5K / 141K keys, through
    // the prefill kernel 34 / 42 / 101 / 321; with 32 / 16 heads at 302K 428 and 1074, with 32 / 8 of d = 64 at 9K 22 and 37.
    // (One row: 12 / 12 / 23 / 52 and 36 / 43 / 103 / 315.)  The limit is what the kernel's arguments hold of
    // the rows' bounds, not where the two meet, which is further up.
    // Every block of keys is read for every head.  That is the work when a text row or a Dense head is there (both
    // see every earlier key); rows of images under sparse heads only keep the tile lists of the prefill kernel.
    bool any_dense = false, all_dense = true, any_text = false, any_image = false;
    for (uint8_t c : tm->head_class) (c == BS_DENSE ? any_dense : all_dense) = c == BS_DENSE;
    int32_t first = L, last = -1;
    for (int32_t i = tm->q_begin; i < L; ++i) {
        int32_t lo, hi, img_lo, img_hi;
        row_bounds(tm, i, &lo, &hi, &img_lo, &img_hi);
        (img_hi > img_lo ? any_image : any_text) = true;
        first = std::min(first, lo);
        last = std::max(last, hi);
    }
    if (!any_text && !any_dense) return p;
    p.use = true;
    p.need_bits = any_image && !all_dense;
    p.k0 = first / kRowsKeys;
    p.k1 = last / kRowsKeys + 1;
    const int32_t S = gqa_group * R;
    p.row_blocks = S > 32 ? 2 : 1;
    p.groups = (S + 32 * p.row_blocks - 1) / (32 * p.row_blocks);
    // One workgroup per CU (two at head dimension 64, whose ring takes half the LDS), but no wave without a block.
    const int32_t wgs = n_cus * (head_dim == 64 ? RowsTraits<64>::kPerCu : RowsTraits<128>::kPerCu);
    const int32_t n_blocks = p.k1 - p.k0;
    p.parts = std::max(1, std::min(wgs / std::max(1, n_kv * p.groups), (n_blocks + kRowsWaves - 1) / kRowsWaves));
    // A row of an image may be handed keys here that no tile list of its head names: those of other images under a sparse
    // head, those in front of its window or behind it that other rows see.
    p.check = any_image;
    if (p.parts > 1 || p.check) p.workspace = (size_t)n_kv * p.groups * p.parts * p.row_blocks * 32 * (head_dim + 2) * sizeof(float);
    return p;
}

template <int D>
static void launch_rows_dim(const RowsPlan &plan, const RowsArgs &a, int n_kv, hipStream_t st)
{
    const dim3 grid((unsigned)plan.parts, (unsigned)n_kv, (unsigned)plan.groups), block(kRowsThreads);
    if (plan.row_blocks == 1)
        hipLaunchKernelGGL((attn_rows_bf16<D, 1>), grid, block, RowsTraits<D>::kLds, st, a);
    else
        hipLaunchKernelGGL((attn_rows_bf16<D, 2>), grid, block, RowsTraits<D>::kLds, st, a);
    if (plan.check)
        hipLaunchKernelGGL(merge_rows_checked<D>, dim3((unsigned)(a.G * a.R), (unsigned)n_kv), dim3(256), 0, st, a, plan.groups,
                           plan.row_blocks * 32, plan.parts);
    else if (plan.parts > 1)
        hipLaunchKernelGGL(merge_rows<D>, dim3((unsigned)(a.G * a.R), (unsigned)n_kv), dim3(256), 0, st, a.part_o, a.part_ml,
                           static_cast<__bf16 *>(a.out), plan.groups, plan.row_blocks * 32, plan.parts, a.scale_log2e);
}

void launch_rows(const RowsPlan &plan, const void *q, const void *k, const void *v, void *out, const bs_tilemap *tm,
                 const DeviceMap *d, void *workspace, int32_t gqa_group, int32_t head_dim, float scale, hipStream_t st)
{
    const int32_t n_kv = tm->n_q_heads / gqa_group;
    RowsArgs a{};
    a.q = q; a.k = k; a.v = v; a.out = out;
    if (plan.workspace > 0) {
        a.part_o = static_cast<float *>(workspace);
        a.part_ml = reinterpret_cast<float2 *>(a.part_o + (size_t)n_kv * plan.groups * plan.parts * plan.row_blocks * 32 * head_dim);
    }
    if (plan.need_bits) { a.text_bits = d->text_bits; a.sink_bits = d->sink_bits; }
    a.L = tm->L; a.R = tm->L - tm->q_begin; a.G = gqa_group;
    a.k0 = plan.k0;
    a.blocks_each = (plan.k1 - plan.k0) / plan.parts;
    a.blocks_more = (plan.k1 - plan.k0) % plan.parts;
    a.scale_log2e = scale * 1.4426950408889634f;
    for (int32_t i = 0; i < a.R; ++i)
        row_bounds(tm, tm->q_begin + i, &a.rows[i].first, &a.rows[i].last, &a.rows[i].img_lo, &a.rows[i].img_hi);
    for (int32_t h = 0; h < tm->n_q_heads; ++h) a.classes[h >> 4] |= (uint32_t)tm->head_class[h] << (2 * (h & 15));
    if (head_dim == 128) launch_rows_dim<128>(plan, a, n_kv, st);
    else launch_rows_dim<64>(plan, a, n_kv, st);
}

hipError_t rows_device_setup()
{
    const void *const k128[] = {reinterpret_cast<const void *>(attn_rows_bf16<128, 1>), reinterpret_cast<const void *>(attn_rows_bf16<128, 2>)};
    const void *const k64[] = {reinterpret_cast<const void *>(attn_rows_bf16<64, 1>), reinterpret_cast<const void *>(attn_rows_bf16<64, 2>)};
    for (int i = 0; i < 2; ++i) {
        hipError_t e = hipFuncSetAttribute(k128[i], hipFuncAttributeMaxDynamicSharedMemorySize, RowsTraits<128>::kLds);
        if (e == hipSuccess) e = hipFuncSetAttribute(k64[i], hipFuncAttributeMaxDynamicSharedMemorySize, RowsTraits<64>::kLds);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace bs
