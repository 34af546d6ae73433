// Sparse causal prefill attention for fp32 inputs: the walk of the bf16 kernel with v_mfma_f32_32x32x2f32 end to end, P
// stays fp32.
//
// Bound: the fp32 matrix pipe (157 TFLOP/s; a 64-key tile is 8,192 cycles of it per wave at head dimension 64, 16,384 at
// 128), on short prompts the number of tiles a wave walks one after the other.  A workgroup is four waves of 32 rows of one
// (head, query tile) item.  K and V tiles go global -> LDS straight from the caller's arrays with LDS-direct loads, one
// tile ahead of the one that is computed, with one barrier per tile; keys of compact tiles are gathered
// by the lanes' addresses.  K rows exchange their 16-byte chunks (XOR with the row), so a column read of four channels per
// lane is free of conflicts and feeds four MFMAs; V is read a row at a time.  Few items are cut along their key tiles into
// equal shares for the whole chip, as in the bf16 kernel, and merged by merge_cut_items.
// Measured, 28 heads of dimension 128 over 4 KV heads, all four classes, 1.1K / 2.5K / 9K tokens: 134 / 328 / 2479 us (103
// useful TFLOP/s at 9K); staged through registers between two barriers, one workgroup per item: 242 / 537 / 3454.  Two heads
// of dimension 64, 1.1K tokens: 27 us, 111 with one workgroup per item.
#include "attn_f32.h"

#include <cstddef>

#include "cut_merge.h"

namespace bs {

constexpr int kF32Threads = 256;

template <int D>
constexpr int f32_lds_bytes() { return 2 * 2 * kBlockN * D * 4; }   // two stages of K and V

// Score block layout (two 32x32 MFMA C tiles): lane (hl = lane/32, col = lane%32) holds, for
// query col, keys 32*kb + 8*(v/4) + 4*hl + v%4, v = 0..15.
__device__ inline void apply_mask(floatx16 (&s)[2], uint64_t allowed, int hl)
{
    const uint32_t w[2] = {(uint32_t)allowed >> (4 * hl), (uint32_t)(allowed >> 32) >> (4 * hl)};
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const uint32_t bit = 1u << (8 * (v / 4) + (v % 4));
            s[kb][v] = (w[kb] & bit) ? s[kb][v] : -INFINITY;
        }
}

// Online-softmax update (running max m, running sum l, rescale factor alpha; App. kernel
// Alg. 4) in the exp2 domain: p = exp2(s*c - m*c).  l is the lane's partial sum (its 32 keys);
// the halves are added once, in the epilogue.  MAY_BE_EMPTY guards rows with no allowed key
// so far (m = -inf), which only PARTIAL tiles can produce.
template <bool MAY_BE_EMPTY>
__device__ inline void softmax_block(floatx16 (&s)[2], float &m_run, float &l_run, float &alpha, float c)
{
    float mx = fmaxf(s[0][0], s[0][1]);
#pragma unroll
    for (int v = 2; v < 16; v += 2) mx = fmaxf(fmaxf(mx, s[0][v]), s[0][v + 1]);
#pragma unroll
    for (int v = 0; v < 16; v += 2) mx = fmaxf(fmaxf(mx, s[1][v]), s[1][v + 1]);
    mx = max_across_halves(mx);
    const float m_new = fmaxf(m_run, mx);
    const float m_use = (MAY_BE_EMPTY && m_new == -INFINITY) ? 0.f : m_new;
    const float mc = m_use * c;
    alpha = __builtin_amdgcn_exp2f(fmaf(m_run, c, -mc));  // m_run = -inf -> 0
    float sum0 = 0.f, sum1 = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const float p0 = __builtin_amdgcn_exp2f(fmaf(s[0][v], c, -mc));
        const float p1 = __builtin_amdgcn_exp2f(fmaf(s[1][v], c, -mc));
        s[0][v] = p0; s[1][v] = p1;
        sum0 += p0; sum1 += p1;
    }
    l_run = fmaf(l_run, alpha, sum0 + sum1);
    m_run = m_new;
}

template <int D>
__global__ __launch_bounds__(kF32Threads, D == 64 ? 2 : 1) void attn_prefill_f32(
    KernelArgs a, const uint64_t *__restrict__ map_text_bits, const uint64_t *__restrict__ map_sink_bits,
    const int4 *__restrict__ map_rows, const int32_t *__restrict__ compact_keys, const int4 *__restrict__ items, const int2 *__restrict__ item_ranges, const int32_t *__restrict__ share_off,
    float *__restrict__ cut_results)
{
    constexpr int ROWB = D * 4, TILE = kBlockN * ROWB, NDB = D / 32;
    constexpr int NI = TILE / 1024 / 4;         // LDS-direct instructions per wave and matrix
    constexpr int CHUNKS = ROWB / 16;           // 16-byte chunks of a row
    extern __shared__ __align__(1024) unsigned char lds[];   // stage 0: K, V; stage 1: K, V
    const int tid = threadIdx.x, lane = tid & 63, hl = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int L = a.L, R = L - a.q_begin;

    // a share of the parts, or one item per workgroup
    const int u_begin = share_off ? share_off[blockIdx.x] : (int)blockIdx.x;
    const int u_end = share_off ? share_off[blockIdx.x + 1] : (int)blockIdx.x + 1;

    // LDS-direct loads: instruction j of this wave fills 1 KB, i.e. 64 / CHUNKS rows of the tile
    typedef __attribute__((address_space(3))) void *lds_ptr;
    const uint32_t lds_base = (uint32_t)(uintptr_t)(lds_ptr)lds;
    const int ld_row = wave * NI * (64 / CHUNKS) + lane / CHUNKS, ld_chunk = lane % CHUNKS;   // (of instruction 0)
    auto load16 = [&](const char *src, uint32_t off, uint32_t dst) __attribute__((always_inline)) {
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(src), "s"(dst) : "memory", "m0");
    };
    auto load16_at = [&](const char *src, uint32_t dst) __attribute__((always_inline)) {
        asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(dst) : "memory", "m0");
    };
    auto issue_tile = [&](const char *kh, const char *vh, int n, int stage) __attribute__((always_inline)) {
        const uint32_t dst = lds_base + stage * 2 * TILE + wave * NI * 1024;
        if (n * kBlockN + kBlockN <= L && n < a.n_prompt_tiles) {
            const char *kt = kh + (size_t)n * TILE, *vt = vh + (size_t)n * TILE;
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                const int r = ld_row + j * (64 / CHUNKS);
                load16(kt, r * ROWB + ((ld_chunk ^ (r & 15)) << 4), dst + j * 1024);
                load16(vt, r * ROWB + (ld_chunk << 4), dst + TILE + j * 1024);
            }
            return;
        }
        // the last keys, or a compact tile, whose slots name the keys (a slot without a key is masked): an address of its own
        // for every lane, in 64 bits, since a key may lie anywhere in the KV head
        int key[NI];
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int s = n * kBlockN + ld_row + j * (64 / CHUNKS);
            key[j] = n < a.n_prompt_tiles ? min(s, L - 1) : max(compact_keys[s - a.n_prompt_tiles * kBlockN], 0);
        }
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int r = ld_row + j * (64 / CHUNKS);
            const size_t at = (size_t)key[j] * ROWB;
            load16_at(kh + at + ((ld_chunk ^ (r & 15)) << 4), dst + j * 1024);
            load16_at(vh + at + (ld_chunk << 4), dst + TILE + j * 1024);
        }
    };

    for (int u = u_begin; u < u_end; ++u) {
        const int4 it0 = items[2 * u], it1 = items[2 * u + 1];
        const int head = __builtin_amdgcn_readfirstlane(it0.x), m = __builtin_amdgcn_readfirstlane(it0.y);
        const int T = __builtin_amdgcn_readfirstlane(it1.z), item_class = __builtin_amdgcn_readfirstlane(it1.w) & 7;
        const int slot_id = __builtin_amdgcn_readfirstlane(it1.w >> 16);   // > 0: a part of a cut item
        const int kvh = head / a.G;
        const char *kh = static_cast<const char *>(a.k) + (size_t)kvh * L * ROWB;
        const char *vh = static_cast<const char *>(a.v) + (size_t)kvh * L * ROWB;
        PairWalker w, w_next;   // the tile in work, and the one that is fetched
        w.init(item_ranges, it1.x, it1.y, 0);
        w_next = w;
        if (T > 0) issue_tile(kh, vh, w.n, 0);

        const int4 r0 = map_rows[2 * (m * kBlockM + wave * 32 + col)], r1 = map_rows[2 * (m * kBlockM + wave * 32 + col) + 1];
        const int row = r0.x;   // L: no row here, computed on a copy of the last one and not stored
        floatx4 q[D / 8];   // Q[row][8j + 4hl .. +4)
        {
            const float *qr = static_cast<const float *>(a.q) + ((size_t)head * R + min(row, L - 1) - a.q_begin) * D;
#pragma unroll
            for (int j = 0; j < D / 8; ++j) q[j] = *reinterpret_cast<const floatx4 *>(qr + 8 * j + 4 * hl);
        }
        QueryView qv;
        qv.init(r0, r1, item_class & 3, (item_class & 4) != 0, a);
        // What was loaded for the rows must be here before the loop: the compiler would wait for it inside, and with it
        // for the LDS-direct loads, which it does not know.
#pragma unroll
        for (int j = 0; j < D / 8; ++j) asm volatile("" : "+v"(q[j]));
        asm volatile("" : "+v"(qv.lo), "+v"(qv.hi), "+v"(qv.free_lo), "+v"(qv.free_hi), "+v"(qv.slot_lo), "+v"(qv.slot_hi));
        floatx16 o[NDB];
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[db][v] = 0.f;
        float m_run = -INFINITY, l_run = 0.f;

        for (int k = 0; k < T; ++k) {
            // this wave's loads of tile k have landed; behind the barrier everyone's have, and nobody reads tile k - 1
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");   // (the barrier itself orders no LDS reads for the compiler)
            const int stage = k & 1;
            if (k + 1 < T) {
                w_next.next();
                issue_tile(kh, vh, w_next.n, stage ^ 1);
            }
            const unsigned char *kt = lds + stage * 2 * TILE, *vt = kt + TILE;
            const uint32_t k_lane = col * ROWB + ((hl ^ (col & 15)) << 4);

            floatx16 s[2];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int v = 0; v < 16; ++v) s[kb][v] = 0.f;
#pragma unroll
            for (int j = 0; j < D / 8; ++j)
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) {
                    const floatx4 f = *reinterpret_cast<const floatx4 *>(kt + 32 * kb * ROWB + (k_lane ^ (j << 5)));
#pragma unroll
                    for (int r = 0; r < 4; ++r) s[kb] = __builtin_amdgcn_mfma_f32_32x32x2f32(f[r], q[j][r], s[kb], 0, 0, 0);
                }
            float alpha;
            const int n = __builtin_amdgcn_readfirstlane(w.n);
            if (w.state(0) == 2) {
                softmax_block<false>(s, m_run, l_run, alpha, a.scale_log2e);
            } else {
                apply_mask(s, allowed_keys(qv, item_class, map_text_bits[n], map_sink_bits[n], n, a), hl);
                softmax_block<true>(s, m_run, l_run, alpha, a.scale_log2e);
            }
            if (__any(alpha != 1.f)) {
#pragma unroll
                for (int db = 0; db < NDB; ++db)
#pragma unroll
                    for (int v = 0; v < 16; ++v) o[db][v] *= alpha;
            }
            // contraction slot hl of MFMA (kb, v) is key 32kb + 8(v/4) + 4hl + v%4
            const unsigned char *v_lane = vt + 4 * hl * ROWB + col * 4;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int v = 0; v < 16; ++v)
#pragma unroll
                    for (int db = 0; db < NDB; ++db) {
                        const float x = *reinterpret_cast<const float *>(v_lane + (32 * kb + 8 * (v / 4) + v % 4) * ROWB + 128 * db);
                        o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(x, s[kb][v], o[db], 0, 0, 0);
                    }
            w.next();
        }

        const float l_tot = sum_across_halves(l_run);
        if (slot_id > 0) {
            store_cut_item<D>(cut_results + (size_t)(slot_id - 1) * kCutItemFloats<D>, o, m_run, l_tot, wave, lane);
        } else if (row < L) {
            const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;   // an empty row gives zeros
            float *orow = static_cast<float *>(a.out) + ((size_t)head * R + (row - a.q_begin)) * D;
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    floatx4 x;
#pragma unroll
                    for (int r = 0; r < 4; ++r) x[r] = o[db][4 * g + r] * inv;
                    *reinterpret_cast<floatx4 *>(orow + 32 * db + 8 * g + 4 * hl) = x;
                }
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();   // the next item's first tile goes where this one's last may still be read
    }
}

size_t f32_workspace(const ShareSet &shares, int32_t head_dim)
{
    return (size_t)shares.n_slots * 4 * (head_dim == 128 ? kCutItemFloats<128> : kCutItemFloats<64>);
}

template <int D>
static void launch_f32_dim(const KernelArgs &a, const DeviceMap *d, const ShareSet &sh, void *workspace, hipStream_t st)
{
    const bool shares = sh.n_shares > 0;
    float *cut_results = static_cast<float *>(workspace);
    hipLaunchKernelGGL(attn_prefill_f32<D>, dim3((unsigned)(shares ? sh.n_shares : d->n_pairs)), dim3(kF32Threads), f32_lds_bytes<D>(), st,
                       a, d->text_bits, d->sink_bits, d->rows, d->compact_keys,
                       shares ? sh.items : d->pair_items, shares ? sh.ranges : d->pair_ranges,
                       shares ? sh.off : nullptr, cut_results);
    if (shares && sh.n_cut > 0)
        hipLaunchKernelGGL((merge_cut_items<D, 1, float>), dim3((unsigned)sh.n_cut, 4, D / 32), dim3(64), 0, st, a, sh.cut_items,
                           d->rows, static_cast<const StackedRows *>(nullptr), cut_results);
}

void launch_f32(const KernelArgs &a, const DeviceMap *d, const ShareSet &shares, void *workspace, int32_t head_dim, hipStream_t st)
{
    if (head_dim == 128) launch_f32_dim<128>(a, d, shares, workspace, st);
    else launch_f32_dim<64>(a, d, shares, workspace, st);
}

hipError_t f32_device_setup()
{
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(attn_prefill_f32<128>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, f32_lds_bytes<128>());
    if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(attn_prefill_f32<64>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, f32_lds_bytes<64>());
    return e;
}

}  // namespace bs
