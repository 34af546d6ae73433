// Sparse causal prefill attention for gfx950 (MI355X): one flash-style pass over the key tiles
// the tile map lists for each (head, query tile).
//
// What is computed: paper Sec. 3.1 (softmax(QK^T * scale + mask) V) with the per-class masks of
// Sec. 3.2.  The tiled recurrence (running max, running sum, rescaled output) is the one of
// App. kernel Alg. 4-7; the four subroutines of Alg. 3 collapse into one loop because the tile
// map already says which key tiles a query tile visits and whether a visited tile needs the
// element predicate (PARTIAL) or not (FULL).  One softmax runs per row over the union of all
// visited keys, and the output is divided by the running sum at the end.
//
// Mapping to CDNA4 (bf16 kernel):
//  * a workgroup of eight 64-lane waves owns one work unit: two (head, query tile) items that
//    read the same KV head, four waves each; wave w of a group owns rows 32w..32w+31 of its item
//    and keeps its Q rows in registers for the whole pass;
//  * the launch is one workgroup per CU; a workgroup stays resident and claims unit after unit from
//    the queue of the XCD it runs on (eight queues, filled by the host; see "Work distribution");
//  * scores are produced transposed, S^T = K Q^T, with 32x32x16 bf16 MFMA tiles, so every lane
//    holds 16 keys of ONE query per 32-key block: row max / row sum are in-lane reductions plus
//    one exchange with the lane 32 apart (v_permlane32_swap);
//  * O^T = V^T P^T reuses the probabilities, rounded to bf16, as the B operand; K comes from where the caller has it, V where
//    its tiles are walked a few times and the operand reads transpose; where they are walked often, V^T comes from a
//    pre-pass that writes it per key tile in exactly the layout the LDS reads want (see transposed_values);
//  * K and V^T tiles travel global -> LDS with 16-byte LDS-direct loads (no VGPR staging) into a
//    ring of 4 K + 4 V^T slots shared by the two groups; ONE barrier per key tile, placed so that
//    on every SIMD one wave runs its matrix phase while the other runs its vector phase;
//  * PARTIAL tiles build one 64-bit allowed-key word per lane from the intervals that the query sees (and, for sparse
//    classes without compact tiles, per-tile text/sink bit masks), then test one bit per score.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <type_traits>
#include <vector>

#include "attn_common.h"
#include "attn_f32.h"
#include "attn_rows.h"
#include "cut_merge.h"
#include "device_map.h"
#include "tilemap_internal.h"

namespace bs {

// Scores of keys that the lane's query may not see become -inf, in place, two instructions per score: the allowed bit is
// spread over a word (0 / all ones) and a bit-field insert then keeps the score or takes -inf.  One statement, so that
// the scheduler cannot hoist the 32 bit tests in front of the 32 selects (32 registers of pressure in a kernel that has none
// to spare).
__device__ inline void apply_mask(floatx16 &s0, floatx16 &s1, uint64_t allowed, int hl)
{
    const uint32_t w[2] = {(uint32_t)allowed >> (4 * hl), (uint32_t)(allowed >> 32) >> (4 * hl)};
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            uint32_t t;
            float x = kb ? s1[v] : s0[v];
            asm("v_bfe_i32 %1, %2, %3, 1\n\t"
                "v_bfi_b32 %0, %1, %0, %4"
                : "+v"(x), "=&v"(t)
                : "v"(w[kb]), "n"(8 * (v / 4) + (v % 4)), "v"(-INFINITY));
            (kb ? s1 : s0)[v] = x;
        }
}

// Online softmax of one tile: the scores are only read and the probabilities go straight into the bf16 B operands of
// the P.V MFMAs: contraction slot e of MFMA group (kb, t) is score
// v = 8t + e of block kb, i.e. key 32kb + 16t + {4hl..4hl+3, 8+4hl..8+4hl+3}[e].  Masked scores are -inf; a row with `drop`
// sees none of the tile's keys: it keeps its running maximum and gets p = 0 through an infinite offset.
// Fast path: the probabilities are first formed against the reference point the row already
// has, without looking for the tile maximum.  Any reference gives the same quotient O / l as long as
// nothing overflows, so this is exact whenever the row sums of the tile stay below kFastLimit -- which
// they do on almost every tile after a row's first (scores of neighbouring tiles differ by a few units in
// the exp2 domain, not by 16).  A wave in which some lane's sum is too large, infinite or NaN repeats the tile on the general
// path, which moves the reference; one with a row that has no reference yet (m = -inf) goes there at once.  alpha: what the
// output tile is multiplied by.  PARTIAL tiles take the fast path as FULL ones do: 220 vector instructions instead of 255,
// 120 instead of 155 where the wave's queries see all keys or none (chat_8k of the timed calls 1052 -> 1035 us, prompt_36k
// 15777 -> 15650, window_27k 1711 -> 1698).  Two copies of the general path: with one that both branches reach, the compiler
// straightens the branches and spills 80 registers.
template <int KT>   // tiles of 64 keys, each with a `drop` of its own
__device__ __forceinline__ void softmax_general(const floatx16 (&s)[2 * KT], bf16x8 (&pf)[2 * KT][2], float &m_run, float &l_run,
                                                float &alpha, float c, const bool (&drop)[KT])
{
    float mxl = -INFINITY;
#pragma unroll
    for (int t = 0; t < KT; ++t) {
        // four independent max chains
        float mx[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) mx[i] = fmaxf(s[2 * t + (i >> 1)][8 * (i & 1)], s[2 * t + (i >> 1)][8 * (i & 1) + 1]);
#pragma unroll
        for (int v = 2; v < 8; v += 2)
#pragma unroll
            for (int i = 0; i < 4; ++i) mx[i] = fmaxf(fmaxf(mx[i], s[2 * t + (i >> 1)][8 * (i & 1) + v]), s[2 * t + (i >> 1)][8 * (i & 1) + v + 1]);
        const float mxt = fmaxf(fmaxf(mx[0], mx[1]), fmaxf(mx[2], mx[3]));
        mxl = t == 0 ? (drop[t] ? -INFINITY : mxt) : fmaxf(mxl, drop[t] ? -INFINITY : mxt);
    }
    mxl = max_across_halves(mxl);   // (the two halves hold keys of one query and drop alike)
    // Lazy reference point: the running reference m only moves when the tile maximum exceeds it
    // by more than kLazyLog2 (in the exp2 domain), so p <= 2^kLazyLog2 instead of p <= 1.  The
    // result is the same quotient O / l; what changes is that alpha is exactly 1 on almost every
    // tile after the first few, and the rescaling of the 64 output accumulators is skipped.
    constexpr float kLazyLog2 = 8.f;
    const bool grow = fmaf(mxl, c, -(m_run * c)) > kLazyLog2;   // m_run = -inf, mxl finite: +inf > 8
    const float m_new = grow ? mxl : m_run;                     // both -inf: NaN > 8 is false
    const float m_use = m_new == -INFINITY ? 0.f : m_new;       // no key seen so far: p = 0
    const float mc = m_use * c;
    alpha = grow ? __builtin_amdgcn_exp2f(fmaf(m_run, c, -mc)) : 1.f;     // m_run = -inf -> 0
    float sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < 2 * KT; ++kb) {
        const float off = drop[kb / 2] ? -INFINITY : -mc;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float pv = __builtin_amdgcn_exp2f(fmaf(s[kb][8 * t + e], c, off));
                sum[e & 3] += pv;
                pf[kb][t][e] = (__bf16)pv;
            }
    }
    l_run = fmaf(l_run, alpha, (sum[0] + sum[1]) + (sum[2] + sum[3]));
    m_run = m_new;
}

template <int KT>
__device__ __forceinline__ void softmax_pack(const floatx16 (&s)[2 * KT], bf16x8 (&pf)[2 * KT][2], float &m_run, float &l_run,
                                             float &alpha, float c, const bool (&drop)[KT])
{
    constexpr float kFastLimit = 65536.f;
    float off[KT];   // m = -inf: +inf, no reference yet
    bool all_dropped = true;
#pragma unroll
    for (int t = 0; t < KT; ++t) {
        off[t] = drop[t] ? -INFINITY : -(m_run * c);
        all_dropped = all_dropped && drop[t];
    }
    if (__any(KT == 1 ? off[0] == INFINITY : !all_dropped && m_run == -INFINITY)) {
        softmax_general<KT>(s, pf, m_run, l_run, alpha, c, drop);
    } else {
        float sum[4];
#pragma unroll
        for (int kb = 0; kb < 2 * KT; ++kb)
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float pv = __builtin_amdgcn_exp2f(fmaf(s[kb][8 * t + e], c, off[kb / 2]));
                    sum[e & 3] = kb + t == 0 && e < 4 ? pv : sum[e & 3] + pv;
                    pf[kb][t][e] = (__bf16)pv;
                }
        const float tile_sum = (sum[0] + sum[1]) + (sum[2] + sum[3]);
        if (!__any(!(tile_sum <= kFastLimit))) {
            l_run += tile_sum;
            alpha = 1.f;
        } else {
            softmax_general<KT>(s, pf, m_run, l_run, alpha, c, drop);
        }
    }
}

typedef __attribute__((address_space(3))) void *lds_void_ptr;
typedef const __attribute__((address_space(1))) void *global_void_ptr;

// ------------------------------------------------------------------------------------ bf16
//
// LDS operand reads of the MFMA phase are issued through inline asm and waited for by hand
// (lds_wait<N>): the compiler would otherwise tie every LDS read to the LDS-direct loads that
// are in flight into the other ring slot and drain the vector-memory counter before it.

template <int OFFSET>
__device__ inline void lds_read_b128(bf16x8 &dst, uint32_t addr)
{
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFFSET));
}

// The transposing read of four keys: a lane gets the values that these keys have in one channel.
template <int OFFSET>
__device__ inline void lds_read_tr_b64(bf16x4 &dst, uint32_t addr)
{
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFFSET));
}

// Wait until at most N LDS operations are outstanding.  The operands tie the wait to the
// registers it protects, so their consumers cannot be scheduled above it.
template <int N>
__device__ inline void lds_wait(bf16x8 (&a)[4])
{
    asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]) : "n"(N));
}

// The MFMAs of the matrix phase are asm as well: together with the asm reads and waits they
// form one chain of volatile statements, which the compiler keeps in program order, and the
// accumulator is an in/out operand, so it is updated in place (no copies of the 64 output
// registers).  The compiler does not see a matrix instruction here, so the wait states between
// the last MFMA writing an accumulator and the first vector instruction reading it are seen to
// by hand: other work of at least that length at the end of the chain, mfma_drain behind a unit's last step.
__device__ inline void mfma_acc(floatx16 &c, const bf16x8 &a, const bf16x8 &b)
{
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}
__device__ inline void mfma_set(floatx16 &c, const bf16x8 &a, const bf16x8 &b)   // c = a b
{
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(c) : "v"(a), "v"(b));
}
// 16 wait states: more than the 8 passes of a 32x32x16 MFMA plus the result write-back.
__device__ inline void mfma_drain(floatx16 &c0, floatx16 &c1)
{
    asm volatile("s_nop 15" : "+v"(c0), "+v"(c1));
}


// LDS tile layouts of the bf16 kernel.  V^T is written like that by the pre-pass below and copied verbatim by the kernel's
// LDS-direct loads; those of K, and of V where it is not transposed, pick it from rows of keys.  Everything an MFMA operand read selects
// at compile time (head-dim slice, key block, key group, channel block) is an immediate offset
// from a per-lane base address (two for K).
//   K tile   [D/32 pairs of slices u][64 keys][64 B]   64 B = channels 32u..32u+31 of one key, as four 16-byte chunks c, stored at
//            c ^ ((key >> 2) & 3): slices 2u and 2u + 1 lie 32 bytes apart, which of them first alternates, so the odd slices
//            take a base address of their own
//   V^T tile [4 key groups g][D channels][32 B]   32 B = the 16 keys of group g of one channel,
//            as two halves h holding keys 16g + {4h..4h+3, 8+4h..8+4h+3} (the contraction slots
//            of lane half h), stored at half h ^ ((channel >> 3) & 1)
// A 128-bit read of 16 consecutive keys (channels) then touches every bank exactly once.
//   V tile   as a K tile.  A transposing 64-bit read of a V operand takes, per lane half, 64 bytes of four neighbouring keys: every
//            bank once.  An operand is two of them, eight keys apart, whose chunks are stored at ^ 2 of each other: two base addresses
// The prompt's tiles hold its keys in position order, the compact tiles of a packed map the keys their slots
// name; slots without a key are zero-filled.
// Query rows lie in LDS as in memory but for their 16-byte chunks: chunk c of row r is at c ^ chunk_swap(r), rows that share their
// banks get different ones.
template <int D>
__device__ inline int chunk_swap(int r) { return D == 128 ? r & 15 : (r >> 1) & 7; }

__device__ inline int slot_key(const int32_t *__restrict__ compact_keys, int n, int key, int L, int N0)   // -1: no key
{
    const int s = n * kBlockN + key;
    return n < N0 ? (s < L ? s : -1) : compact_keys[s - N0 * kBlockN];
}

template <int D>
__device__ inline void pack_vt_tile(const __bf16 *__restrict__ v, __bf16 *__restrict__ vt,
                                    const int32_t *__restrict__ compact_keys, int L, int n, int N, int N0, __bf16 *tile)
{
    constexpr int PAD = D + 2;  // odd word stride: the column gathers below spread over banks
    const int kvh = blockIdx.y, tid = threadIdx.x;
    const __bf16 *src = v + (size_t)kvh * L * D;
    for (int idx = tid; idx < kBlockN * (D / 8); idx += 256) {
        const int key = idx / (D / 8), ch = idx % (D / 8);
        const int pos = slot_key(compact_keys, n, key, L, N0);
        bf16x8 val;
#pragma unroll
        for (int e = 0; e < 8; ++e) val[e] = (__bf16)0.f;
        if (pos >= 0) val = *reinterpret_cast<const bf16x8 *>(src + (size_t)pos * D + ch * 8);
#pragma unroll
        for (int e = 0; e < 8; ++e) tile[key * PAD + ch * 8 + e] = val[e];
    }
    __syncthreads();
    __bf16 *dst = vt + ((size_t)kvh * N + n) * (size_t)(D * kBlockN);
    for (int idx = tid; idx < D * 8; idx += 256) {   // one 16-byte half per iteration
        const int hp = idx & 1, d = (idx >> 1) % D, g = idx / (2 * D);
        const int h = hp ^ ((d >> 3) & 1);
        bf16x8 val;
#pragma unroll
        for (int e = 0; e < 8; ++e) val[e] = tile[(16 * g + 8 * (e >> 2) + 4 * h + (e & 3)) * PAD + d];
        *reinterpret_cast<bf16x8 *>(dst + (size_t)idx * 8) = val;
    }
}

// The prompt's complete K tiles are not packed: the attention kernel reads them where the caller has them.  The others -- the
// ragged last tile and the compact tiles, from tile `in_place` = L / 64 on -- hold their rows one behind the other as well.  So do the
// V tiles of a launch that reads V where the caller has it.
template <int D>
__device__ inline void pack_rows(const __bf16 *__restrict__ rows, __bf16 *__restrict__ packed,
                                 const int32_t *__restrict__ compact_keys, int L, int n, int N, int N0, int in_place)
{
    const int kvh = blockIdx.y;
    const __bf16 *src = rows + (size_t)kvh * L * D;
    __bf16 *dst = packed + ((size_t)kvh * (N - in_place) + n - in_place) * (size_t)(D * kBlockN);
    for (int idx = threadIdx.x; idx < kBlockN * (D / 8); idx += 256) {   // 16 bytes per iteration
        const int key = idx / (D / 8), ch = idx % (D / 8);
        const int pos = slot_key(compact_keys, n, key, L, N0);
        uint4 val = make_uint4(0, 0, 0, 0);
        if (pos >= 0) val = *reinterpret_cast<const uint4 *>(src + (size_t)pos * D + ch * 8);
        *reinterpret_cast<uint4 *>(dst + (size_t)idx * 8) = val;
    }
}

// The pre-pass of a bf16 call, one launch: grid (V^T tiles or the V tiles that lie nowhere else, then such K tiles, then workgroups that
// bring the work units from a pinned buffer; KV heads), of the
// tiles that the units of the launch walk.  Bound: HBM, so what counts is what is not packed: a chunk of 300 rows in a window
// of 1024 needs 21 of a 27K prompt's 429 tiles (three layers: 153 us, 253 with all of them), an all-Dense layer no compact
// ones (2048 rows behind 141K keys 9089 -> 8824 us, with the text tiles of Intra-Image).
struct PackTiles {
    int32_t first[6], count[6];   // runs of V tiles (prompt, free keys, text keys), then of K tiles
    int32_t n_tiles;              // all of them
    int32_t transpose;            // V tiles: all of the prompt's, as V^T; else like the K tiles
};
template <int D>
__global__ __launch_bounds__(256) void pack_kv_tiles(const __bf16 *__restrict__ k, const __bf16 *__restrict__ v,
                                                     __bf16 *__restrict__ kp, __bf16 *__restrict__ vp,
                                                     const int32_t *__restrict__ compact_keys, int L, int N, int N0, int in_place,
                                                     PackTiles todo, int32_t *__restrict__ queue_ctr,
                                                     const uint4 *__restrict__ copy_src, uint4 *__restrict__ copy_dst, size_t n_copy)
{
    __shared__ __bf16 tile[kBlockN * (D + 2)];
    if ((int)blockIdx.x >= todo.n_tiles && n_copy > 0) {   // (with it come the unit queues, at their beginning)
        const size_t stride = (size_t)(gridDim.x - todo.n_tiles) * gridDim.y * 256;
        for (size_t i = ((size_t)(blockIdx.x - todo.n_tiles) * gridDim.y + blockIdx.y) * 256 + threadIdx.x; i < n_copy; i += stride) copy_dst[i] = copy_src[i];
        return;
    }
    // the attention kernel that follows starts on fresh unit queues
    if (n_copy == 0 && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < 8) queue_ctr[threadIdx.x] = 0;
    if ((int)blockIdx.x >= todo.n_tiles) return;
    int x = blockIdx.x, run = 0;
#pragma unroll
    for (int i = 0; i < 5; ++i)
        if (run == i && x >= todo.count[i]) { x -= todo.count[i]; run = i + 1; }
    int n = todo.first[0];
#pragma unroll
    for (int i = 1; i < 6; ++i) n = run == i ? todo.first[i] : n;
    n += x;
    if (run < 3 && todo.transpose) pack_vt_tile<D>(v, vp, compact_keys, L, n, N, N0, tile);
    else pack_rows<D>(run < 3 ? v : k, run < 3 ? vp : kp, compact_keys, L, n, N, N0, in_place);
}

constexpr int kPingPongThreads = 512;

// Batch tags of the matrix phase: four operand reads + four MFMAs each.
template <int G> struct PvBatch { static constexpr int kind = 1, idx = G; static constexpr bool first = false; };            // O^T += V^T(group G) P^T(group G)
template <int B, bool FIRST> struct ScBatch { static constexpr int kind = 2, idx = B; static constexpr bool first = FIRST; }; // S += K(slices 2B, 2B+1) Q^T
struct NoBatch { static constexpr int kind = 0, idx = 0; static constexpr bool first = false; };

constexpr int kRing = 4;   // K slots = V^T slots of the LDS ring
constexpr int kMailboxBytes = 128;                  // the record of a workgroup's next unit, then the unit's number
constexpr int kPatchRow = 128 + 16;                 // a row of an output patch: 64 channels, where the row goes, the next unit's query row
constexpr int kPatchBytes = 32 * kPatchRow;         // of one wave
// LDS: ring, mailbox, output patches.  The patches lie beside the ring slots of a unit's first tiles and query rows, which are
// on their way while the patches are in use; seven of them fill the CU's LDS beside 16 KB slots, the eighth is in V^T slot 3, which is
// written in the second step.
template <int D, int KT>
constexpr int bf16_slot_bytes() { return KT * kBlockN * D * 2; }   // of the ring: the K or V^T tiles of a step
template <int D, int KT>
constexpr int bf16_lds_bytes() { return 2 * kRing * bf16_slot_bytes<D, KT>() + kMailboxBytes + 7 * kPatchBytes; }
static_assert(bf16_lds_bytes<128, 1>() <= 160 * 1024 && bf16_lds_bytes<64, 1>() <= 160 * 1024 && bf16_lds_bytes<64, 2>() <= 160 * 1024, "the CU's LDS");

// One workgroup = two groups of four waves = one work unit: two (head, query tile) items that
// read the same KV head and walk one merged key-tile list (heads of a GQA group with the same
// class, or two neighbouring query tiles of one head), so each K / V^T tile is fetched ONCE for
// 256 query rows.  The tiles live in a shared ring of 4 K + 4 V^T slots.  Per key tile a group
// runs two phases:
//   X (matrix):  O += P(k-1) V(k-1)  and  S(k) = K(k) Q^T        -- MFMA + LDS reads only
//   Y (vector):  mask, online softmax of S(k) -> P(k), rescale O  -- VALU only
// and the workgroup meets at ONE barrier per tile, placed so that the two groups run the phases
// in opposite order between two barriers (X then Y / Y then X): on every SIMD one wave is in X
// while the other is in Y, and the matrix pipe and the vector ALU stay busy together instead
// of the two waves queueing for the same unit.
// A step takes KT key tiles: one, and at d = 64 two where the lists are long (see steps_of_two).
// VT: V^T tiles, packed by the pre-pass; else V tiles lie as K tiles do, the complete ones of the prompt where the caller has them, and
// the operand reads transpose.
template <int D, int KT, bool VT>
__device__ __forceinline__ void walk_units(
    KernelArgs a, const uint64_t *__restrict__ map_text_bits, const uint64_t *__restrict__ map_sink_bits,
    const int4 *__restrict__ map_rows, const UnitRecord *__restrict__ units,
    const int2 *__restrict__ pair_ranges, const __bf16 *__restrict__ kp, const __bf16 *__restrict__ vp,
    int32_t n_k_tiles, int32_t *__restrict__ queue_ctr, const int32_t *__restrict__ queue_off,
    const int32_t *__restrict__ share_off, const StackedRows *__restrict__ stacked, float *__restrict__ cut_results)
{
    constexpr int ROW = D * 2;            // bytes per K row in LDS
    constexpr int TILE = kBlockN * ROW;   // bytes per K or V^T tile
    constexpr int kSlotBytes = bf16_slot_bytes<D, KT>();   // of the ring: the tiles of a step
    constexpr int DMA_PER_WAVE = kSlotBytes / 8192;        // LDS-direct loads per wave per matrix per step (8 waves)
    constexpr int NDB = D / 32;           // 32-channel blocks of the output
    constexpr int NPV = KT == 2 ? 4 : NDB;   // operands of a PV batch
    constexpr int RPV = VT ? 1 : 2;          // reads of such an operand
    constexpr int NT = D / 16;            // 16-wide slices of the head dim
    extern __shared__ __align__(1024) unsigned char lds[];   // K slots 0..3, then V (V^T) slots 0..3

    const int tid = threadIdx.x, lane = tid & 63, hl = lane >> 5, col = lane & 31;
    const int grp = __builtin_amdgcn_readfirstlane(tid >> 8);          // wave group 0 / 1
    const int wave8 = __builtin_amdgcn_readfirstlane(tid >> 6);        // wave within the workgroup
    const int L = a.L;

    const int R = L - a.q_begin;   // query rows per head
    const int in_place = L / kBlockN;   // complete K tiles of the prompt, read where the caller has them

    // ---- state of the work unit in progress (a workgroup takes units from its XCD's queue until
    // ---- the queues are empty; see the unit loop below)
    int head = 0, T = 0, item_class = 0;
    int slot_id = 0;                // > 0: a part of a cut unit, its results go to slot slot_id - 1
    bool have_item = false;
    const char *kph = nullptr, *vph = nullptr;            // K and V of the unit's KV head (VT: its V^T tiles)
    const char *kpackh = nullptr, *vpackh = nullptr;      // its other tiles (packed), by the same numbers
    bf16x8 qreg[NT];                // Q^T operand: Q[row][16t + 8hl .. +8] for every 16-wide slice t
    QueryView qv;

    // LDS byte address of this lane's MFMA operand fragments inside a K / V^T tile (see the
    // tile layouts above): key or channel `col`, half hl; slices, blocks and groups are
    // immediate offsets, the ring slot is added per step.
    const uint32_t ring = (uint32_t)(uintptr_t)(lds_void_ptr)lds;
    // (a transposing read: 16 lanes name the 8-byte pieces of 32 bytes of four keys, a lane gets its channel; the operand's upper
    // four keys lie eight rows further, at ^ 32)
    const uint32_t vaddr0 = VT ? ring + col * 32 + ((hl ^ ((col >> 3) & 1)) << 4)
                               : ring + (4 * hl + ((lane & 15) >> 2)) * 64 + (((2 * ((lane >> 4) & 1) + ((lane >> 1) & 1)) ^ hl) << 4) + (lane & 1) * 8;
    const uint32_t kaddr0 = ring + col * 64 + ((hl ^ ((col >> 2) & 3)) << 4);   // odd slices: ^ 32

    floatx16 o[NDB];
    floatx16 s[2 * KT];
    bf16x8 pf[2 * KT][2];   // P^T of the previous step as MFMA B operands
    float m_run = -INFINITY, l_run = 0.f;
    int out_row = -1;               // where this lane's row goes in `out`; -1: nowhere
    // The tiles of the vector phase and of the steps behind it, with their states: step k of a unit refills K with the tiles from
    // the one on that the walker stands on, those of step k + 3, and V^T with the ones before.
    TileWalker<KT> walk;
    int tile_y[KT] = {}, tile_1[KT] = {}, tile_2[KT] = {}, tile_3[KT] = {};
    // Both groups fetch, in the barrier interval k, their shares of K(k+3) and V^T(k+2): the second group
    // at the end of its matrix phase k, the first group right behind barrier k, before its vector phase.
    constexpr int ahead = 1;
    auto reset_unit_state = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[db][v] = 0.f;
#pragma unroll
        for (int kb = 0; kb < 2 * KT; ++kb)
#pragma unroll
            for (int v = 0; v < 16; ++v) s[kb][v] = 0.f;
#pragma unroll
        for (int i = 0; i < 4 * KT; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) pf[i >> 1][i & 1][e] = (__bf16)0.f;
        m_run = -INFINITY;
        l_run = 0.f;
    };

    // LDS-direct loads of packed tiles into ring slots: straight TILE-byte copies.  Each wave
    // instruction moves 1 KB (lane l -> bytes 16l..16l+15); instruction r of wave w (0..7) covers
    // bytes (8r + w) KB .. +1 KB of the tile, so the eight waves together fetch a tile.  The instruction
    // takes its address as a scalar base (the tile, uniform) plus a vector offset that never changes, and
    // its LDS destination in M0: nothing of it goes through the vector ALU, which the other wave of the
    // SIMD keeps busy (asm: the compiler forms a 64-bit vector address with a vector add per load instead).
    const uint32_t dma_lane_off = wave8 * 1024 + lane * 16;
    auto dma = [&](int r, const char *const (&tiles)[KT], int slot_byte) __attribute__((always_inline)) {
        const uint32_t dst = ring + slot_byte + wave8 * 1024 + r * 8 * 1024;   // lane 0's 16 bytes
        const char *src = KT == 1 ? tiles[0] + r * 8 * 1024 : tiles[r % KT];
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                     :
                     : "v"(dma_lane_off), "s"(src), "s"(dst)
                     : "memory", "m0");
    };
    // (a walker always names a tile that is there, behind its list the last one)
    auto v_ptr = [&](int n) { return (VT || n < in_place ? vph : vpackh) + (size_t)n * TILE; };
    auto k_ptr = [&](int n) { return (n < in_place ? kph : kpackh) + (size_t)n * TILE; };
    // The same for a K tile, whose rows lie one behind the other: 64 bytes of 16 rows per instruction, as many lookups in the vector
    // cache as for a copy (the other waves read the rest of the lines at the same time).  A lane picks the 16 bytes that belong
    // at its place.  So the caller's K is as good as a packed copy at any length; with 32 bytes of 32 rows it was 1-1.6 % slower
    // where a tile is fetched hundreds of times, and calls of that kind packed K.  (Whole rows per instruction, with chunks
    // exchanged by key: eight base addresses for the operand reads instead of two, 36K tokens 1.5 % slower.)
    const uint32_t kdma_key = (wave8 & 3) * 16 + (lane >> 2);
    const uint32_t kdma_lane_off = kdma_key * ROW + (wave8 >> 2) * 64 + (((lane & 3) ^ ((kdma_key >> 2) & 3)) << 4);
    auto kdma = [&](int r, const char *const (&tiles)[KT], int slot_byte) __attribute__((always_inline)) {
        const uint32_t dst = ring + slot_byte + wave8 * 1024 + r * 8 * 1024;
        const char *src = KT == 1 ? tiles[0] + r * 128 : tiles[r % KT];
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                     :
                     : "v"(kdma_lane_off), "s"(src), "s"(dst)
                     : "memory", "m0");
    };
    auto vdma = [&](int r, const char *const (&tiles)[KT], int slot_byte) __attribute__((always_inline)) {
        if constexpr (VT) dma(r, tiles, slot_byte);
        else kdma(r, tiles, slot_byte);
    };

    // ---- phase X building blocks (step k reads K slot k mod 4 and V^T slot (k - 1) mod 4) ----
    // A batch is four 128-bit operand reads feeding four MFMAs:
    //   PV batch g: O^T block db += V^T(db, group g) . P^T(group g); two tiles a step: key groups 2g and 2g + 1, db = 0, 1
    //   S  batch b: head-dim slices 2b, 2b+1 for both 32-key blocks; two tiles a step: slice b for the four of them
    uint32_t kbase = 0, kbase_odd = 0, vbase = 0, vbase_upper = 0;  // fragment base addresses inside the ring slots of this step
    // one operand read / one MFMA of a batch (element i = 0..3)
    auto read_one = [&](auto tag, auto ic, bf16x8 &dst) __attribute__((always_inline)) {
        using T = decltype(tag);
        constexpr int i = decltype(ic)::value;
        if constexpr (T::kind == 1) {
            // channel block i (two tiles: i & 1 of group 2 idx + (i >> 1))
            if constexpr (i < NPV && VT) {
                lds_read_b128<T::idx * NPV * 1024 + i * 1024>(dst, vbase);
            } else if constexpr (i < NPV) {
                constexpr int group = KT == 1 ? T::idx : 2 * T::idx + (i >> 1);
                constexpr int at = (group >> 2) * TILE + (i % NDB) * 4096 + (group & 3) * 1024;
                bf16x4 lower, upper;
                lds_read_tr_b64<at>(lower, vbase);
                lds_read_tr_b64<at + 512>(upper, vbase_upper);
                dst = __builtin_shufflevector(lower, upper, 0, 1, 2, 3, 4, 5, 6, 7);
            }
        } else if constexpr (T::kind == 2) {
            if constexpr (KT == 1) lds_read_b128<T::idx * 4096 + (i & 1) * 2048>(dst, (i >> 1) ? kbase_odd : kbase);   // slice 2 idx + (i >> 1), key block
            else lds_read_b128<(T::idx >> 1) * 4096 + (i >> 1) * TILE + (i & 1) * 2048>(dst, (T::idx & 1) ? kbase_odd : kbase);   // slice idx, key block i
        }
    };
    auto mul_one = [&](auto tag, auto ic, const bf16x8 &f) __attribute__((always_inline)) {
        using T = decltype(tag);
        constexpr int i = decltype(ic)::value;
        if constexpr (T::kind == 1) {
            constexpr int group = KT == 1 ? T::idx : 2 * T::idx + (i >> 1);
            if constexpr (i < NPV) mfma_acc(o[i % NDB], f, pf[group >> 1][group & 1]);
        } else if constexpr (T::kind == 2) {
            constexpr int block = KT == 1 ? i & 1 : i, slice = KT == 1 ? 2 * T::idx + (i >> 1) : T::idx;
            if constexpr (T::first && (KT == 2 || i < 2)) mfma_set(s[block], f, qreg[slice]);
            else mfma_acc(s[block], f, qreg[slice]);
        }
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I3 = std::integral_constant<int, 3>;

    // Phase X of step k: O += P(k-1) V(k-1) and S(k) = K(k) Q^T.  Always the same straight-line
    // chain of asm statements: before the first tile -- and behind tiles this item skips -- P is zero,
    // and the scores of a tile it skips are ignored.  Operand reads run up to three batches ahead of the MFMAs that
    // consume them (at the head of the chain two, three where batches are halves), in three rotating register sets; each
    // lds_wait<N> count is the number of reads issued after the batch waited for (a transposing operand takes two).
    // A register is refilled right after the MFMA that read it has issued (operands are read at issue, LDS data
    // returns later), so the reads issue in the shadow of the MFMAs.
    // text / sink key bits of the tile of the coming phase Y (scalar registers)
    uint64_t tb_cur[KT] = {}, sb_cur[KT] = {};
    const char *ksrc[KT] = {}, *vsrc[KT] = {};   // tiles of the coming refill ...
    // The scalar work of a step -- tiles of the refill, the walk, key bit masks for the coming phase Y -- stands inside
    // phase X, between two MFMA batches, where the wave has issue slots to spare (every MFMA keeps the matrix pipe busy for
    // 32 cycles).  Anything in front of the first MFMA costs its full length: with the walk there the same kernel takes 2 % longer
    // (36K tokens 15573 us, 15220 with it here), with three walkers instead of the one and a look-ahead 3 % on windows.
    // The masks are asked for only where the item needs them (a sparse class without compact tiles, Intra-Image with mixed ones): a
    // scalar load in flight is counted together with the operand reads, which are then waited for early.  This kernel asking for
    // them at every step and as it is, one box: 302K tokens 185.1 / 182.8 ms, 36K 15599 / 15471 us, window of 1024 on 27K 1529 / 1517.
    bool need_bits = false;
    auto advance_walk = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < KT; ++t) {
            if constexpr (KT == 1) {
                ksrc[t] = k_ptr(walk.cur >> 4);
                vsrc[t] = v_ptr(tile_3[t] >> 4);
            }
            tile_y[t] = tile_1[t];
            tile_1[t] = tile_2[t];
            tile_2[t] = tile_3[t];
            tile_3[t] = walk.cur;
            walk.next();
        }
        if (need_bits) {
#pragma unroll
            for (int t = 0; t < KT; ++t) {
                tb_cur[t] = scalar_load<uint64_t>(map_text_bits + (tile_y[t] >> 4));
                sb_cur[t] = scalar_load<uint64_t>(map_sink_bits + (tile_y[t] >> 4));
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    int Sk_dst = 0, Sv_dst = 0;                    // ... and their ring slots
    auto issue_refill = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
        // (two tiles a step: eight scalar registers from the walk to here were eight too many, and the step loop of the first group moved
        // others to vector lanes and back; 9K tokens 843 -> 833 us, window of 4096 on 40K 1752 -> 1722)
        if constexpr (KT > 1) {
#pragma unroll
            for (int t = 0; t < KT; ++t) {
                ksrc[t] = k_ptr(tile_3[t] >> 4);
                vsrc[t] = v_ptr(tile_2[t] >> 4);
            }
        }
#pragma unroll
        for (int r = 0; r < DMA_PER_WAVE; ++r) kdma(r, ksrc, Sk_dst * kSlotBytes);
#pragma unroll
        for (int r = 0; r < DMA_PER_WAVE; ++r) vdma(r, vsrc, (kRing + Sv_dst) * kSlotBytes);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto phase_x = [&](int S, int Sv, auto refill_here) __attribute__((always_inline)) {  // S = k mod 4, Sv: slot of V^T(k-1)
        auto ring = [](int x) { return x >= kRing ? x - kRing : x; };
        Sk_dst = ring(ring(S + 2) + ahead); Sv_dst = ring(S + 1 + ahead);
        kbase = kaddr0 + S * kSlotBytes;
        kbase_odd = kbase ^ 32;
        vbase = vaddr0 + (kRing + Sv) * kSlotBytes;
        vbase_upper = vbase ^ 32;
        bf16x8 fa[4], fb[4], fc[4];
        if constexpr (NPV < 4) {
#pragma unroll
            for (int i = NPV; i < 4; ++i)
#pragma unroll
                for (int e = 0; e < 8; ++e) { fa[i][e] = (__bf16)0.f; fb[i][e] = (__bf16)0.f; fc[i][e] = (__bf16)0.f; }
        }
        // whole-batch reads of the pipeline head
        auto read_batch = [&](auto tag, bf16x8 (&f)[4]) __attribute__((always_inline)) {
            read_one(tag, I0{}, f[0]); read_one(tag, I1{}, f[1]);
            read_one(tag, I2{}, f[2]); read_one(tag, I3{}, f[3]);
        };
        // MFMA batch `cur` on fragment set f, each MFMA followed by the read that refills its
        // operand register for batch `nxt` (three batches ahead)
        auto batch = [&](auto cur, auto nxt, bf16x8 (&f)[4]) __attribute__((always_inline)) {
            mul_one(cur, I0{}, f[0]); read_one(nxt, I0{}, f[0]);
            mul_one(cur, I1{}, f[1]); read_one(nxt, I1{}, f[1]);
            mul_one(cur, I2{}, f[2]); read_one(nxt, I2{}, f[2]);
            mul_one(cur, I3{}, f[3]); read_one(nxt, I3{}, f[3]);
        };
        // The same with two reads behind each MFMA: the refill of its own register (batch `nxt`) and
        // one read of batch `mid` into the idle set g.
        auto batch2 = [&](auto cur, auto mid, bf16x8 (&g)[4], auto nxt, bf16x8 (&f)[4]) __attribute__((always_inline)) {
            mul_one(cur, I0{}, f[0]); read_one(mid, I0{}, g[0]); read_one(nxt, I0{}, f[0]);
            mul_one(cur, I1{}, f[1]); read_one(mid, I1{}, g[1]); read_one(nxt, I1{}, f[1]);
            mul_one(cur, I2{}, f[2]); read_one(mid, I2{}, g[2]); read_one(nxt, I2{}, f[2]);
            mul_one(cur, I3{}, f[3]); read_one(mid, I3{}, g[3]); read_one(nxt, I3{}, f[3]);
        };
        if constexpr (NPV == 4) {
            // batch order: S0 PV0 S1 PV1 S2 PV2 S3 PV3, four MFMAs each, with four reads (eight for a PV batch that transposes).  The
            // scores are there four MFMAs before the end of
            // the chain, so the vector phase starts under the last ones: with the scores last, and a wait for them, 36K tokens 16327 us,
            // 16179 so, 2048 rows behind 141K keys 8489 -> 8406, 16K tokens characterised 3214 -> 3183.
            // Only two batches are read ahead of the first MFMA (the burst of all four waves of a group
            // costs every wave its share of the LDS time); the third goes out behind the first four
            // MFMAs together with their refills.
            read_batch(ScBatch<0, true>{}, fa); read_batch(PvBatch<0>{}, fb);
            lds_wait<4 * RPV>(fa); batch2(ScBatch<0, true>{}, ScBatch<1, false>{}, fc, PvBatch<1>{}, fa);
            lds_wait<4 + 4 * RPV>(fb); batch(PvBatch<0>{}, ScBatch<2, false>{}, fb);
            lds_wait<4 + RPV>(fc); batch(ScBatch<1, false>{}, PvBatch<2>{}, fc);   // behind the last S1 read: the last of PV1, four S2
            lds_wait<4 + 4 * RPV>(fa); batch(PvBatch<1>{}, ScBatch<3, false>{}, fa);
            advance_walk();
            lds_wait<4 + 4 * RPV>(fb); batch(ScBatch<2, false>{}, PvBatch<3>{}, fb);
            lds_wait<4 + 4 * RPV>(fc); batch(PvBatch<2>{}, NoBatch{}, fc);
            lds_wait<4 * RPV>(fa); batch(ScBatch<3, false>{}, NoBatch{}, fa);
            lds_wait<0>(fb); batch(PvBatch<3>{}, NoBatch{}, fb);
            // No wait for the accumulators: the last scores were finished by the MFMAs behind them, and the output tile is next
            // touched at the end of the vector phase.  (The statement keeps the vector phase behind the chain.)
            asm volatile("" : "+v"(s[0]), "+v"(s[1]));
            if constexpr (KT == 2) asm volatile("" : "+v"(s[2]), "+v"(s[3]));
        } else {
            // PV batches are half as large, S has two batches of four.  The chain is half as long, and scores first gain nothing (window of
            // 512 on 30K tokens 540 us, 536 with values first, 1.4K tokens 49.4 and 48.4)
            read_batch(PvBatch<0>{}, fa); read_batch(ScBatch<0, true>{}, fb); read_batch(PvBatch<1>{}, fc);
            lds_wait<4 + 2 * RPV>(fa); batch(PvBatch<0>{}, PvBatch<2>{}, fa);
            lds_wait<4 * RPV>(fb); batch(ScBatch<0, true>{}, ScBatch<1, false>{}, fb);
            lds_wait<4 + 2 * RPV>(fc); batch(PvBatch<1>{}, PvBatch<3>{}, fc);
            advance_walk();
            lds_wait<4 + 2 * RPV>(fa); batch(PvBatch<2>{}, NoBatch{}, fa);
            lds_wait<2 * RPV>(fb); batch(ScBatch<1, false>{}, NoBatch{}, fb);
            lds_wait<0>(fc); batch(PvBatch<3>{}, NoBatch{}, fc);
            mfma_drain(o[0], o[1]);   // the scores finished two MFMAs earlier
        }
        // Every LDS read and scalar load of the phase has returned (the last lds_wait was for zero): say so
        // in a form the compiler sees, or it waits for its own scalar loads in the middle of the next chain.
        __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
        // Refill: this wave's share of K(k+3) and V^T(k+2) into the slots of the tiles four steps older,
        // which nobody reads after barrier k.  Unconditional: past the end of the list a valid tile is
        // fetched again and never used.  An LDS-direct load issued while the other wave of the SIMD issues
        // matrix or vector instructions stalls this wave several times longer, so each group issues it in a
        // window in which its mate is quiet: the second group here, after its last MFMA, while the first
        // group waits for the head reads of its next matrix phase; the first group right behind the barrier
        // (see the step loop), while the second group waits for its head reads.
        if constexpr (decltype(refill_here)::value) issue_refill();
        // Wait for the loads issued one step ago (only this step's may stay in flight): after
        // the next barrier every wave has passed this wait, and the tile is read in the interval
        // that follows it.
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * DMA_PER_WAVE));
    };

    // The last step: O += P(T-1) V(T-1), nothing else.
    auto phase_last = [&](int Sv) __attribute__((always_inline)) {
        vbase = vaddr0 + (kRing + Sv) * kSlotBytes;
        vbase_upper = vbase ^ 32;
        bf16x8 fa[4], fb[4], fc[4];
        if constexpr (NPV < 4) {
#pragma unroll
            for (int i = NPV; i < 4; ++i)
#pragma unroll
                for (int e = 0; e < 8; ++e) { fa[i][e] = (__bf16)0.f; fb[i][e] = (__bf16)0.f; fc[i][e] = (__bf16)0.f; }
        }
        auto read_batch = [&](auto tag, bf16x8 (&f)[4]) __attribute__((always_inline)) {
            read_one(tag, I0{}, f[0]); read_one(tag, I1{}, f[1]);
            read_one(tag, I2{}, f[2]); read_one(tag, I3{}, f[3]);
        };
        auto mul_batch = [&](auto tag, bf16x8 (&f)[4]) __attribute__((always_inline)) {
            mul_one(tag, I0{}, f[0]); mul_one(tag, I1{}, f[1]);
            mul_one(tag, I2{}, f[2]); mul_one(tag, I3{}, f[3]);
        };
        constexpr int kReads = NPV * RPV;   // of a batch
        read_batch(PvBatch<0>{}, fa); read_batch(PvBatch<1>{}, fb);
        lds_wait<kReads>(fa); mul_batch(PvBatch<0>{}, fa); read_batch(PvBatch<2>{}, fc);
        lds_wait<kReads>(fb); mul_batch(PvBatch<1>{}, fb); read_batch(PvBatch<3>{}, fa);
        lds_wait<kReads>(fc); mul_batch(PvBatch<2>{}, fc);
        lds_wait<0>(fa); mul_batch(PvBatch<3>{}, fa);
        mfma_drain(o[0], o[1]);
        if constexpr (NDB > 2) asm volatile("" : "+v"(o[2]), "+v"(o[3]));
    };

    // Phase Y of a step: mask (PARTIAL tiles), online softmax, rescale O, round P to bf16.
    auto phase_y = [&]() __attribute__((always_inline)) {
        // state of the tile for this group's item: 0 skip (only the other item wants the
        // tile), 1 partial, 2 full.  A skipped tile goes through the row-uniform path with
        // every row dropped (P = 0, running max and sum unchanged): rare, and one straight
        // code path keeps the register allocation of the loop simple.
        // (what stays the same for a unit is hidden from the compiler here: it made loops of their own for its values)
        int hd = head, cls = item_class;
        asm("" : "+s"(hd), "+s"(cls));
        bool drop[KT];
#pragma unroll
        for (int t = 0; t < KT; ++t) {
            const int st = hd >= 0 ? (grp ? tile_y[t] : tile_y[t] >> 2) & 3 : 0;
            drop[t] = false;
            if (st != 2) {
                const int nu = tile_y[t] >> 4;
                const uint64_t allowed = st == 0 ? 0ull : allowed_keys(qv, cls, tb_cur[t], sb_cur[t], nu, a);
                drop[t] = allowed == 0ull;
                // where every query of the wave sees all 64 keys or none (e.g. a text row and an
                // image row over keys of another image) there is no per-score work.  (Behind a list of an odd length its last tile
                // comes again: scores that were masked the first time, whatever they are, may not reach anything now.)
                const bool again = t > 0 && nu == tile_y[0] >> 4;
                if (again || !__all(drop[t] || allowed == ~0ull)) apply_mask(s[2 * t], s[2 * t + 1], allowed, hl);
            }
        }
        float alpha;
        softmax_pack<KT>(s, pf, m_run, l_run, alpha, a.scale_log2e, drop);
        asm volatile("" : "+v"(alpha));   // one place where the output tile may change, reached by every path: two cost 64 register copies
        if (__any(alpha != 1.f)) {
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[db][v] *= alpha;
        }
    };

    // ---- Work distribution.  The host deals the units (heaviest first) to eight queues, one per XCD,
    // so that units walking the same K / V^T tiles at about the same time share an L2.  A workgroup
    // reads the id of the XCD it runs on from the hardware register (it does not depend on the launch
    // order, which other streams can perturb) and claims the next unit of that queue with an atomic
    // counter; when the queue is empty it helps out on the next one.  The first wave takes the ticket
    // for the next unit three steps before the current one ends -- late, so that the units of a queue
    // start in queue order (units that start together walk the same tiles together and share them in
    // L2; a ticket taken a whole unit ahead was measured to cost half of that sharing), early enough
    // for the atomic to return under the last steps -- and requests the unit's record into a mailbox behind
    // the ring in the last one.  Every wave reads the same mailbox entry, so the workgroup leaves the loop together.
    typedef volatile __attribute__((address_space(3))) int32_t *lds_int_ptr;
    const uint32_t mailbox_addr = ring + 2 * kRing * kSlotBytes;
    constexpr int kRecordInts = sizeof(UnitRecord) / 4;
    const lds_int_ptr mailbox = (lds_int_ptr)(uintptr_t)mailbox_addr;
    int xcc;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID, 0, 4)" : "=s"(xcc));
    xcc &= 7;
    // The unit of a ticket of the own queue; if that is empty, a claim on the next one that is not, or -1.  One look
    // at all counters says which queues to ask (a counter only grows: what is empty stays empty); asking seven
    // empty queues one after the other took 10 us at the end of every launch.
    const int own_begin = scalar_load<int>(queue_off + xcc), own_len = scalar_load<int>(queue_off + xcc + 1) - own_begin;
    auto claim_from = [&](int ticket) {
        if (ticket < own_len) return own_begin + ticket;
        const int q = lane & 7, begin = queue_off[q], len = queue_off[q + 1] - begin;
        const bool left = __hip_atomic_load(&queue_ctr[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < len;
        for (uint32_t open = (uint32_t)__ballot(left && q != xcc) & 0xff; open;) {
            const uint32_t turned = ((open >> xcc) | (open << (8 - xcc))) & 0xff;   // bit 0: the own queue
            const int next = (xcc + __builtin_ctz(turned)) & 7;
            const int next_begin = queue_off[next], next_len = queue_off[next + 1] - next_begin;
            int r = 0;
            if (lane == 0) r = atomicAdd(&queue_ctr[next], 1);
            r = __builtin_amdgcn_readfirstlane(r);
            if (r < next_len) return next_begin + r;
            open &= ~(1u << next);
        }
        return -1;
    };
    auto take_ticket = [&]() {   // one atomic on the own queue; lane 0's result counts
        int r = 0;
        if (lane == 0) r = atomicAdd(&queue_ctr[xcc], 1);
        return r;
    };
    // The same without waiting for the answer: lane 0 alone issues the atomic (asm, so that the compiler
    // does not wait for it on the spot) and the ticket is in lane 0 of the result once the vector-memory
    // counter has drained (ticket_wait).  Until then the register must not be read.
    auto take_ticket_async = [&]() __attribute__((always_inline)) {
        int r;
        unsigned long long save;
        int32_t *ctr = queue_ctr + xcc;
        const int one = 1;
        asm volatile("s_mov_b64 %[save], exec\n\t"
                     "s_mov_b64 exec, 1\n\t"
                     "global_atomic_add %[r], %[ptr], %[one], off sc0\n\t"
                     "s_mov_b64 exec, %[save]"
                     : [r] "=&v"(r), [save] "=&s"(save)
                     : [ptr] "v"(ctr), [one] "v"(one)
                     : "memory");
        return r;
    };
    auto ticket_wait = [&](int &ticket) __attribute__((always_inline)) {
        asm volatile("s_waitcnt vmcnt(0)" : "+v"(ticket)::"memory");
    };
    // Equal shares (few units; planned by the host): workgroup b first walks the parts of its share, then helps with
    // what the queues hold.  Workgroups go round-robin over the XCDs, so the shares of an XCD are neighbours and
    // meet in its L2.
    int share_next = 0, share_end = 0;
    if (share_off) {
        const int n = gridDim.x, per = n >> 3, b = blockIdx.x;
        const int share = (n & 7) == 0 ? (b & 7) * per + (b >> 3) : b;
        share_next = share_off[share];
        share_end = share_off[share + 1];
    }
    // The record of a unit goes to the mailbox by itself (64 bytes: four lanes of an LDS-direct load).
    auto fetch_record = [&](int u) __attribute__((always_inline)) {
        const char *src = reinterpret_cast<const char *>(units) + (size_t)u * sizeof(UnitRecord);
        const uint32_t off = lane * 16;
        unsigned long long save;
        asm volatile("s_mov_b64 %[save], exec\n\t"
                     "s_mov_b64 exec, 15\n\t"
                     "s_mov_b32 m0, %[dst]\n\t"
                     "s_nop 0\n\t"
                     "global_load_lds_dwordx4 %[off], %[src]\n\t"
                     "s_mov_b64 exec, %[save]"
                     : [save] "=&s"(save)
                     : [off] "v"(off), [src] "s"(src), [dst] "s"(mailbox_addr)
                     : "memory", "m0");
    };
    constexpr int kUnknown = -2;
    int next_unit = -1;                            // first wave: the unit that the mailbox is filled for
    if (wave8 == 0) {
        next_unit = share_next < share_end ? share_next : claim_from(__builtin_amdgcn_readfirstlane(take_ticket()));
        if (next_unit >= 0) fetch_record(next_unit);
        if (lane == 0) mailbox[kRecordInts] = next_unit;
    }
    ++share_next;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    // ---- the loop over units.  The end of one and the beginning of the next overlap: with the barrier behind the last step
    // everybody knows the next unit's record, its row records are requested before the first half of the epilogue and its
    // query rows and first tiles between the two halves, so that their latencies run side by side and under the stores.
    // The query rows come through LDS, whole rows per load (into the slots of K(2), K(3) and V^T(1), V^T(2), which are
    // requested when every wave has its rows): as operands straight from memory every lane would take 16 bytes of another
    // row, 64 lines per instruction, and the 64 instructions of a workgroup kept the vector cache busy for 4,000 cycles.
    // From the last step to the first one (time stamps): 13,500 -> 9,500 cycles on long prompts, 19,000 -> 13,000 on a windowed
    // one; passes 1590 -> 1554 us (27K tokens, window of 1024, 13 units a workgroup), 1029 -> 1008 (8K tokens, 4 units), d = 64 910 ->
    // 894 (9K).  Overlapping alone, with the operands straight from memory, gained nothing.
    constexpr int kRowsPerLoad = 1024 / ROW, kChunks = ROW / 16, kQueryLoads = 32 / kRowsPerLoad;
    bool first_unit = true;
    for (;;) {
        const int unit = __builtin_amdgcn_readfirstlane(mailbox[kRecordInts]);
        const bool more = unit >= 0;
        // (hidden from the compiler, or addresses that only this part needs would stay in registers through the step loops)
        int ln = lane, w8 = wave8;
        asm volatile("" : "+v"(ln), "+s"(w8));
        const int hl = ln >> 5, col = ln & 31;
        unsigned char *const stage = lds + (w8 == 7 ? (2 * kRing - 1) * kSlotBytes : 2 * kRing * kSlotBytes + kMailboxBytes + w8 * kPatchBytes);
        const int query_at = (w8 >= 4 ? kRing + 1 : 2) * kSlotBytes + (w8 & 3) * 32 * ROW;
        // of the previous unit, for its epilogue
        const int done_slot = slot_id;
        const bool done_item = have_item && !first_unit;
        int4 r0, r1;
        RowRef ref;
        int rec[kRecordInts];
#pragma unroll
        for (int i = 0; i < kRecordInts / 4; ++i) {
            const intx4 x = *(const __attribute__((address_space(3))) intx4 *)(uintptr_t)(mailbox_addr + 16 * i);
#pragma unroll
            for (int j = 0; j < 4; ++j) rec[4 * i + j] = __builtin_amdgcn_readfirstlane(x[j]);
        }
        if (more) {
            head = grp ? rec[2] : rec[0];
            have_item = head >= 0;
            T = (rec[4] + KT - 1) / KT;                           // steps: key tiles in the merged list, or pairs of them
            slot_id = rec[5] >> 16;
            item_class = (grp ? rec[5] >> 8 : rec[5]) & 7;        // head classes travel with the unit
            need_bits = (item_class & 3) != 0 && !((item_class & 4) && ((item_class & 1) || a.text_tile0 < a.n_tiles));
            const int kvh = rec[6];                               // both items share it
            // a tile slot without a row behaves like a row past the end of the prompt (computed on a
            // copy of the last row, never stored)
            ref = row_of(stacked, ((grp ? rec[5] >> 8 : rec[5]) & 8) != 0, a.G, max(head, 0), max(grp ? rec[3] : rec[1], 0), (w8 & 3) * 32 + col);
            r0 = map_rows[2 * ref.record];
            r1 = map_rows[2 * ref.record + 1];
            // one TILE-byte block per key tile
            kph = reinterpret_cast<const char *>(a.k) + (size_t)kvh * L * ROW;
            kpackh = reinterpret_cast<const char *>(kp) + ((int64_t)kvh * (n_k_tiles - in_place) - in_place) * (int64_t)TILE;
            if constexpr (VT) {
                vph = reinterpret_cast<const char *>(vp + (size_t)kvh * n_k_tiles * (size_t)(D * kBlockN));
            } else {
                vph = reinterpret_cast<const char *>(a.v) + (size_t)kvh * L * ROW;
                vpackh = reinterpret_cast<const char *>(vp) + ((int64_t)kvh * (n_k_tiles - in_place) - in_place) * (int64_t)TILE;
            }
        }

        // epilogue of the previous unit: divide by the running sum, round, store.  Empty rows (l = 0) give zeros.  A lane holds
        // four channels of one row at a time (O^T accumulators), which would make every store instruction
        // touch 64 rows with 8 bytes each; the tile goes through LDS instead, 64 channels at a time in a wave-private patch, and
        // leaves as 16-byte pieces of 128-byte row segments.
        const float l_tot = sum_across_halves(l_run);
        const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
        if (hl == 0) *reinterpret_cast<int32_t *>(stage + col * kPatchRow + 128) = out_row;
        auto store_half = [&](int half) __attribute__((always_inline)) {
#pragma unroll
            for (int dbl = 0; dbl < 2; ++dbl)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    bf16x4 w;
#pragma unroll
                    for (int r = 0; r < 4; ++r) w[r] = (__bf16)(o[2 * half + dbl][4 * g + r] * inv);
                    *reinterpret_cast<bf16x4 *>(stage + col * kPatchRow + (32 * dbl + 8 * g + 4 * hl) * 2) = w;
                }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = 8 * j + (ln >> 3), chunk = ln & 7;
                const uint4 piece = *reinterpret_cast<const uint4 *>(stage + r * kPatchRow + chunk * 16);
                const int32_t to = *reinterpret_cast<const int32_t *>(stage + r * kPatchRow + 128);
                if (to >= 0) *reinterpret_cast<uint4 *>(reinterpret_cast<__bf16 *>(a.out) + (size_t)to * D + 64 * half + chunk * 8) = piece;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        };
        if (done_item) {
            // a part of a cut unit: accumulators, reference point and row sum as they are
            if (done_slot > 0) store_cut_item<D>(cut_results + ((size_t)(done_slot - 1) * 2 + grp) * kCutItemFloats<D>, o, m_run, l_tot, w8 & 3, ln);
            else store_half(0);
        }
        if (more) {
            const int row = ref.there ? r0.x : L;
            out_row = row < L ? ref.head * R + (row - a.q_begin) : -1;
            // rows past the end compute on a copy and are not stored
            if (hl == 0) *reinterpret_cast<int32_t *>(stage + col * kPatchRow + 132) = ref.head * R + min(row, L - 1) - a.q_begin;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int j = 0; j < kQueryLoads; ++j) {
                const int r = j * kRowsPerLoad + ln / kChunks;
                // (a whole address per lane: the rows of a head alone may take more than 4 GiB)
                const char *src = static_cast<const char *>(a.q) + (size_t)*reinterpret_cast<const uint32_t *>(stage + r * kPatchRow + 132) * ROW +
                                  (((ln % kChunks) ^ chunk_swap<D>(r)) << 4);
                asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                             :
                             : "v"(src), "s"(ring + query_at + j * 1024)
                             : "memory", "m0");
            }
            // (the walkers name tiles that this launch's pre-pass wrote, also those of an empty list)
            const int none = a.first_tile << 4;
            const char *k0[KT], *k1[KT], *v0[KT];
#pragma unroll
            for (int t = 0; t < KT; ++t) {
                tile_1[t] = T > 0 ? rec[8 + t] : none;
                tile_2[t] = T > 0 ? rec[8 + KT + t] : none;
                k0[t] = k_ptr(tile_1[t] >> 4); k1[t] = k_ptr(tile_2[t] >> 4); v0[t] = v_ptr(tile_1[t] >> 4);
            }
            // K(0), K(1) and V^T(0) to the slots of these numbers (unconditional)
#pragma unroll
            for (int r = 0; r < DMA_PER_WAVE; ++r) kdma(r, k0, 0);
#pragma unroll
            for (int r = 0; r < DMA_PER_WAVE; ++r) kdma(r, k1, kSlotBytes);
#pragma unroll
            for (int r = 0; r < DMA_PER_WAVE; ++r) vdma(r, v0, kRing * kSlotBytes);
            // (the walker stands on the fourth tile; with two tiles a step it walks on while the loads are on their way)
            walk = {pair_ranges, T > 0 ? rec[11] : none, T > 0 ? rec[12] : none + 16, rec[13], rec[14], rec[15], rec[7]};
            if constexpr (KT == 1) {
                tile_3[0] = T > 0 ? rec[10] : none;
            } else {
                walk.next();
#pragma unroll
                for (int t = 0; t < KT; ++t) {
                    tile_3[t] = walk.cur;
                    walk.next();
                }
            }
#pragma unroll
            for (int t = 0; t < KT; ++t) {
                ksrc[t] = k_ptr(tile_3[t] >> 4);
                vsrc[t] = v_ptr(tile_2[t] >> 4);
            }
        }
        if constexpr (NDB == 4) {
            if (done_item && done_slot == 0) store_half(1);
        }
        if (!more) break;
        first_unit = false;
        reset_unit_state();
        qv.init(r0, r1, item_class & 3, (item_class & 4) != 0, a);
        int next_ticket = 0;
        if (wave8 == 0) next_unit = kUnknown;
        const int k_late = wave8 == 0 && T >= 3 ? T - 3 : INT32_MAX;   // the first wave's steps with something to do for the next unit
        // Raw barriers: every LDS access of the loop is an LDS-direct load (drained with vmcnt
        // at the end of phase X) or an asm read (drained with lgkmcnt inside phase X), so no fence
        // is wanted there -- a fence would drain loads that are meant to stay in flight.
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): query rows and first tiles
        asm volatile("" ::: "memory");
#pragma unroll
        for (int t = 0; t < NT; ++t)
            qreg[t] = *(const __attribute__((address_space(3))) bf16x8 *)(uintptr_t)((ring + query_at + col * ROW + ((hl ^ chunk_swap<D>(col)) << 4)) ^ (t << 5));
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the query rows, the unit's scalar loads (none stays pending into the loop)
#pragma unroll
        for (int t = 0; t < NT; ++t) asm volatile("" : "+v"(qreg[t]));
        __builtin_amdgcn_s_barrier();
        Sk_dst = 2; Sv_dst = 1;
        issue_refill();                      // K(2) and V^T(1), as a step before the first one would
        // ONE barrier per step.  Group 0 runs  X(k) | barrier | refill Y(k),  group 1  barrier | X(k) refill Y(k):
        // between two barriers group 0 does Y(k) then X(k+1) while group 1 does X(k) then Y(k), so
        // the waves of a SIMD are in opposite phases by program order but nothing holds them to a
        // half-step grid.  Between barrier k and k+1 the ring is read at K(k), K(k+1), V^T(k-1),
        // V^T(k) and written by both groups at K(k+3), V^T(k+2), whose slots (of K(k-1), V^T(k-2))
        // nobody reads after barrier k; at the end of every matrix phase a wave lets only its newest
        // loads stay in flight (vmcnt), so the loads of interval k have landed before barrier k + 2,
        // and the tiles are read from the interval after that barrier on: four slots each.
        // The last step only adds P(T-1) V(T-1) and stands behind the loop: half a matrix phase, no refill.
        // With the look at all queues at once (claim_from) a windowed prompt of 27K tokens, 13 units per
        // workgroup of 20 tiles each, takes 2058 instead of 2093 us a pass.
        int slot = 0, v_slot = 0;   // (before the first step P is zero, and any finite tile will do for V^T(-1): V^T(0))
        if (grp == 0) {
            // (no first iteration of its own: the compiler puts the zeroing of the accumulators and fragments right in front of
            // the MFMAs that read them, too close for the hardware, and does not know; tests/isa_check.py looks for that)
#pragma nounroll
            for (int k = 0; k < T; ++k) {
                if (k >= k_late) {
                    if (k == T - 3) {
                        if (share_next >= share_end) next_ticket = take_ticket_async();
                    } else if (k == T - 1) {
                        // (the ticket is there: the phases since have waited for all but the newest loads)
                        int ticket = next_ticket;
                        asm volatile("" : "+v"(ticket));
                        ticket = __builtin_amdgcn_readfirstlane(ticket);
                        if (share_next < share_end) next_unit = share_next;
                        else if (ticket < own_len) next_unit = own_begin + ticket;
                        if (next_unit >= 0) fetch_record(next_unit);
                    }
                }
                phase_x(slot, v_slot, std::false_type{});
                __builtin_amdgcn_s_barrier();
                issue_refill();   // under the second group's head reads, before its chain starts
                phase_y();
                v_slot = slot;
                slot = slot == kRing - 1 ? 0 : slot + 1;
            }
            if (T > 0) phase_last(v_slot);
        } else {
#pragma nounroll
            for (int k = 0; k < T; ++k) {
                __builtin_amdgcn_s_barrier();
                phase_x(slot, v_slot, std::true_type{});
                phase_y();
                v_slot = slot;
                slot = slot == kRing - 1 ? 0 : slot + 1;
            }
            if (T > 0) phase_last(v_slot);
        }
        // End of the unit: the refills of its last steps (tiles nobody needs) must have landed
        // before the next unit's first tiles go into the same slots, and every wave must be done
        // reading the ring.  The next unit's record has arrived by then as well.
        ticket_wait(next_ticket);            // vmcnt(0)
        if (wave8 == 0) {
            if (next_unit == kUnknown) {     // a unit of less than three steps, or an empty queue
                if (share_next < share_end) next_unit = share_next;
                else next_unit = claim_from(T >= 3 ? __builtin_amdgcn_readfirstlane(next_ticket) : __builtin_amdgcn_readfirstlane(take_ticket()));
                if (next_unit >= 0) fetch_record(next_unit);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
            if (lane == 0) mailbox[kRecordInts] = next_unit;
            __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the mailbox write is in LDS before the barrier
        }
        __builtin_amdgcn_s_barrier();
        ++share_next;
    }
}

template <int D>
__global__ __launch_bounds__(kPingPongThreads, 2) void attn_prefill_bf16(
    KernelArgs a, const uint64_t *__restrict__ map_text_bits, const uint64_t *__restrict__ map_sink_bits,
    const int4 *__restrict__ map_rows, const UnitRecord *__restrict__ units,
    const int2 *__restrict__ pair_ranges, const __bf16 *__restrict__ kp, const __bf16 *__restrict__ vp,
    int32_t n_k_tiles, int32_t *__restrict__ queue_ctr, const int32_t *__restrict__ queue_off,
    const int32_t *__restrict__ share_off, const StackedRows *__restrict__ stacked, float *__restrict__ cut_results)
{
    walk_units<D, 1, true>(a, map_text_bits, map_sink_bits, map_rows, units, pair_ranges, kp, vp, n_k_tiles, queue_ctr, queue_off, share_off, stacked, cut_results);
}

template <int D>
__global__ __launch_bounds__(kPingPongThreads, 2) void attn_prefill_bf16_two(
    KernelArgs a, const uint64_t *__restrict__ map_text_bits, const uint64_t *__restrict__ map_sink_bits,
    const int4 *__restrict__ map_rows, const UnitRecord *__restrict__ units,
    const int2 *__restrict__ pair_ranges, const __bf16 *__restrict__ kp, const __bf16 *__restrict__ vp,
    int32_t n_k_tiles, int32_t *__restrict__ queue_ctr, const int32_t *__restrict__ queue_off,
    const int32_t *__restrict__ share_off, const StackedRows *__restrict__ stacked, float *__restrict__ cut_results)
{
    walk_units<D, 2, true>(a, map_text_bits, map_sink_bits, map_rows, units, pair_ranges, kp, vp, n_k_tiles, queue_ctr, queue_off, share_off, stacked, cut_results);
}

template <int D>
__global__ __launch_bounds__(kPingPongThreads, 2) void attn_prefill_bf16_v(
    KernelArgs a, const uint64_t *__restrict__ map_text_bits, const uint64_t *__restrict__ map_sink_bits,
    const int4 *__restrict__ map_rows, const UnitRecord *__restrict__ units,
    const int2 *__restrict__ pair_ranges, const __bf16 *__restrict__ kp, const __bf16 *__restrict__ vp,
    int32_t n_k_tiles, int32_t *__restrict__ queue_ctr, const int32_t *__restrict__ queue_off,
    const int32_t *__restrict__ share_off, const StackedRows *__restrict__ stacked, float *__restrict__ cut_results)
{
    walk_units<D, 1, false>(a, map_text_bits, map_sink_bits, map_rows, units, pair_ranges, kp, vp, n_k_tiles, queue_ctr, queue_off, share_off, stacked, cut_results);
}

template <int D>
__global__ __launch_bounds__(kPingPongThreads, 2) void attn_prefill_bf16_two_v(
    KernelArgs a, const uint64_t *__restrict__ map_text_bits, const uint64_t *__restrict__ map_sink_bits,
    const int4 *__restrict__ map_rows, const UnitRecord *__restrict__ units,
    const int2 *__restrict__ pair_ranges, const __bf16 *__restrict__ kp, const __bf16 *__restrict__ vp,
    int32_t n_k_tiles, int32_t *__restrict__ queue_ctr, const int32_t *__restrict__ queue_off,
    const int32_t *__restrict__ share_off, const StackedRows *__restrict__ stacked, float *__restrict__ cut_results)
{
    walk_units<D, 2, false>(a, map_text_bits, map_sink_bits, map_rows, units, pair_ranges, kp, vp, n_k_tiles, queue_ctr, queue_off, share_off, stacked, cut_results);
}

}  // namespace bs

using bs::DeviceMap;

// ------------------------------------------------------------------------------------ launch

// Scratch of the entry point that allocates nothing (bs_attn_prefill_static): packed K tiles, then
// packed V^T tiles.  Every GPU the library runs on holds its own copy until the process ends.  In
// host code the name below is only a handle for hipGetSymbolAddress; kernels get the per-device
// address that call returns.
constexpr size_t kStaticScratchBytes = (size_t)BS_STATIC_SCRATCH_MIB << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_device_mutex;
void *g_scratch_ptr[kMaxDevices];       // device address of `scratch` on each device (looked up once)
bool g_attr_set[kMaxDevices];           // dynamic-LDS limits of the kernels raised on this device
int g_n_cus[kMaxDevices];               // compute units of the device

// Once per device, with that device current: the address of its copy of `scratch`, and the
// kernels' dynamic LDS limits.  Allocates nothing.
int device_setup(int dev, void **scratch_out, int *n_cus_out)
{
    if (dev < 0 || dev >= kMaxDevices) return bs::fail_msg(BS_EUNSUPPORTED, "device ordinal above 63");
    std::lock_guard<std::mutex> lock(g_device_mutex);
    hipError_t e;
    if (!g_attr_set[dev]) {
        const auto lds_limit = [&](const void *kernel, int bytes) { if (e == hipSuccess) e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes); };
        e = hipSuccess;
        lds_limit(reinterpret_cast<const void *>(bs::attn_prefill_bf16<128>), bs::bf16_lds_bytes<128, 1>());
        lds_limit(reinterpret_cast<const void *>(bs::attn_prefill_bf16<64>), bs::bf16_lds_bytes<64, 1>());
        lds_limit(reinterpret_cast<const void *>(bs::attn_prefill_bf16_two<64>), bs::bf16_lds_bytes<64, 2>());
        lds_limit(reinterpret_cast<const void *>(bs::attn_prefill_bf16_v<128>), bs::bf16_lds_bytes<128, 1>());
        lds_limit(reinterpret_cast<const void *>(bs::attn_prefill_bf16_v<64>), bs::bf16_lds_bytes<64, 1>());
        lds_limit(reinterpret_cast<const void *>(bs::attn_prefill_bf16_two_v<64>), bs::bf16_lds_bytes<64, 2>());
        if (e == hipSuccess) e = bs::f32_device_setup();
        if (e == hipSuccess) e = bs::rows_device_setup();
        if (e != hipSuccess) return bs::fail_hip(e, "hipFuncSetAttribute");
        int cus = 0;
        e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess || cus <= 0) return bs::fail_hip(e, "hipDeviceGetAttribute(compute units)");
        g_n_cus[dev] = cus;
        g_attr_set[dev] = true;
    }
    if (n_cus_out) *n_cus_out = g_n_cus[dev];
    if (scratch_out) {
        if (!g_scratch_ptr[dev]) {
            void *ptr = nullptr;
            e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
            if (e != hipSuccess || !ptr) return bs::fail_hip(e, "hipGetSymbolAddress(scratch)");
            g_scratch_ptr[dev] = ptr;
        }
        *scratch_out = g_scratch_ptr[dev];
    }
    return BS_OK;
}

int check_call(const void *q, const void *k, const void *v, void *out, const bs_tilemap *tm, int32_t dtype,
               int32_t n_q_heads, int32_t gqa_group, int32_t head_dim, float scale)
{
    if (!q || !k || !v || !out || !tm) return BS_EINVAL;
    if (n_q_heads <= 0 || gqa_group <= 0 || n_q_heads % gqa_group != 0) return BS_EINVAL;
    if (n_q_heads != tm->n_q_heads) return BS_EINVAL;
    if (!(scale > 0.f) || !(scale < INFINITY)) return BS_EINVAL;  // masking relies on -inf * scale = -inf
    if (tm->bm != bs::kBlockM || tm->bn != bs::kBlockN) return BS_EUNSUPPORTED;
    if (head_dim != 64 && head_dim != 128) return BS_EUNSUPPORTED;
    if (dtype != BS_BF16 && dtype != BS_F32) return BS_EUNSUPPORTED;
    if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)out) & 15) return BS_EINVAL;
    return BS_OK;
}

bs::KernelArgs kernel_args(const void *q, const void *k, const void *v, void *out, const bs_tilemap *tm,
                           int32_t gqa_group, float scale)
{
    bs::KernelArgs a;
    a.q = q; a.k = k; a.v = v; a.out = out;
    a.L = tm->L; a.G = gqa_group;
    a.scale_log2e = scale * 1.4426950408889634f;
    a.n_prompt_tiles = tm->N0;
    a.text_tile0 = tm->text_tile0;
    a.n_tiles = tm->n_tiles;
    a.first_tile = 0;
    a.window = tm->window;
    a.bidir = tm->bidir;
    a.q_begin = tm->q_begin;
    return a;
}

// The key tiles that a launch of the bf16 kernel reads, at least one: runs of the prompt's, of free keys, of text keys.
struct TileRuns { int32_t first[3], end[3]; };

// Those of the classes that the map is bound to, or of all that the kernels know.
TileRuns tiles_read(const bs_tilemap *tm, bool all)
{
    TileRuns t = {{0, tm->N0, tm->text_tile0}, {tm->N0, tm->text_tile0, tm->n_tiles}};
    if (all) return t;
    bool bound[4] = {false, false, false, false};
    for (uint8_t c : tm->head_class) bound[c] = true;
    for (int kind = 0; kind < 3; ++kind) {
        int32_t first = INT32_MAX, end = 0;
        for (int c = 0; c < 4; ++c) {
            if (!bound[c] || tm->walked(c).span[kind].end == 0) continue;
            first = std::min(first, tm->walked(c).span[kind].first);
            end = std::max(end, tm->walked(c).span[kind].end);
        }
        t.first[kind] = end == 0 ? t.first[kind] : first;
        t.end[kind] = end == 0 ? t.first[kind] : end;
    }
    if (t.end[0] == t.first[0]) t.end[0] = t.first[0] + 1;   // (an empty list's walker names it)
    return t;
}

// Whether the bf16 kernel walks two key tiles a step at d = 64.  A step of one tile is 16 MFMAs and the softmax of 64 keys, behind the
// same barrier, head reads and walk as the 32 MFMAs at d = 128; two tiles share them: 32 heads, all Dense, 36K tokens 5.72 -> 5.18 ms
// (1.10 -> 1.00 us a tile; the vector ALU is busy for some 0.75 of that).  A list of an odd length costs one tile more, and in front of
// a unit's first step lie twice the bytes.  Passes with one / two, by tiles per unit or share: 7 (700 tokens) 65.9 / 68.5 us, 8 (100
// rows behind 9K) 84.9 / 87.6, 8-10 (window of 512) 291 / 300, 11-20 (window of 1024 on 27K) 972 / 973, 16 (4K) 107.4 / 107.1,
// 30-72 (9K) 885 / 834, 126 (40K) 2833 / 2596.
bool steps_of_two(const DeviceMap *d, const bs::ShareSet *sh)
{
    constexpr int64_t kTilesPerUnit = 12;
    return d->n_steps >= kTilesPerUnit * std::max(d->n_pairs, sh ? sh->n_shares : 0);
}

// Key tiles that the runs name, of all KV heads.
int64_t tiles_of(const TileRuns &read, int n_kv_heads)
{
    int64_t tiles = 0;
    for (int i = 0; i < 3; ++i) tiles += read.end[i] - read.first[i];
    return tiles * n_kv_heads;
}

bool overlap(const void *a, size_t a_bytes, const void *b, size_t b_bytes)
{
    return (uintptr_t)a < (uintptr_t)b + b_bytes && (uintptr_t)b < (uintptr_t)a + a_bytes;
}

// Pre-pass (K and V or V^T into per-key-tile blocks of `workspace`) and the attention kernel.  kv_packed: the workspace
// holds these tiles already and the binding was just uploaded, its queue counters at zero; shared_pack: they are for calls with several
// bindings.  sh: null, the queues.  k_bytes:
// what the packed K tiles take, in front of the V^T tiles.  units: the copy of the work units, if it is still to do.  A launch that
// fails is the last one: the kernels behind it would read what it did not write.
template <int D>
hipError_t launch_bf16(bs::KernelArgs a, const bs_tilemap *tm, const DeviceMap *d, const TileRuns &todo_tiles, void *workspace, size_t k_bytes,
                       float *cut_results, int n_kv_heads, int n_cus, const bs::ShareSet *sh, bool shared_pack, bool kv_packed, bs::PendingCopy *units, hipStream_t st, void *ev_main_start)
{
    a.first_tile = todo_tiles.first[0];
    __bf16 *kp = static_cast<__bf16 *>(workspace);
    __bf16 *vp = reinterpret_cast<__bf16 *>(static_cast<char *>(workspace) + k_bytes);
    const int32_t in_place = tm->L / bs::kBlockN;
    // (a result that is written over V needs the copy, and the calls that share a pre-pass take what it made)
    const size_t row_bytes = (size_t)D * 2;
    const bool transpose = shared_pack || bs::transposed_values(D, d->n_steps, tiles_of(todo_tiles, n_kv_heads)) ||
                           overlap(a.out, row_bytes * tm->n_q_heads * (tm->L - tm->q_begin), a.v, row_bytes * n_kv_heads * tm->L);
    // one workgroup per CU (160 KB of LDS each; 96 KB for steps of one tile at d = 64), which take the units from the queues until they are empty
    const dim3 pgrid((unsigned)(sh ? sh->n_shares : std::min(d->n_pairs, n_cus))), pblock(bs::kPingPongThreads);
    const size_t n_copy = units && !kv_packed ? units->n : 0;   // comes with the pre-pass
    hipError_t e = hipSuccess;
    if (kv_packed) {
        if (units) e = bs::copy_pending(units, st);
    } else {
        bs::PackTiles todo;
        int32_t n_todo = 0;
        for (int i = 0; i < 6; ++i) {
            const int32_t first = std::max(todo_tiles.first[i % 3], i < 3 && transpose ? 0 : in_place);
            todo.first[i] = first;
            todo.count[i] = std::max(0, todo_tiles.end[i % 3] - first);
            n_todo += todo.count[i];
        }
        // the copy of the units: one load a thread, as the latency of the bus is all there is to it, up to 4 MB
        const size_t copy_wgs = std::min<size_t>((n_copy + 255) / 256, 1024);
        const size_t copy_x = (copy_wgs + n_kv_heads - 1) / n_kv_heads;
        todo.n_tiles = n_todo;
        todo.transpose = transpose;
        e = bs::launch_kernel(bs::pack_kv_tiles<D>, dim3((unsigned)std::max<size_t>(n_todo + copy_x, 1), (unsigned)n_kv_heads), dim3(256), 0, st, static_cast<const __bf16 *>(a.k),
                              static_cast<const __bf16 *>(a.v), kp, vp, d->compact_keys, tm->L, tm->n_tiles, tm->N0, in_place, todo, d->queue_ctr,
                              n_copy ? units->src : nullptr, n_copy ? units->dst : nullptr, n_copy);
        if (e != hipSuccess && n_copy) bs::staging_abandon(units->staging);
    }
    if (e != hipSuccess) return e;
    if (ev_main_start) (void)hipEventRecord(static_cast<hipEvent_t>(ev_main_start), st);
    const auto launch = [&](auto *kernel, int lds_bytes) {
        return bs::launch_kernel(kernel, pgrid, pblock, lds_bytes, st, a, d->text_bits,
                                 d->sink_bits, d->rows, sh ? sh->units : d->units, sh ? sh->ranges : d->pair_ranges, kp, vp, tm->n_tiles,
                                 d->queue_ctr, sh ? sh->queue_off : d->queue_off, sh ? sh->off : nullptr, d->stacked, cut_results);
    };
    if constexpr (D == 64) {
        if (steps_of_two(d, sh)) e = launch(transpose ? &bs::attn_prefill_bf16_two<64> : &bs::attn_prefill_bf16_two_v<64>, bs::bf16_lds_bytes<64, 2>());
        else e = launch(transpose ? &bs::attn_prefill_bf16<64> : &bs::attn_prefill_bf16_v<64>, bs::bf16_lds_bytes<64, 1>());
    } else {
        e = launch(transpose ? &bs::attn_prefill_bf16<128> : &bs::attn_prefill_bf16_v<128>, bs::bf16_lds_bytes<128, 1>());
    }
    if (e == hipSuccess && sh && sh->n_cut > 0)
        e = bs::launch_kernel(bs::merge_cut_items<D, 2, __bf16>, dim3((unsigned)sh->n_cut, 4, D / 32), dim3(64), 0, st, a, sh->cut_items,
                              d->rows, d->stacked, cut_results);
    if (n_copy) {   // (an event between the two kernels would hold the second one up)
        const hipError_t queued = bs::staging_queued(units->staging, st);
        if (e == hipSuccess) e = queued;
    }
    return e;
}

// Bytes of the results of cut units (0 without equal shares).
size_t cut_bytes(const bs::ShareSet &shares, int head_dim)
{
    return (size_t)shares.n_slots * 2 * 4 * (head_dim == 128 ? bs::kCutItemFloats<128> : bs::kCutItemFloats<64>);
}

// The workspace of the map's calls, owned by the map: at least `bytes`, for work queued on `st` after this.
int take_workspace(DeviceMap *d, size_t bytes, hipStream_t st)
{
    if (d->vt_bytes >= bytes) return BS_OK;
    // (a workspace that grows takes a quarter more, so that the outgrown ones add up to a few times the last)
    const size_t want = std::max(bytes, d->vt_bytes + d->vt_bytes / 4);
    if (d->vt_buf) {
        try {
            d->outgrown.push_back({d->vt_buf, d->vt_bytes});
        } catch (const std::bad_alloc &) {
            return BS_ENOMEM;
        }
    }
    d->vt_buf = nullptr; d->vt_bytes = 0;
    hipError_t e = bs::pool_acquire(d->device, want, st, &d->vt_buf, &d->vt_bytes);
    if (e != hipSuccess && want > bytes) {
        (void)hipGetLastError();
        e = bs::pool_acquire(d->device, bytes, st, &d->vt_buf, &d->vt_bytes);
    }
    if (e == hipSuccess) return BS_OK;
    d->vt_buf = nullptr; d->vt_bytes = 0;
    return bs::fail_hip(e, "hipMalloc(workspace)");
}

size_t bf16_pack_bytes(int32_t n_tiles, int n_kv_heads, int head_dim)
{
    return (size_t)n_kv_heads * n_tiles * (size_t)head_dim * bs::kBlockN * 2;   // of K or V^T
}

// What the pre-pass writes at most: the K tiles that are not read in place, then all V^T tiles.
struct PackBytes { size_t k, all; };
PackBytes bf16_pack_bytes(const bs_tilemap *tm, int n_kv_heads, int head_dim)
{
    const size_t k = bf16_pack_bytes(tm->n_tiles - tm->L / bs::kBlockN, n_kv_heads, head_dim);
    return {k, k + bf16_pack_bytes(tm->n_tiles, n_kv_heads, head_dim)};
}

}  // namespace

extern "C" int bs_tilemap_upload(bs_tilemap *tm)
{
    if (!tm) return BS_EINVAL;
    if (tm->dev && tm->dev->blob) return BS_OK;
    const int rc = bs::upload_prompt_part(tm, nullptr);
    if (rc != BS_OK) return rc;
    const hipError_t e = hipStreamSynchronize(nullptr);   // this entry point promises a finished upload
    return e == hipSuccess ? BS_OK : bs::fail_hip(e, "hipStreamSynchronize");
}

extern "C" int bs_tilemap_prepare(bs_tilemap *tm, int32_t dtype, int32_t gqa_group, void *stream)
{
    if (!tm || gqa_group <= 0 || tm->n_q_heads % gqa_group != 0) return BS_EINVAL;
    if (dtype != BS_BF16 && dtype != BS_F32) return BS_EUNSUPPORTED;
    if (tm->bm != bs::kBlockM || tm->bn != bs::kBlockN) return BS_EUNSUPPORTED;
    hipStream_t st = static_cast<hipStream_t>(stream);
    int rc = bs::upload_prompt_part(tm, st);
    if (rc != BS_OK) return rc;
    DeviceMap *d = tm->dev;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return bs::fail_hip(e, "hipGetDevice");
    if (dev != d->device) return BS_EINVAL;  // the map lives on another device
    void *unused = nullptr;
    int n_cus = 0;
    if ((rc = device_setup(dev, &unused, &n_cus)) != BS_OK) return rc;
    if ((rc = bs::order_after_last_use(d, st)) != BS_OK) return rc;
    if (dtype == BS_BF16) {
        rc = bs::upload_binding(tm, bs::kBindPairPlan, gqa_group, n_cus, 0, st, nullptr);
        if (rc == BS_OK) {   // results of cut units that have no room in the static scratch (the head dimension is not known yet)
            const int n_kv_heads = tm->n_q_heads / gqa_group;
            const size_t cut = cut_bytes(*d->shares_for(n_cus), 128);
            if (2 * bf16_pack_bytes(tm->N, n_kv_heads, 64) <= kStaticScratchBytes &&
                bf16_pack_bytes(tm, n_kv_heads, 128).all + cut > kStaticScratchBytes) rc = take_workspace(d, cut, st);
        }
    } else {   // for either head dimension, and the workspace of the larger plan
        const int32_t wgs128 = n_cus * bs::f32_wgs_per_cu(128), wgs64 = n_cus * bs::f32_wgs_per_cu(64);
        rc = bs::upload_binding(tm, bs::kBindSolo, gqa_group, wgs128, wgs64, st, nullptr);
        if (rc == BS_OK)
            rc = take_workspace(d, std::max(bs::f32_workspace(*d->shares_for(wgs128), 128), bs::f32_workspace(*d->shares_for(wgs64), 64)), st);
    }
    e = hipEventRecord(d->last_use->ev, st);   // (also without a workspace: the units are on their way)
    if (rc != BS_OK) return rc;
    return e == hipSuccess ? BS_OK : bs::fail_hip(e, "hipEventRecord");
}

extern "C" int bs_attn_prefill(const void *q, const void *k, const void *v, void *out, bs_tilemap *tm,
                               int32_t dtype, int32_t n_q_heads, int32_t gqa_group, int32_t head_dim,
                               float scale, void *stream)
{
    return bs_attn_prefill_ex(q, k, v, out, tm, dtype, n_q_heads, gqa_group, head_dim, scale, stream, nullptr, nullptr);
}

extern "C" int bs_attn_prefill_ex(const void *q, const void *k, const void *v, void *out, bs_tilemap *tm,
                                  int32_t dtype, int32_t n_q_heads, int32_t gqa_group, int32_t head_dim,
                                  float scale, void *stream, void *ev_main_start, void *ev_main_stop)
{
    return bs::attn_prefill(q, k, v, out, tm, dtype, n_q_heads, gqa_group, head_dim, scale, stream, ev_main_start, ev_main_stop, nullptr);
}

int bs::attn_prefill(const void *q, const void *k, const void *v, void *out, bs_tilemap *tm, int32_t dtype,
                     int32_t n_q_heads, int32_t gqa_group, int32_t head_dim, float scale, void *stream,
                     void *ev_main_start, void *ev_main_stop, bool *kv_packed)
{
    int rc = check_call(q, k, v, out, tm, dtype, n_q_heads, gqa_group, head_dim, scale);
    if (rc != BS_OK) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if ((rc = bs::ensure_device_map(tm, st)) != BS_OK) return rc;
    DeviceMap *d = tm->dev;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return bs::fail_hip(e, "hipGetDevice");
    if (dev != d->device) return BS_EINVAL;  // the map lives on another device
    int n_cus = 0;
    if ((rc = device_setup(dev, nullptr, &n_cus)) != BS_OK) return rc;
    if ((rc = bs::order_after_last_use(d, st)) != BS_OK) return rc;
    const bs::RowsPlan rows = bs::plan_rows(tm, dtype, gqa_group, head_dim, n_cus);
    const uint64_t bound = d->bind_epoch;
    // The work units on their way: the bf16 pre-pass brings them, for fp32 the kernel that makes the prompt part (which for
    // bf16 is launched before the units are planned: the two then run side by side).
    bs::PendingCopy units;
    const auto give_up = [&](int code) {
        if (units.n == 0) return code;
        if (bs::copy_pending(&units, st) != hipSuccess) d->bind_kind = bs::kBindNone;
        (void)hipEventRecord(d->last_use->ev, st);   // the copy uses the map's block
        return code;
    };
    const int32_t n_wgs = dtype == BS_BF16 ? n_cus : n_cus * bs::f32_wgs_per_cu(head_dim);
    const auto bind = [&] { return bs::upload_binding(tm, dtype == BS_BF16 ? bs::kBindPairPlan : bs::kBindSolo, gqa_group, n_wgs, 0, st, &units); };
    if (!rows.use || rows.need_bits) {
        rc = dtype == BS_F32 ? bs::upload_prompt_part(tm, st, &units, bind) : bs::upload_prompt_part(tm, st);
        if (rc != BS_OK) return give_up(rc);
    }
    if (!rows.use)
        if ((rc = bind()) != BS_OK) return rc;

    const bs::KernelArgs a = kernel_args(q, k, v, out, tm, gqa_group, scale);
    if (rows.use) {
        if ((rc = take_workspace(d, rows.workspace, st)) != BS_OK) return rc;
        if (ev_main_start) (void)hipEventRecord(static_cast<hipEvent_t>(ev_main_start), st);
        bs::launch_rows(rows, q, k, v, out, tm, d, d->vt_buf, gqa_group, head_dim, scale, st);
        d->rows_epoch = tm->class_epoch;
        d->rows_G = gqa_group;
    } else if (dtype == BS_BF16) {
        const int n_kv_heads = n_q_heads / gqa_group;
        const PackBytes pack = bf16_pack_bytes(tm, n_kv_heads, head_dim);
        const bs::ShareSet &shares = *d->shares_for(n_wgs);
        const bs::ShareSet *const sh = shares.n_shares > 0 ? &shares : nullptr;
        const void *const old_workspace = d->vt_buf;
        if ((rc = take_workspace(d, pack.all + cut_bytes(shares, head_dim), st)) != BS_OK) return give_up(rc);
        const bool packed = kv_packed && *kv_packed && d->vt_buf == old_workspace && d->bind_epoch != bound;
        float *const cut = reinterpret_cast<float *>(static_cast<char *>(d->vt_buf) + pack.all);
        // (a caller with several bindings of the map packs for all of them)
        const TileRuns todo = tiles_read(tm, kv_packed != nullptr);
        e = head_dim == 128 ? launch_bf16<128>(a, tm, d, todo, d->vt_buf, pack.k, cut, n_kv_heads, n_cus, sh, kv_packed != nullptr, packed, &units, st, ev_main_start)
                            : launch_bf16<64>(a, tm, d, todo, d->vt_buf, pack.k, cut, n_kv_heads, n_cus, sh, kv_packed != nullptr, packed, &units, st, ev_main_start);
        if (e != hipSuccess) {
            d->bind_kind = bs::kBindNone;   // the units may not have arrived
            if (kv_packed) *kv_packed = false;
            (void)hipEventRecord(d->last_use->ev, st);   // what was launched uses the map's blocks
            return bs::fail_hip(e, "kernel launch");
        }
    } else {
        const bs::ShareSet &shares = *d->shares_for(n_wgs);
        if ((rc = take_workspace(d, bs::f32_workspace(shares, head_dim), st)) != BS_OK) return give_up(rc);
        if ((e = bs::copy_pending(&units, st)) != hipSuccess) {
            d->bind_kind = bs::kBindNone;
            return bs::fail_hip(e, "copy of the work units");
        }
        if (ev_main_start) (void)hipEventRecord(static_cast<hipEvent_t>(ev_main_start), st);
        bs::launch_f32(a, d, shares, d->vt_buf, head_dim, st);
    }
    if (kv_packed) *kv_packed = !rows.use && dtype == BS_BF16;
    e = hipGetLastError();
    if (e != hipSuccess) return bs::fail_hip(e, "kernel launch");
    if (ev_main_stop) (void)hipEventRecord(static_cast<hipEvent_t>(ev_main_stop), st);
    e = hipEventRecord(d->last_use->ev, st);
    if (e != hipSuccess) return bs::fail_hip(e, "hipEventRecord");
    return BS_OK;
}

extern "C" int64_t bs_static_scratch_bytes(void) { return (int64_t)kStaticScratchBytes; }

extern "C" int bs_attn_prefill_static(const void *q, const void *k, const void *v, void *out, bs_tilemap *tm,
                                      int32_t n_q_heads, int32_t gqa_group, int32_t head_dim, float scale, void *stream)
{
    int rc = check_call(q, k, v, out, tm, BS_BF16, n_q_heads, gqa_group, head_dim, scale);
    if (rc != BS_OK) return rc;
    DeviceMap *d = tm->dev;
    const auto not_prepared = [] {
        return bs::fail_msg(BS_EINVAL, "bs_attn_prefill_static: call bs_tilemap_prepare(tm, BS_BF16, gqa_group, stream) first "
                                       "(after every bs_tilemap_rebind); this entry point uploads and allocates nothing");
    };
    if (!d) return not_prepared();
    const bool units_bound = d->bind_kind == bs::kBindPairPlan && d->bind_G == gqa_group && d->bind_epoch == tm->class_epoch;
    const bool rows_bound = d->rows_G == gqa_group && d->rows_epoch == tm->class_epoch;
    if (!units_bound && !rows_bound) return not_prepared();
    const int n_kv_heads = n_q_heads / gqa_group;
    const PackBytes pack = bf16_pack_bytes(tm, n_kv_heads, head_dim);
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return bs::fail_hip(e, "hipGetDevice");
    if (dev != d->device) return BS_EINVAL;  // the map lives on another device
    void *ws = nullptr;
    int n_cus = 0;
    if ((rc = device_setup(dev, &ws, &n_cus)) != BS_OK) return rc;   // looks the address up on the first call per device
    const bs::RowsPlan rows = bs::plan_rows(tm, BS_BF16, gqa_group, head_dim, n_cus);
    if (!units_bound && !rows.use) return not_prepared();
    // (one limit for all calls and maps, on the published tiles, K and V^T: the call needs less -- the few-row kernel, K tiles read
    // in place -- and with at most half as many more tiles that only the kernels know it fits all the same)
    const size_t limit_bytes = 2 * bf16_pack_bytes(tm->N, n_kv_heads, head_dim);
    if (std::max(rows.workspace, limit_bytes) > kStaticScratchBytes || pack.all > kStaticScratchBytes) {
        snprintf(bs::g_last_error, sizeof bs::g_last_error,
                 "bs_attn_prefill_static: packed K / V^T tiles need %zu bytes, the static scratch holds %zu "
                 "(n_kv_heads * key tiles * head_dim * 256 bytes); use bs_attn_prefill", limit_bytes, kStaticScratchBytes);
        return BS_EUNSUPPORTED;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    if ((rc = bs::order_after_last_use(d, st)) != BS_OK) return rc;
    const bs::KernelArgs a = kernel_args(q, k, v, out, tm, gqa_group, scale);
    // the results of cut units go behind the packed tiles or, if they do not fit there, to the workspace that
    // bs_tilemap_prepare took (too small only if a call at head dimension 64 made the binding: then nothing is cut)
    const bs::ShareSet *sh = d->shares_for(n_cus);
    if (sh && sh->n_shares == 0) sh = nullptr;
    float *cut = reinterpret_cast<float *>(static_cast<char *>(ws) + pack.all);
    if (sh && pack.all + cut_bytes(*sh, head_dim) > kStaticScratchBytes) {
        cut = static_cast<float *>(d->vt_buf);
        if (cut_bytes(*sh, head_dim) > d->vt_bytes) sh = nullptr;
    }
    // the pre-pass (the few-row kernel) writes all of the scratch that is read after it: nothing of the previous
    // call's contents is
    e = hipSuccess;
    if (rows.use) bs::launch_rows(rows, q, k, v, out, tm, d, ws, gqa_group, head_dim, scale, st);
    else if (head_dim == 128) e = launch_bf16<128>(a, tm, d, tiles_read(tm, false), ws, pack.k, cut, n_kv_heads, n_cus, sh, false, false, nullptr, st, nullptr);
    else e = launch_bf16<64>(a, tm, d, tiles_read(tm, false), ws, pack.k, cut, n_kv_heads, n_cus, sh, false, false, nullptr, st, nullptr);
    if (e == hipSuccess) e = hipGetLastError();
    if (e != hipSuccess) return bs::fail_hip(e, "kernel launch");
    e = hipEventRecord(d->last_use->ev, st);
    if (e != hipSuccess) return bs::fail_hip(e, "hipEventRecord");
    return BS_OK;
}

extern "C" const char *bs_last_error(void) { return bs::g_last_error; }
