// Internal layout of bs_tilemap, shared by the host builder and the HIP launcher.
#pragma once
#include <cstdint>
#include <mutex>
#include <utility>
#include <vector>

#include "blindsight.h"

namespace bs {

constexpr int32_t kMaxSpans = 0x3fffffff;

// One image span and the prompt up to it.
struct SpanInfo {
    int32_t start, end;
    int32_t prefix;        // leading sink tokens: the span's own sink count, or the prompt's sink prefix if that reaches further
    int32_t text_before;   // text tokens at positions < start
    int32_t free_before;   // text or sink tokens at positions < start
    int32_t last_text;     // last text position < start, or -1
    int32_t next_text;     // first text position >= end, or L
    int32_t pad;
};

// The prompt as its span table: everything the builders, the introspection calls and the device copy need is a closed
// form of it, so no array over the tokens exists on the host.
struct PromptGeometry {
    int32_t L = 0, bm = 0, bn = 0, M = 0, N0 = 0, n_spans = 0, sink_len = 0, q_begin = 0, window = 0;
    bool bidir = false;                 // tokens of one image also see the later tokens of that image
    bool regrouped = false;             // query rows: image rows first, then text rows
    int32_t n_img_rows = 0, m_img = 0;  // regrouped: image rows and the tiles that hold them
    std::vector<SpanInfo> spans;        // n_spans + 1: a sentinel that starts at L
    std::vector<int32_t> offsets;       // sorted in-image offsets that are sinks in every image
    std::vector<int32_t> block_first;   // first span that ends behind position 64 b

    void init(const bs_span *sp, int32_t n, int32_t seq_len, int32_t sink_prefix, const int32_t *offs, int32_t n_offs);
    // first span with end > t (n_spans if none), 0 <= t <= L
    int32_t span_at(int32_t t) const
    {
        int32_t g = block_first[t >> 6];
        while (g < n_spans && spans[g].end <= t) ++g;
        return g;
    }
    int32_t offsets_below(int32_t x) const
    {
        int32_t i = 0;
        if (!offsets.empty() && offsets.back() < x) return (int32_t)offsets.size();
        for (int32_t n = (int32_t)offsets.size(); n > 0;) {   // lower bound
            const int32_t half = n / 2;
            if (offsets[i + half] < x) { i += half + 1; n -= half + 1; } else n = half;
        }
        return i;
    }
    // sink tokens among the first x of image g
    int32_t sinks_in(int32_t g, int32_t x) const
    {
        const int32_t p = x < spans[g].prefix ? x : spans[g].prefix;
        return offsets.empty() ? p : p + offsets_below(x) - offsets_below(p);
    }
    // text tokens / text or sink tokens at positions < t
    int32_t n_text(int32_t t) const
    {
        const SpanInfo &s = spans[span_at(t)];
        return t > s.start ? s.text_before : s.text_before - (s.start - t);
    }
    int32_t n_free(int32_t t) const
    {
        const int32_t g = span_at(t);
        const SpanInfo &s = spans[g];
        return t > s.start ? s.free_before + sinks_in(g, t - s.start) : s.free_before - (s.start - t);
    }
    // free keys for a class: text, with the sink bit also sinks
    int32_t free_count(int cls, int32_t t) const { return (cls & 1) ? n_free(t) : n_text(t); }
    int32_t last_text(int32_t t) const   // largest text position <= t, or -1 (t < L)
    {
        const SpanInfo &s = spans[span_at(t)];
        return t >= s.start ? s.last_text : t;
    }
    int32_t next_text(int32_t t) const   // smallest text position >= t, or L
    {
        const SpanInfo &s = spans[span_at(t)];
        return t >= s.start ? s.next_text : t;
    }
    int32_t next_free(int cls, int32_t t) const;       // smallest free position >= t, or L
    int32_t free_position(int32_t slot) const;         // position of the slot-th free token
    int32_t text_position(int32_t slot) const;         // position of the slot-th text token
    int32_t first_visible(int32_t i) const             // first position a query at i may see (window > 0)
    {
        const int32_t w = i >= window ? i - window + 1 : 0;
        if (!bidir) return w;
        const SpanInfo &s = spans[span_at(i)];
        return i >= s.start && s.start < w ? s.start : w;
    }
    int32_t n_text_rows() const { return regrouped ? L - q_begin - n_img_rows : 0; }
    int32_t n_other_rows() const { return L - q_begin - n_text_rows(); }
    // rows number first .. last - 1 of the text rows, or of the others (the image rows of a regrouped map, else all), as runs
    // [first, second) of positions, behind those in `runs`
    void row_runs(bool text, int32_t first, int32_t last, std::vector<std::pair<int32_t, int32_t>> &runs) const;
    // the rows of query tile m as such runs; returns how many rows
    int32_t tile_runs(int32_t m, std::vector<std::pair<int32_t, int32_t>> &runs) const;
};

// Half-open run of key tiles [begin, end) that all share one state.
struct TileRange {
    int32_t begin;
    int32_t end_state;  // (end << 1) | (1 if FULL, 0 if PARTIAL)
    int32_t end() const { return end_state >> 1; }
    bool full() const { return end_state & 1; }
};

struct ClassLists {
    std::vector<int64_t> row_ptr;     // M + 1 offsets into ranges; empty: not built
    std::vector<TileRange> ranges;
    std::vector<int32_t> row_tiles;   // visited tiles per query tile (scheduling weight)
    std::vector<uint8_t> compact;     // per query tile: its image rows take the keys outside their own image from compact tiles
    int64_t visited = 0, full = 0, partial = 0;
    // Per kind of key tile (prompt, free keys, text keys): the visited ones lie in [first, end); both 0: none.
    struct { int32_t first = 0, end = 0; } span[3];
};

// Work unit of the bf16 kernel: two (head, query tile) items that read the SAME KV head and walk
// one merged key-tile list, so a workgroup streams each K / V tile once for both.
//   item B is absent when head_b < 0.
struct PairItem {
    int32_t head_a, tile_a, head_b, tile_b;
    int32_t list_begin, list_end;  // entries of PairPlan::ranges
    int32_t n_tiles;               // key tiles in the merged list (scheduling weight)
    int32_t classes;               // item A | item B << 8; an item: its head's class | ClassLists::compact of its tile << 2 | stacked << 3
};

// Run of key tiles [begin, end) with one state per item: 0 skip, 1 partial, 2 full.
struct PairRange {
    int32_t begin;
    int32_t end_states;  // (end << 4) | (state_a << 2) | state_b
};

// A unit of the bf16 kernel in the device copy, with the beginning of its walk: its first tiles and what follows them are known as
// soon as the record is.  A tile is named with its states, (n << 4) | states.
struct UnitRecord {
    int32_t head_a, tile_a, head_b, tile_b;
    int32_t n_tiles, classes;                 // as in PairItem
    int32_t kv_head;
    int32_t list_end;                         // of its runs
    int32_t tile[4];                          // the first four; of a shorter list the last one again, skipped by both items
    int32_t run_end;                          // end_states of the run that tile[3] is in
    int32_t next_begin, next_end_states;      // the run behind that, if next <= list_end
    int32_t next;                             // the run behind that one
};
static_assert(sizeof(UnitRecord) == 64, "one line; fetched by four lanes");

// Stacked query tiles: 128 rows of ALL heads of a KV group, ordered by row and then by head, of rows that see the same keys under
// every head of the group -- text rows, and the other rows of a group whose heads are all Dense.  Their ids follow the M
// tiles of a head: first those of the text rows, then those of the others.
struct StackedTiles {
    struct Unit { int32_t list_begin, list_end, n_tiles; };   // of `ranges`
    struct Kind {
        bool decided = false;
        int32_t n_tiles = 0;              // query tiles; 0: not worth it
        std::vector<Unit> units;          // of two neighbouring tiles, the last one of an odd number alone
        std::vector<PairRange> ranges;
    };
    int32_t gqa_group = 0;                // made for groups of this size; 0: not yet
    Kind text, other;
};

// The same for the kernels.
struct alignas(16) StackedRows {
    int32_t first_tile, n_text_tiles;     // the ids are first_tile + ...
    int32_t n_text_rows, n_other_rows;
    int32_t text_slot0;                   // row records: the others from 0 on, text rows from here on
};

struct PairPlan {
    int32_t gqa_group = 0;  // the plan depends on which heads share a KV head ...
    uint64_t epoch = 0;     // ... and on the class vector (bs_tilemap::class_epoch when it was made)
    std::vector<PairRange> ranges;
    std::vector<PairItem> items;  // eight queues, one per XCD, each heaviest first
    int32_t queue_off[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};   // queue x = items[queue_off[x] .. queue_off[x + 1])
    int32_t back_block = 0;       // dealt there and back in blocks of so many units; 0: in turn
};

// One item of a unit that was cut: its partial results lie in slots first_slot .. first_slot + n_parts - 1.
struct CutItem { int32_t head, tile, first_slot, n_parts_item; };   // n_parts_item: parts << 1 | item of the unit (0 A, 1 B)

// The units of a PairPlan in equal shares, one per workgroup, with units cut along their key tiles where a share
// ends (see bs_plan_shares).
struct SharePlan {
    int32_t gqa_group = 0, n_wgs = 0;     // made for these ...
    uint64_t epoch = 0;                   // ... and for this class vector
    std::vector<PairItem> parts;          // PairItem::classes carries slot + 1 in its upper half for a part of a cut unit
    std::vector<PairRange> ranges;        // the parts' lists
    std::vector<int32_t> share_off;       // workgroup w takes parts[share_off[w] .. share_off[w + 1]); empty: not worth it
    int32_t queue_off[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};   // parts for whoever is done, in eight queues behind the shares
    std::vector<CutItem> cut;
    int32_t n_slots = 0;
};

struct DeviceMap;  // defined by the HIP side

// Whether the pre-pass transposes V for a launch of the bf16 kernel of so many steps, whose units read so many key tiles (of all KV heads).
// If not, V tiles come from where the caller has them and the operand reads transpose: two reads of 64 bits for one of 128, at half the
// rate, so a step takes 0.04-0.055 us longer at d = 128 (2.3 % on 36K tokens), 0.15-0.2 ns with 256 workgroups; V^T costs 32 KB of traffic
// a tile, 6 ns.  The line lies at the tiles' quotient.  Passes of two sparse layers with V^T / V, by steps a tile: 7 (1000 rows behind 99K)
// 1746 / 1654 us, 10 (4.2K tokens, 16 KV heads) 264 / 260, 11 (window of 1024 on 27K) 962 / 947, 12 (1300 rows behind 28K) 436 / 427, 18 (2000
// behind 58K) 1172 / 1149, 25 (3000 behind 37K) 1091 / 1078, 25 (16K, 16 KV heads) 1666 / 1664, 26 (3000 behind 17K) 602 / 602, 27 (window of
// 4096 on 20K) 1359 / 1364, 27 (6K) 407 / 404, 29 (5.3K) 387 / 388, 33 (4000 behind 36K) 1412 / 1396, 34 (6.5K) 527 / 530, 39 (window of 4096 on
// 27K) 1317 / 1329, 60 (11K) 737 / 743, 83 (16K) 1387 / 1408.
// Up to 256 tiles (4 MB of V^T at d = 128) the copy is still in the L2s and costs little beside its launch, which is there either way: 20
// (1.7K, 120 tiles) 107 / 106, 24 (1.7K, 60) 87.3 / 88.3, 24 (2.1K, 148) 122 / 124, 26 (2.6K, 188) 145 / 147, 27 (2.1K, 37) 100.5 / 101.4; but 11 (1.3K,
// 192) 108 / 104, 15 (1.7K, 240) 125 / 119.
// At d = 64 a step, which is bound by the vector ALU and by what stands around it, loses more (4-5 %), and V^T, half as large, is still in
// the caches where it is up to some 32 MB: 1.2 (0.5K, 88 tiles) 69.7 / 70.4, 2.9 (1K, 144) 83.9 / 84.8, 3.6 (2K, 148) 82.9 / 84.1; 1.2 (300 rows
// behind 18K, 2576) 110 / 105, 2.9 (1K, 576) 93.8 / 92.6, 3.0 (2000 rows behind 24K, 3688) 177 / 169; 4.6 (4K, 2336) 178.3 / 180.2, 8.8 (9K,
// 1280) 170 / 173, 30 (9K) 406 / 413; above 4096 tiles 5.6 (1000 rows behind 29K, 4264) 309 / 297, 8.8 (9K, 5120) 475 / 468, 8.7-8.8
// (window of 1024, 4304, 5248 and 7648) 551 / 554, 664 / 664 and 959 / 956, 10.7 (2000 behind 32K, 4808) 557 / 547, 12 (2500 behind 77K)
// 1378 / 1357, 12.5 (16K, 9088) 1128 / 1137, 20 (30K, 17056) 3089 / 3111.
inline bool transposed_values(int32_t head_dim, int64_t steps, int64_t tiles)
{
    const int64_t steps_per_tile = tiles <= 256 ? (head_dim == 128 ? 22 : 0) : head_dim == 128 ? 32 : tiles <= 4096 ? 4 : 10;
    return steps >= steps_per_tile * tiles;
}

// What the query at position i sees apart from its head's class: keys *first .. *last; its image (empty for text).
void row_bounds(const bs_tilemap *tm, int32_t i, int32_t *first, int32_t *last, int32_t *img_lo, int32_t *img_hi);

}  // namespace bs

// Pair up the work items for KV-sharing workgroups (host only; see PairItem).
void bs_plan_pairs(bs_tilemap *tm, int32_t gqa_group);
// The units of the fp32 kernel: every (head, query tile) on its own, heaviest first (host only).
void bs_plan_solo(bs_tilemap *tm);
// Cut the units of the pair plan (of the solo plan if gqa_group is 0) into equal shares for n_wgs workgroups, if that
// pays (host only; see SharePlan).
void bs_plan_shares(bs_tilemap *tm, int32_t gqa_group, int32_t n_wgs);

struct bs_tilemap {
    int32_t L = 0, bm = 0, bn = 0, M = 0, N = 0, n_q_heads = 0;
    // Key tiles: ids [0, N0) are the prompt's keys in position order; with packed keys, ids
    // [N0, N) are compact tiles holding the free keys (text and sink keys) in position order.  The kernels know further
    // compact tiles, ids [text_tile0, n_tiles), with the text keys alone (text_tile0 = n_tiles: none), see build_run_lists.
    int32_t N0 = 0, text_tile0 = 0, n_tiles = 0;
    bool packed = false;
    bool bidir = false;                    // image tokens also attend to the later tokens of their own image
    int32_t window = 0;                    // > 0: sliding window, keys with i - j >= window are masked
    int32_t q_begin = 0;                   // the query rows are positions q_begin .. L - 1 (q / out hold L - q_begin rows per head)
    bool regrouped = false;                // the query rows are not in the natural order
    bs::PromptGeometry geo;
    std::vector<uint8_t> head_class;
    // The published lists and what is counted, made when first asked for (mutex) where the kernels walk lists of their own.
    mutable std::mutex lists_mutex;
    mutable bool counted = false;
    mutable int64_t allowed_pairs[4] = {0, 0, 0, 0}, empty_rows[4] = {0, 0, 0, 0};
    mutable bool intra_compact = false;    // packed: the published lists of Intra-Image take the text keys from the compact tiles
    mutable bs::ClassLists cls[4];
    bs::ClassLists run[4];                 // what the kernels walk instead of cls, if built
    const bs::ClassLists &walked(int c) const { return run[c].row_ptr.empty() ? cls[c] : run[c]; }
    bs::StackedTiles stacked;              // of the bf16 kernel's units; made for a group size when first planned
    uint64_t class_epoch = 1;              // bumped by bs_tilemap_rebind: work units and their device copies are stale
    bs::PairPlan pairs;                    // built on first use for a given gqa_group and class vector
    bs::PairPlan solo;                     // one item per unit; built on first use
    bs::SharePlan shares;
    bs::DeviceMap *dev = nullptr;          // created lazily by bs_tilemap_upload
    void (*dev_free)(bs::DeviceMap *) = nullptr;
};
