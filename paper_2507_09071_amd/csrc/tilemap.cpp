// Host-side tile-map builder: span table + head classes -> per-class, per-query-tile lists of
// key-tile ranges (FULL / PARTIAL), by interval arithmetic on the span geometry.
//
// Mask definition: paper Sec. 3.2 (head classes; text queries see every earlier token; text
// keys stay visible to every class) and Sec. 3.1 (causal prefill).  The lists take the place
// of the paper kernel's sink_end[M] / first_image[M] arrays and its all/any(istext_m) dispatch
// (App. kernel, Notation and Alg. 3): a query tile that holds a text row walks every causal
// key tile, an image-only query tile walks only tiles that hold a text key, an enabled sink
// key, or a key of its own image.
#include <algorithm>
#include <climits>
#include <cstring>
#include <functional>
#include <mutex>
#include <new>

#include "tilemap_internal.h"

namespace {

using bs::ClassLists;
using bs::TileRange;

// Rows [a, b) of the query tile lie in image g (0-based).  [ea, eb): the same rows by the last key
// position they may see (+1 for eb): themselves under the causal mask; with bidirectional images
// every row of image g sees up to the image's last token, as if it were that token's query.
struct Segment { int32_t g, a, b, ea, eb; };

using bs::PromptGeometry;

// What the list builders need on top of the prompt's geometry (per-tile tables, no per-token ones).
struct Geometry : PromptGeometry {
    explicit Geometry(const PromptGeometry &g) : PromptGeometry(g) {}
    explicit Geometry(PromptGeometry &&g) : PromptGeometry(std::move(g)) {}
    // Per key tile, for classes without / with the sink bit; filled on first use.  The lists ask for every (query tile, key
    // tile): from the closed forms alone, a list of 36K tokens with sinks at fixed offsets took 14 ms instead of 4.
    struct FreeTiles {                     // N0 + 1 entries each
        std::vector<int32_t> before;       // free keys (text, or text / sink) in the tiles before n
        std::vector<int32_t> next_any;     // smallest n' >= n with a free key; N0 if none
        std::vector<int32_t> next_all;     // smallest n' >= n that is a complete tile of free keys; N0 if none
    };
    mutable FreeTiles free_tiles[2];
    bool packed = false, intra_compact = false;
    int32_t Nc = 0, text_tile0 = 0;        // text_tile0 > 0: Intra-Image walks the text tiles
    std::vector<int32_t> ctext;            // packed: text keys in the compact tiles before tile c (Nc + 1)
    std::vector<TileRange> ctext_runs;     // runs of complete compact tiles by their text keys: FULL all, PARTIAL some
    std::vector<int32_t> text_tiles_before;   // text_tile0 > 0: prompt tiles with a text key before the first tile of each span

    int32_t lo(int32_t i) const { return window > 0 ? first_visible(i) : 0; }
    const FreeTiles &tiles_of_free(int cls) const
    {
        FreeTiles &t = free_tiles[cls & 1];
        if (t.before.empty()) {
            t.next_any.assign(N0 + 1, N0);
            t.next_all.assign(N0 + 1, N0);
            std::vector<int32_t> before(N0 + 1);
            for (int32_t n = 0; n < N0; ++n) before[n] = free_count(cls, n * bn);
            before[N0] = free_count(cls, L);
            for (int32_t n = N0 - 1; n >= 0; --n) {
                const int32_t free = before[n + 1] - before[n];
                t.next_any[n] = free > 0 ? n : t.next_any[n + 1];
                t.next_all[n] = free == bn ? n : t.next_all[n + 1];
            }
            t.before = std::move(before);
        }
        return t;
    }
    // free keys of a class at positions [a, b) inside key tile n
    int32_t free_in_tile(int cls, int32_t n, int32_t a, int32_t b) const
    {
        if (a == n * bn && b == std::min(a + bn, L)) {
            const FreeTiles &t = tiles_of_free(cls);
            return t.before[n + 1] - t.before[n];
        }
        return free_count(cls, b) - free_count(cls, a);
    }
};

struct QueryTile {
    int32_t r0, r1;       // rows [r0, r1), clipped to L
    int32_t e0, e1;       // last visible key position of the first row, and of the last row + 1 (r0, r1 if causal)
    bool ragged;          // fewer than bm rows
    int32_t last_text;    // last text row inside, or -1
    std::vector<Segment> segs;
};

// Describe rows [r0, r1) of one query tile.  `ragged`: the tile holds fewer than bm rows (then
// no key tile can be FULL: the missing rows count as masked).  A query tile whose rows are
// not contiguous (regrouped order) is described run by run.
void describe_query_rows(const Geometry &G, int32_t r0, int32_t r1, bool ragged, QueryTile &qt)
{
    qt.r0 = r0;
    qt.r1 = r1;
    qt.ragged = ragged;
    int32_t lt = G.last_text(qt.r1 - 1);
    qt.last_text = (lt >= qt.r0) ? lt : -1;
    qt.segs.clear();
    const bs::SpanInfo *sp = G.spans.data();
    for (int32_t g = G.span_at(qt.r0); g < G.n_spans && sp[g].start < qt.r1; ++g) {
        const int32_t a = std::max(sp[g].start, qt.r0), b = std::min(sp[g].end, qt.r1);
        qt.segs.push_back({g, a, b, G.bidir ? sp[g].end - 1 : a, G.bidir ? sp[g].end : b});
    }
    // the visible range grows with the row position, so the first / last row bound the tile
    qt.e0 = (!qt.segs.empty() && qt.segs.front().a == qt.r0) ? qt.segs.front().ea : qt.r0;
    qt.e1 = (!qt.segs.empty() && qt.segs.back().b == qt.r1) ? qt.segs.back().eb : qt.r1;
}

// Exact state of tile (query tile qt, key tile n) for class cls: 0 skip, 1 partial, 2 full.
int tile_state(const Geometry &G, const QueryTile &qt, int cls, int32_t n)
{
    const int32_t c0 = n * G.bn, c1 = std::min(c0 + G.bn, G.L);
    if (c0 > qt.e1 - 1) return 0;  // beyond what the last row sees
    if (c1 - 1 < G.lo(qt.r0)) return 0;  // before the first row's window (and every later row's)
    const bs::SpanInfo *sp = G.spans.data();

    // Every row i sees the keys of its class pattern inside [lo(i), e(i)]; both ends grow with i, so
    // the rows of a run together see [lo(first), e(last)] and share [lo(last), e(first)].
    bool any = false;
    if (cls == BS_DENSE || qt.segs.empty()) {
        any = true;
    } else {
        // a text row at or after the tile's first key, close enough to see the tile's last key
        if (qt.last_text >= c0) {
            const int32_t t = G.next_text(std::max(qt.r0, c0));
            if (t < qt.r1 && G.lo(t) <= c1 - 1) any = true;
        }
        for (const Segment &s : qt.segs) {
            if (any) break;
            const int32_t lo = std::max(c0, G.lo(s.a)), hi = std::min(c1, s.eb);  // keys the segment's rows may see
            if (hi <= lo) continue;
            if (G.free_in_tile(cls, n, lo, hi) > 0) { any = true; break; }
            if (cls & 2) {
                int32_t lo2 = std::max(lo, sp[s.g].start), hi2 = std::min(hi, sp[s.g].end);
                if (hi2 > lo2) { any = true; break; }
            }
        }
    }
    if (!any) return 0;

    bool all;
    if (qt.ragged || (c1 - c0) < G.bn || c1 - 1 > qt.e0 || c0 < G.lo(qt.r1 - 1)) {
        all = false;  // masked out-of-range positions, or the diagonal / the window's edge cuts through
    } else if (cls == BS_DENSE || qt.segs.empty()) {
        all = true;
    } else {
        int32_t nonfree = G.bn - G.free_in_tile(cls, n, c0, c1);
        if (nonfree == 0) {
            all = true;
        } else if (!(cls & 2) || qt.segs.size() > 1) {
            all = false;  // a masked image key, or two images that cannot both own it
        } else {
            const bs::SpanInfo &own = sp[qt.segs[0].g];
            int32_t lo2 = std::max(c0, own.start), hi2 = std::min(c1, own.end);
            int32_t nonfree_own = (hi2 > lo2) ? (hi2 - lo2) - G.free_in_tile(cls, n, lo2, hi2) : 0;
            all = (nonfree_own == nonfree);
        }
    }
    return all ? 2 : 1;
}

// Key tiles that can hold an allowed pair for this query tile (a superset is fine; sorted, unique).
void candidate_tiles(const Geometry &G, const QueryTile &qt, int cls, std::vector<int32_t> &cand)
{
    cand.clear();
    const int32_t n_last = (qt.e1 - 1) / G.bn;
    if (cls == BS_DENSE || qt.last_text >= 0) {
        cand.resize(n_last + 1);
        for (int32_t n = 0; n <= n_last; ++n) cand[n] = n;
        return;
    }
    // image-only query tile of a sparse class: tiles with a free key (text / enabled sink) ...
    const std::vector<int32_t> &next = G.tiles_of_free(cls).next_any;
    for (int32_t n = next[0]; n <= n_last; n = next[n + 1])
        if (n < n_last || G.next_free(cls, n * G.bn) < qt.e1) cand.push_back(n);   // (the last tile may go on behind the rows)
    // ... and tiles overlapping the part of an own image that lies at or before the tile's rows
    if (cls & 2) {
        const bs::SpanInfo *sp = G.spans.data();
        for (const Segment &s : qt.segs)
            for (int32_t n = sp[s.g].start / G.bn; n <= (s.eb - 1) / G.bn; ++n) cand.push_back(n);
        std::sort(cand.begin(), cand.end());
        cand.erase(std::unique(cand.begin(), cand.end()), cand.end());
    }
}

// Key-tile ranges (FULL / PARTIAL; skipped tiles are absent) of one run of contiguous query rows.
void build_run(const Geometry &G, int cls, const QueryTile &qt, std::vector<int32_t> &cand,
               std::vector<TileRange> &out)
{
    out.clear();
    int32_t run_begin = -1, run_end = -1, run_state = 0;
    auto flush = [&]() {
        if (run_begin >= 0) out.push_back({run_begin, (run_end << 1) | (run_state == 2)});
        run_begin = -1;
    };
    // append tiles [b, e) of one state (1 partial, 2 full), merging adjacent runs
    auto emit = [&](int32_t b, int32_t e, int st) {
        if (e <= b) return;
        if (run_begin >= 0 && b == run_end && st == run_state) {
            run_end = e;
        } else {
            flush();
            run_begin = b; run_end = e; run_state = st;
        }
    };
    const int32_t n_last = (qt.e1 - 1) / G.bn;
    // key tiles wholly within what the first row of a complete query tile sees can be FULL
    const int32_t n_full_limit = qt.ragged ? 0 : (qt.e0 + 1) / G.bn;

    if (G.window > 0) {
        // sliding window: few key tiles per query tile, each classified exactly
        for (int32_t n = G.lo(qt.r0) / G.bn; n <= n_last; ++n) {
            const int st = tile_state(G, qt, cls, n);
            if (st) emit(n, n + 1, st);
        }
    } else if (cls == BS_DENSE || qt.segs.empty()) {
        // every earlier key is visible: FULL below the diagonal, PARTIAL on it
        emit(0, n_full_limit, 2);
        emit(n_full_limit, n_last + 1, 1);
    } else if (qt.last_text >= 0) {
        // mixed text/image rows: every causal key tile up to the last text row is visited.
        // Only a few of them can differ from PARTIAL: all-free tiles and tiles overlapping an
        // own image (candidates for FULL), and the tiles past the last text row (may be SKIP).
        // Those are classified exactly; the rest are PARTIAL.
        cand.clear();
        const std::vector<int32_t> &naf = G.tiles_of_free(cls).next_all;
        for (int32_t n = naf[0]; n < n_full_limit; n = naf[n + 1]) cand.push_back(n);
        const bs::SpanInfo *sp = G.spans.data();
        for (const Segment &sg : qt.segs)
            for (int32_t n = sp[sg.g].start / G.bn; n <= (sg.eb - 1) / G.bn && n < n_full_limit; ++n) cand.push_back(n);
        for (int32_t n = qt.last_text / G.bn + 1; n <= n_last; ++n) cand.push_back(n);
        std::sort(cand.begin(), cand.end());
        cand.erase(std::unique(cand.begin(), cand.end()), cand.end());
        int32_t cur = 0;
        for (int32_t n : cand) {
            emit(cur, n, 1);
            const int st = tile_state(G, qt, cls, n);
            if (st) emit(n, n + 1, st);
            cur = n + 1;
        }
        emit(cur, qt.last_text / G.bn + 1, 1);
    } else {
        candidate_tiles(G, qt, cls, cand);
        for (int32_t n : cand) {
            const int st = tile_state(G, qt, cls, n);
            if (st) emit(n, n + 1, st);
        }
    }
    flush();
}

// Range list of a sparse class for the rows of a segment, all inside one image, that take the keys outside their own
// image from compact tiles.  Two parts, disjoint by construction:
//   own-image keys (classes with the intra bit): the prompt's own tiles; a pair (i, j) counts there iff
//     j is in the image and visible to i;
//   the others: compact tiles, of which row i sees the slots
//       Sink:             of the free keys up to its last visible position
//       Intra-Image:      of the text keys before its image (in the text tiles, or mixed with sinks in the free tiles)
//       Intra-Image+Sink: of the free keys before its image (the image's own are counted above)
//     from the first position in its window on.
void build_run_packed(const Geometry &G, int cls, const Segment &s, bool ragged, std::vector<TileRange> &out)
{
    out.clear();
    int32_t run_begin = -1, run_end = -1, run_state = 0;
    auto flush = [&]() {
        if (run_begin >= 0) out.push_back({run_begin, (run_end << 1) | (run_state == 2)});
        run_begin = -1;
    };
    auto emit = [&](int32_t bg, int32_t en, int st) {
        if (en <= bg || st == 0) return;
        if (run_begin >= 0 && bg == run_end && st == run_state) {
            run_end = en;
        } else {
            flush();
            run_begin = bg; run_end = en; run_state = st;
        }
    };
    // tiles of consecutive keys of which the rows together see [lo, hi), all of them [all_lo, all_hi)
    auto emit_keys = [&](int32_t tile0, int32_t lo, int32_t all_lo, int32_t all_hi, int32_t hi) {
        if (hi <= lo) return;
        const int32_t n0 = lo / G.bn, n1 = (hi - 1) / G.bn + 1;
        const int32_t f0 = std::min(n1, (all_lo + G.bn - 1) / G.bn);
        const int32_t f1 = ragged ? f0 : std::max(f0, std::min(n1, all_hi / G.bn));
        emit(tile0 + n0, tile0 + f0, 1);
        emit(tile0 + f0, tile0 + f1, 2);
        emit(tile0 + f1, tile0 + n1, 1);
    };
    const bs::SpanInfo &own = G.spans[s.g];
    const int32_t lo = G.lo(s.a), all_lo = G.lo(s.b - 1);   // first visible position of the first / last row
    if (cls & 2) emit_keys(0, std::max(own.start, lo), std::max(own.start, all_lo), s.ea + 1, s.eb);
    if (cls == BS_SINK) {
        emit_keys(G.N0, G.n_free(lo), G.n_free(all_lo), G.n_free(s.ea + 1), G.n_free(s.eb));
    } else if (cls == BS_INTRA_SINK) {
        emit_keys(G.N0, G.n_free(lo), G.n_free(all_lo), own.free_before, own.free_before);
    } else if (G.text_tile0 > 0) {
        emit_keys(G.text_tile0, G.n_text(lo), G.n_text(all_lo), own.text_before, own.text_before);
    } else {
        const int32_t fb = own.free_before, c_all = ragged ? 0 : fb / G.bn;
        for (const TileRange &r : G.ctext_runs) {
            if (r.begin >= c_all) break;
            emit(G.N0 + r.begin, G.N0 + std::min(r.end(), c_all), r.full() ? 2 : 1);
        }
        for (int32_t c = c_all; c * G.bn < fb; ++c) {   // (the free keys before the image: the text before it counts)
            const int32_t text = ((c + 1) * G.bn <= fb ? G.ctext[c + 1] : own.text_before) - G.ctext[c];
            emit(G.N0 + c, G.N0 + c + 1, text > 0 ? 1 : 0);
        }
    }
    flush();
}

// Union of two range lists of one query tile's runs.  A key tile is FULL for the tile only if
// it is FULL for every run; visited by some run and not FULL for all of them: PARTIAL.
// `a_runs` tells how many runs list a stands for (a tile absent from a is skipped by all of them).
void combine_runs(const std::vector<TileRange> &a, const std::vector<TileRange> &b, std::vector<TileRange> &out)
{
    out.clear();
    size_t ia = 0, ib = 0;
    int32_t pos = 0;
    auto push = [&](int32_t bg, int32_t en, bool full) {
        if (en <= bg) return;
        if (!out.empty() && out.back().end() == bg && out.back().full() == full) out.back().end_state = (en << 1) | full;
        else out.push_back({bg, (en << 1) | (int32_t)full});
    };
    while (ia < a.size() || ib < b.size()) {
        // state of a and b at `pos` and the next boundary
        int32_t next = INT32_MAX;
        int sa = 0, sb = 0;
        if (ia < a.size()) {
            if (a[ia].end() <= pos) { ++ia; continue; }
            if (a[ia].begin <= pos) { sa = a[ia].full() ? 2 : 1; next = std::min(next, a[ia].end()); }
            else next = std::min(next, a[ia].begin);
        }
        if (ib < b.size()) {
            if (b[ib].end() <= pos) { ++ib; continue; }
            if (b[ib].begin <= pos) { sb = b[ib].full() ? 2 : 1; next = std::min(next, b[ib].end()); }
            else next = std::min(next, b[ib].begin);
        }
        if (next == INT32_MAX) break;
        if (sa || sb) push(pos, next, sa == 2 && sb == 2);
        pos = next;
    }
}

// Do the text tiles hold the text keys that these image rows of Intra-Image heads see in no more tiles than the prompt's own,
// not counting those of their own images?  (Text tiles are FULL but for the last, so they win a tie.)
bool text_tiles_pay(const Geometry &G, const std::vector<std::pair<int32_t, int32_t>> &runs)
{
    const int32_t last = G.span_at(runs.back().second - 1);
    return (G.spans[last].text_before + G.bn - 1) / G.bn <= G.text_tiles_before[last];
}

// `sample`: only every so many query tiles, for what they cost: returns (cost) of them, without and with compact tiles.
struct ListCosts { int64_t plain = 0, compact = 0; };
ListCosts build_class(const Geometry &G, int cls, ClassLists &out, int32_t sample = 0)
{
    ListCosts costs;
    out.row_ptr.assign(G.M + 1, 0);
    out.row_tiles.assign(G.M, 0);
    out.compact.assign(G.M, 0);
    out.ranges.clear();
    for (auto &s : out.span) s = {};
    QueryTile qt;
    std::vector<int32_t> cand;
    std::vector<TileRange> run, seg_run, acc, tmp;
    std::vector<std::pair<int32_t, int32_t>> runs;
    // the list of a query tile whose rows are `runs`, to `acc`
    auto build_tile = [&](bool ragged, bool compact) {
        acc.clear();
        bool first = true;
        for (const auto &rr : runs) {
            describe_query_rows(G, rr.first, rr.second, ragged, qt);
            if (compact && qt.last_text < 0 && !qt.segs.empty()) {
                // image rows of a sparse class: one packed list per image the run touches
                // (two images can be adjacent without a text token between them)
                bool first_seg = true;
                for (const Segment &sg : qt.segs) {
                    build_run_packed(G, cls, sg, ragged, first_seg ? run : seg_run);
                    if (!first_seg) {
                        combine_runs(run, seg_run, tmp);
                        run.swap(tmp);
                    }
                    first_seg = false;
                }
            } else {
                build_run(G, cls, qt, cand, run);
            }
            if (first) {
                acc.swap(run);
                first = false;
            } else {
                combine_runs(acc, run, tmp);
                acc.swap(tmp);
            }
        }
    };
    // (a PARTIAL tile takes an eighth longer than a FULL one)
    auto cost = [](const std::vector<TileRange> &list) {
        int64_t c = 0;
        for (const TileRange &r : list) c += (int64_t)(r.end() - r.begin) * (r.full() ? 8 : 9);
        return c;
    };
    for (int32_t m = 0; m < G.M; ++m) {
        // the tile's rows as runs of consecutive positions (one run in the natural order)
        const bool ragged = G.tile_runs(m, runs) < G.bm;
        // (the rows of a map with compact tiles are regrouped: all of a tile are image rows, or none)
        bool compact = G.packed && cls != BS_DENSE;
        if (cls == BS_INTRA && G.window == 0) compact = compact && (G.text_tile0 > 0 ? text_tiles_pay(G, runs) : G.intra_compact);
        for (int pass = sample > 0 ? 0 : 1; pass < 2; ++pass) {
            build_tile(ragged, pass == 1 && compact);
            if (sample > 0) (pass == 0 ? costs.plain : costs.compact) += cost(acc);
        }
        if (sample > 0) {
            m += sample - 1;
            continue;
        }
        out.compact[m] = compact;
        for (const TileRange &r : acc) {
            const int32_t len = r.end() - r.begin;
            out.row_tiles[m] += len;
            if (r.full()) out.full += len; else out.partial += len;
            out.ranges.push_back(r);
        }
        if (!acc.empty()) {
            auto add = [&](int kind, int32_t b, int32_t e) {
                auto &s = out.span[kind];
                s.first = s.end == 0 ? b : std::min(s.first, b);
                s.end = std::max(s.end, e);
            };
            if (acc.back().end() <= G.N0) {
                add(0, acc.front().begin, acc.back().end());
            } else {   // (a run of tiles may go on from one kind into the next)
                const int32_t edge[4] = {0, G.N0, G.text_tile0 > 0 ? G.text_tile0 : INT32_MAX, INT32_MAX};
                for (const TileRange &r : acc)
                    for (int kind = 0; kind < 3; ++kind)
                        if (std::max(r.begin, edge[kind]) < std::min(r.end(), edge[kind + 1]))
                            add(kind, std::max(r.begin, edge[kind]), std::min(r.end(), edge[kind + 1]));
            }
        }
        out.row_ptr[m + 1] = (int64_t)out.ranges.size();
    }
    out.visited = out.full + out.partial;
    return costs;
}

// Allowed pairs and empty rows per class, from prefix counts (no pair enumeration).
void count_pairs(const PromptGeometry &G, int64_t allowed_pairs[4], int64_t empty_rows[4])
{
    int64_t pairs[4] = {0, 0, 0, 0}, empty[4] = {0, 0, 0, 0};
    for (int32_t i = G.q_begin, g = G.span_at(i); i < G.L; ++i) {
        while (g < G.n_spans && G.spans[g].end <= i) ++g;
        const bool image = g < G.n_spans && G.spans[g].start <= i;
        const int32_t lo = G.window > 0 ? G.first_visible(i) : 0;   // first key position the row may see
        if (!image) {
            for (int c = 0; c < 4; ++c) pairs[c] += i + 1 - lo;
            continue;
        }
        const bs::SpanInfo &sp = G.spans[g];
        const int32_t e = G.bidir ? sp.end - 1 : i;   // last key position the row may see
        const int32_t s0 = std::max(sp.start, lo);    // first own-image key it may see
        const int64_t text = sp.text_before - G.n_text(lo);
        const int64_t free = sp.free_before + G.sinks_in(g, e + 1 - sp.start) - G.n_free(lo);   // text or sink, in [lo, e]
        const int64_t own = e - s0 + 1;
        const int64_t own_sink = G.sinks_in(g, e + 1 - sp.start) - G.sinks_in(g, s0 - sp.start);
        const int64_t row[4] = {e + 1 - lo, free, text + own, free + own - own_sink};
        for (int c = 0; c < 4; ++c) {
            pairs[c] += row[c];
            if (row[c] == 0) ++empty[c];
        }
    }
    for (int c = 0; c < 4; ++c) { allowed_pairs[c] = pairs[c]; empty_rows[c] = empty[c]; }
}

// The lists that the map publishes for class c (lists_mutex held, or the map not handed out yet).  G: of the map's prompt.
void build_published(const bs_tilemap *tm, Geometry &G, int c)
{
    const PromptGeometry &P = G;
    const int32_t block_n = P.bn, L = P.L, n_spans = P.n_spans;
    G.packed = tm->packed;
    if (!tm->packed || c != BS_INTRA) {
        build_class(G, c, tm->cls[c]);
        return;
    }
    G.Nc = tm->N - tm->N0;
    // text keys before every compact tile
    G.ctext.assign(G.Nc + 1, 0);
    for (int32_t t = 0; t < G.Nc; ++t) G.ctext[t] = P.n_text(P.free_position(t * block_n));
    G.ctext[G.Nc] = P.n_text(L);
    for (int32_t t = 0; t < G.Nc; ++t) {
        const int32_t text = G.ctext[t + 1] - G.ctext[t];
        const bool full = text == block_n;
        if (text == 0) continue;
        if (!G.ctext_runs.empty() && G.ctext_runs.back().end() == t && G.ctext_runs.back().full() == full)
            G.ctext_runs.back().end_state = ((t + 1) << 1) | (int32_t)full;
        else
            G.ctext_runs.push_back({t, ((t + 1) << 1) | (int32_t)full});
    }
    // Intra-Image rows need the text keys only.  Among the compact tiles they are mixed
    // with the sink keys; where text is rare (a few long images) the prompt's own tiles
    // hold it in fewer tiles.  Both lists are exact, so the choice is a matter of cost
    // only: count, for the last row of every image, the tiles with a text key either
    // way (prefix counts over the two tile spaces) and take the smaller total; a close
    // call is settled below by building both.
    std::vector<int32_t> compact_tiles(G.Nc + 1, 0);
    for (int32_t t = 0; t < G.Nc; ++t) compact_tiles[t + 1] = compact_tiles[t] + (G.ctext[t + 1] > G.ctext[t]);
    int64_t cost_prompt = 0, cost_compact = 0;
    int32_t text_tiles = 0, counted = 0, text_from = 0;   // prompt tiles with a text key before tile `counted`
    for (int32_t g = 0; g < n_spans; ++g) {
        const bs::SpanInfo &s = P.spans[g];
        if (s.start > text_from) {                         // the text before image g
            const int32_t n0 = std::max(counted, text_from / block_n), n1 = (s.start - 1) / block_n + 1;
            text_tiles += std::max(0, n1 - n0);
            counted = std::max(counted, n1);
        }
        text_from = s.end;
        // (the tile of the image's last token counts if it holds a text key behind the image)
        const int32_t n_last = (s.end - 1) / block_n;
        const bool tail = n_last >= counted && P.n_text(std::min((n_last + 1) * block_n, L)) > P.n_text(s.end);
        const int64_t rows = s.end - s.start;
        cost_prompt += rows * (text_tiles + tail);
        cost_compact += rows * compact_tiles[(s.free_before + P.sinks_in(g, s.end - s.start) + block_n - 1) / block_n];
    }
    G.intra_compact = cost_compact < cost_prompt;
    build_class(G, c, tm->cls[c]);
    if (cost_compact * 4 >= cost_prompt * 3 && cost_prompt * 4 >= cost_compact * 3) {
        // the estimate is within a quarter: build the other variant as well and keep the shorter list
        ClassLists alt;
        G.intra_compact = !G.intra_compact;
        build_class(G, c, alt);
        if (alt.visited < tm->cls[c].visited) tm->cls[c] = std::move(alt);
        else G.intra_compact = !G.intra_compact;
    }
    tm->intra_compact = G.intra_compact;
}

// The published lists of class c; made now if nobody has asked for them yet.
const ClassLists &published(const bs_tilemap *tm, int c)
{
    std::lock_guard<std::mutex> lock(tm->lists_mutex);
    if (tm->cls[c].row_ptr.empty()) {
        try {
            Geometry G(tm->geo);
            build_published(tm, G, c);
        } catch (...) {
            tm->cls[c] = ClassLists();
            throw;
        }
    }
    return tm->cls[c];
}

// Lists of the kernels' own, where further compact tiles make them shorter than the published ones.
// Intra-Image rows see the text keys and their own image.  The map's compact tiles mix the text with the sinks, which are more
// (a tenth of every image): in tiles of their own the text keys of a long prompt are a fraction of that, and all but the
// last of them FULL.  302K tokens, 1100 images of 256, 26 sinks and 18 text tokens each: 155 text tiles instead of 380
// mixed ones on average, a layer takes 185.9 ms (208.1 with the mixed ones); 16K tokens characterised, images of 1-4K: 3253 us
// (3319, from the prompt's own tiles).  The kernels' tiles number at most half of the prompt's more than the published ones, so that the
// static scratch, sized by these, holds all if K is read in place; with more text than that the class is nearly dense.
//
// In a window the map publishes no compact tiles, but a row of a sparse class sees as small a part of the window's tiles as it
// does of a prompt's (a sixth of the pairs under Sink, a third under Intra-Image+Sink with images of 256), so the kernels know
// both kinds, and the lists are cut at both ends.  A class that saves less than a thirtieth of its steps that way, by some
// four of its query tiles, keeps the published lists: packing the compact tiles costs about that (images of 1-5K, window
// of 512: 1036 us with them, 1032 without).  Images of more than twice the window are not looked at: their rows see
// little but their own image, and looking costs host time (10 us of a call of 127 us).
// Three layers, 27K tokens, images of 256: window of 512 1487 -> 1373 us, 1024 1979 -> 1679, 4096 4667 -> 3289; d = 64, 1024:
// 1342 -> 1097; fp32, 6K tokens: 2998 -> 2339.
void build_run_lists(bs_tilemap *tm, Geometry &G)
{
    const PromptGeometry &P = G;
    G.packed = true;
    G.text_tile0 = tm->text_tile0 < tm->n_tiles ? tm->text_tile0 : 0;
    if (P.window > 0) {
        for (int c : {BS_SINK, BS_INTRA, BS_INTRA_SINK}) {
            if (c == BS_INTRA && G.text_tile0 == 0) continue;
            const ListCosts costs = build_class(G, c, tm->run[c], std::max(1, (P.regrouped ? P.m_img : P.M) / 4));
            tm->run[c] = ClassLists();
            if (costs.compact < costs.plain - costs.plain / 30) build_class(G, c, tm->run[c]);
        }
        return;
    }
    G.text_tiles_before.resize((size_t)P.n_spans + 1);
    int32_t text_tiles = 0, counted = 0, text_from = 0;   // prompt tiles with a text key before tile `counted`
    for (int32_t g = 0; g <= P.n_spans; ++g) {
        const bs::SpanInfo &s = P.spans[g];
        if (s.start > text_from) {
            const int32_t n0 = std::max(counted, text_from / P.bn), n1 = (s.start - 1) / P.bn + 1;
            text_tiles += std::max(0, n1 - n0);
            counted = std::max(counted, n1);
        }
        text_from = s.end;
        G.text_tiles_before[g] = text_tiles - (counted > s.start / P.bn);
    }
    build_class(G, BS_INTRA, tm->run[BS_INTRA]);
}

// The state of every key tile for query tile m: 0 skip, 1 partial, 2 full.
void expand_states(const ClassLists &cl, int32_t m, std::vector<uint8_t> &states)
{
    std::fill(states.begin(), states.end(), 0);
    for (int64_t p = cl.row_ptr[m]; p < cl.row_ptr[m + 1]; ++p)
        for (int32_t n = cl.ranges[p].begin; n < cl.ranges[p].end(); ++n) states[n] = cl.ranges[p].full() ? 2 : 1;
}

bool spans_valid(const bs_span *spans, int32_t n, int32_t L)
{
    int32_t prev_end = 0;
    for (int32_t g = 0; g < n; ++g) {
        const bs_span &s = spans[g];
        if (s.start < prev_end || s.end <= s.start || s.end > L) return false;
        if (s.sink < 0 || s.sink > s.end - s.start) return false;
        prev_end = s.end;
    }
    return true;
}

}  // namespace

extern "C" int bs_build_tilemap(const bs_span *spans, int32_t n_spans, int32_t seq_len,
                                const uint8_t *head_class, int32_t n_q_heads, int32_t sink_len,
                                int32_t block_m, int32_t block_n, bs_tilemap **out)
{
    return bs_build_tilemap_ex(spans, n_spans, seq_len, head_class, n_q_heads, sink_len, block_m, block_n, 0, out);
}

extern "C" int bs_build_tilemap_ex(const bs_span *spans, int32_t n_spans, int32_t seq_len,
                                   const uint8_t *head_class, int32_t n_q_heads, int32_t sink_len,
                                   int32_t block_m, int32_t block_n, uint32_t flags, bs_tilemap **out)
{
    return bs_build_tilemap_model(spans, n_spans, seq_len, head_class, n_q_heads, sink_len, block_m, block_n, flags,
                                  nullptr, 0, 0, out);
}

extern "C" int bs_build_tilemap_model(const bs_span *spans, int32_t n_spans, int32_t seq_len,
                                      const uint8_t *head_class, int32_t n_q_heads, int32_t sink_len,
                                      int32_t block_m, int32_t block_n, uint32_t flags,
                                      const int32_t *sink_offsets, int32_t n_sink_offsets, int32_t window,
                                      bs_tilemap **out)
{
    return bs_build_tilemap_suffix(spans, n_spans, seq_len, head_class, n_q_heads, sink_len, block_m, block_n, flags,
                                   sink_offsets, n_sink_offsets, window, 0, out);
}

extern "C" int bs_build_tilemap_suffix(const bs_span *spans, int32_t n_spans, int32_t seq_len,
                                       const uint8_t *head_class, int32_t n_q_heads, int32_t sink_len,
                                       int32_t block_m, int32_t block_n, uint32_t flags,
                                       const int32_t *sink_offsets, int32_t n_sink_offsets, int32_t window,
                                       int32_t q_begin, bs_tilemap **out)
{
    if (q_begin < 0 || (seq_len > 0 && q_begin >= seq_len)) return BS_EINVAL;
    if (flags & ~(uint32_t)(BS_MAP_REGROUP_ROWS | BS_MAP_PACK_KEYS | BS_MAP_BIDIR_IMAGES)) return BS_EINVAL;
    if (window < 0) return BS_EINVAL;
    if (window >= seq_len) window = 0;   // every earlier key is inside the window
    const bool pack_window = window > 0 && (flags & BS_MAP_PACK_KEYS);
    // a map with a window publishes no compact tiles, the kernels know some (build_run_lists); the rows are regrouped
    if (pack_window) flags = (flags & ~(uint32_t)BS_MAP_PACK_KEYS) | BS_MAP_REGROUP_ROWS;
    if (n_sink_offsets < 0 || (n_sink_offsets > 0 && !sink_offsets)) return BS_EINVAL;
    for (int32_t o = 0; o < n_sink_offsets; ++o)
        if (sink_offsets[o] < 0) return BS_EINVAL;
    if (flags & BS_MAP_PACK_KEYS) flags |= BS_MAP_REGROUP_ROWS;   // packed lists exist for image-only query tiles
    if (!out || !head_class || n_q_heads <= 0 || seq_len <= 0 || n_spans < 0) return BS_EINVAL;
    if (n_spans > 0 && !spans) return BS_EINVAL;
    if (sink_len < 0 || sink_len > seq_len || block_m <= 0 || block_n <= 0) return BS_EINVAL;
    if ((int64_t)n_spans >= (int64_t)bs::kMaxSpans) return BS_EINVAL;
    for (int32_t h = 0; h < n_q_heads; ++h)
        if (head_class[h] > 3) return BS_EINVAL;
    if (!spans_valid(spans, n_spans, seq_len)) return BS_EINVAL;

    bs_tilemap *tm = nullptr;
    try {
        tm = new bs_tilemap();
        const int32_t L = seq_len;
        tm->L = L; tm->bm = block_m; tm->bn = block_n;
        tm->q_begin = q_begin;
        tm->N0 = tm->N = (L + block_n - 1) / block_n;
        tm->n_q_heads = n_q_heads;
        tm->head_class.assign(head_class, head_class + n_q_heads);
        tm->bidir = (flags & BS_MAP_BIDIR_IMAGES) != 0 && n_spans > 0;
        tm->window = window;
        bs::PromptGeometry &P = tm->geo;
        P.init(spans, n_spans, L, sink_len, sink_offsets, n_sink_offsets);
        P.bm = block_m; P.bn = block_n; P.N0 = tm->N0;
        P.bidir = tm->bidir; P.window = window; P.q_begin = q_begin;

        // Key tiles: the prompt's keys in position order, then (packed) compact tiles with the
        // free keys -- text keys and sink keys, what an image query of a sparse class may see
        // outside its own image -- in position order.  The paper's kernel permutes K / V so that
        // these keys are contiguous (App. kernel, "Attention Sink Subroutine"); here they are a
        // second copy, because text queries and Dense heads keep walking the original order.
        const int32_t n_free = P.n_free(L);
        if ((flags & BS_MAP_PACK_KEYS) && n_spans > 0 && n_free > 0 && n_free < L) {
            tm->packed = true;
            tm->N = tm->N0 + (int32_t)(((int64_t)n_free + block_n - 1) / block_n);
        }

        // Order of the query rows.  Natural: tile m holds rows m*bm ... .  Regrouped: the image
        // rows first, then the text rows, each group in position order and padded to whole
        // tiles.  A text row attends to every earlier token, so a tile that holds even one
        // walks every causal key tile for every class; gathered into tiles of their own, the
        // text rows stop costing the image rows of the sparse classes their skipped tiles.
        {
            const int32_t n_txt = P.n_text(L) - P.n_text(q_begin), n_img = L - q_begin - n_txt;
            auto tiles = [&](int32_t rows) { return (int32_t)(((int64_t)rows + block_m - 1) / block_m); };   // (any block_m fits)
            if ((flags & BS_MAP_REGROUP_ROWS) && n_txt > 0 && n_img > 0) {   // else nothing to separate
                P.regrouped = tm->regrouped = true;
                P.n_img_rows = n_img;
                P.m_img = tiles(n_img);
                tm->M = P.m_img + tiles(n_txt);
            } else {
                tm->M = tiles(L - q_begin);
            }
        }

        P.M = tm->M;
        tm->n_tiles = tm->text_tile0 = tm->N;
        // compact tiles that the map does not publish, at most half of the prompt's (see build_run_lists)
        const int64_t n_text_tiles = ((int64_t)P.n_text(L) + block_n - 1) / block_n, n_free_tiles = ((int64_t)n_free + block_n - 1) / block_n;
        const bool long_images = (int64_t)(L - P.n_text(L)) > (int64_t)2 * window * n_spans;
        if (pack_window && !long_images && n_spans > 0 && n_free > 0 && n_free < L && 2 * n_free_tiles + 1 <= tm->N0)
            tm->n_tiles = tm->text_tile0 = tm->N0 + (int32_t)n_free_tiles;
        if (tm->N0 < tm->n_tiles && n_text_tiles > 0 && 2 * (n_text_tiles + tm->n_tiles - tm->N) + 1 <= tm->N0)
            tm->n_tiles += (int32_t)n_text_tiles;
        Geometry G(std::move(P));   // (one for all lists: they share its tables; the prompt's geometry goes back to the map below)
        if (tm->N < tm->n_tiles) {
            build_run_lists(tm, G);
            // tiles that none of them walks are not there: every one that is has its room in the workspace of a call
            bool walked[3] = {false, false, false};
            for (const ClassLists &cl : tm->run)
                for (int kind = 1; kind < 3; ++kind) walked[kind] |= cl.span[kind].end > 0;
            if (!walked[2]) tm->n_tiles = tm->text_tile0;
            if (!walked[1] && !walked[2]) tm->n_tiles = tm->text_tile0 = tm->N;
        }
        G.text_tile0 = 0;
        for (int c = 0; c < 4; ++c)
            if (tm->run[c].row_ptr.empty()) build_published(tm, G, c);
        P = std::move(static_cast<PromptGeometry &>(G));
    } catch (const std::bad_alloc &) {
        delete tm;
        return BS_ENOMEM;
    }
    *out = tm;
    return BS_OK;
}

void bs::PromptGeometry::init(const bs_span *sp, int32_t n, int32_t seq_len, int32_t sink_prefix, const int32_t *offs, int32_t n_offs)
{
    L = seq_len;
    n_spans = n;
    sink_len = sink_prefix;
    offsets.assign(offs, offs + n_offs);
    std::sort(offsets.begin(), offsets.end());
    offsets.erase(std::unique(offsets.begin(), offsets.end()), offsets.end());
    spans.resize((size_t)n + 1);
    int32_t text = 0, free = 0, pos = 0, last = -1;   // of everything before `pos`
    for (int32_t g = 0; g < n; ++g) {
        if (sp[g].start > pos) last = sp[g].start - 1;
        text += sp[g].start - pos;
        free += sp[g].start - pos;
        const int32_t len = sp[g].end - sp[g].start;
        spans[g] = {sp[g].start, sp[g].end, std::max(sp[g].sink, std::min(len, std::max(0, sink_len - sp[g].start))), text, free, last, L, 0};
        free += sinks_in(g, len);
        pos = sp[g].end;
    }
    if (L > pos) last = L - 1;
    spans[n] = {L, INT32_MAX, 0, text + L - pos, free + L - pos, last, L, 0};   // sentinel behind the last token
    for (int32_t g = n - 1; g >= 0; --g)
        spans[g].next_text = spans[g].end < spans[g + 1].start ? spans[g].end : (g + 1 < n ? spans[g + 1].next_text : L);
    block_first.resize((size_t)(L >> 6) + 1);
    for (int32_t b = 0, g = 0; b < (int32_t)block_first.size(); ++b) {
        while (g < n && spans[g].end <= b << 6) ++g;
        block_first[b] = g;
    }
}

int32_t bs::PromptGeometry::next_free(int cls, int32_t t) const
{
    if (!(cls & 1)) return next_text(t);
    for (int32_t g = span_at(t); g < n_spans; ++g) {
        const SpanInfo &s = spans[g];
        if (t < s.start) return t;                      // text
        const int32_t o = t - s.start;
        if (o < s.prefix) return t;
        const auto it = std::lower_bound(offsets.begin(), offsets.end(), o);
        if (it != offsets.end() && *it < s.end - s.start) return s.start + *it;
        t = s.end;
    }
    return t;   // text behind the last image, or L
}

int32_t bs::PromptGeometry::free_position(int32_t slot) const
{
    // the last image that begins at or before the slot, then its sinks and the text behind it
    const auto it = std::upper_bound(spans.begin(), spans.begin() + n_spans, slot, [](int32_t s, const SpanInfo &x) { return s < x.free_before; });
    if (it == spans.begin()) return slot;
    const SpanInfo &s = *(it - 1);
    const int32_t r = slot - s.free_before, sinks = sinks_in((int32_t)(it - 1 - spans.begin()), s.end - s.start);
    if (r >= sinks) return s.end + (r - sinks);
    return s.start + (r < s.prefix ? r : offsets[offsets_below(s.prefix) + (r - s.prefix)]);
}

int32_t bs::PromptGeometry::text_position(int32_t slot) const
{
    // the span that the text token lies in front of
    const auto it = std::upper_bound(spans.begin(), spans.end(), slot, [](int32_t t, const SpanInfo &s) { return t < s.text_before; });
    return it->start - (it->text_before - slot);
}

int32_t bs::PromptGeometry::tile_runs(int32_t m, std::vector<std::pair<int32_t, int32_t>> &runs) const
{
    runs.clear();
    if (!regrouped) {
        const int64_t r0 = q_begin + (int64_t)m * bm, r1 = std::min<int64_t>(r0 + bm, L);
        runs.push_back({(int32_t)r0, (int32_t)r1});
        return (int32_t)(r1 - r0);
    }
    const bool text = m >= m_img;
    const int32_t first = (text ? m - m_img : m) * bm;
    const int32_t last = (int32_t)std::min<int64_t>((int64_t)first + bm, text ? n_text_rows() : n_img_rows);
    row_runs(text, first, last, runs);
    return last - first;
}

void bs::PromptGeometry::row_runs(bool text, int32_t first, int32_t last, std::vector<std::pair<int32_t, int32_t>> &runs) const
{
    auto add = [&](int32_t a, int32_t b) {
        if (b <= a) return;
        if (!runs.empty() && runs.back().second == a) runs.back().second = b;
        else runs.push_back({a, b});
    };
    if (!regrouped) return add(q_begin + first, q_begin + last);
    const int32_t text0 = n_text(q_begin), img0 = q_begin - text0;   // text / image tokens before the first row
    if (!text) {   // image rows j0 .. j1 - 1 of all image tokens
        const int32_t j0 = img0 + first, j1 = img0 + last;
        auto it = std::upper_bound(spans.begin(), spans.begin() + n_spans, j0, [](int32_t j, const SpanInfo &s) { return j < s.start - s.text_before; }) - 1;
        for (int32_t j = j0; j < j1; ++it) {
            const int32_t a = it->start + (j - (it->start - it->text_before)), b = std::min(it->end, a + (j1 - j));
            add(a, b);
            j += b - a;
        }
        return;
    }
    const int32_t t0 = text0 + first, t1 = text0 + last;
    auto it = std::upper_bound(spans.begin(), spans.end(), t0, [](int32_t t, const SpanInfo &s) { return t < s.text_before; });
    for (int32_t t = t0; t < t1; ++it) {   // the text before *it
        if (it->text_before <= t) continue;
        const int32_t a = it->start - (it->text_before - t), b = std::min(it->start, a + (t1 - t));
        add(a, b);
        t += b - a;
    }
}

void bs::row_bounds(const bs_tilemap *tm, int32_t i, int32_t *first, int32_t *last, int32_t *img_lo, int32_t *img_hi)
{
    *first = tm->window > 0 ? std::max(0, i - tm->window + 1) : 0;
    *last = i;
    *img_lo = *img_hi = 0;
    const PromptGeometry &P = tm->geo;
    const int32_t g = P.span_at(i);
    if (g >= P.n_spans || i < P.spans[g].start) return;
    *img_lo = P.spans[g].start;
    *img_hi = P.spans[g].end;
    if (tm->bidir) {   // the whole own image, also beyond a window
        *last = P.spans[g].end - 1;
        *first = std::min(*first, P.spans[g].start);
    }
}

// Units of the fp32 kernel: every (head, query tile) on its own, heaviest first so the tail of the launch is short;
// ties keep one KV group's heads of a query tile next to each other.
void bs_plan_solo(bs_tilemap *tm)
{
    bs::PairPlan &plan = tm->solo;
    if (plan.epoch == tm->class_epoch) return;
    plan.ranges.clear();
    plan.items.clear();
    const int32_t H = tm->n_q_heads, M = tm->M;
    int32_t base[4];   // the class's lists in plan.ranges
    for (int c = 0; c < 4; ++c) {
        base[c] = -1;
        if (std::find(tm->head_class.begin(), tm->head_class.end(), (uint8_t)c) == tm->head_class.end()) continue;
        base[c] = (int32_t)plan.ranges.size();
        for (const TileRange &r : tm->walked(c).ranges) plan.ranges.push_back({r.begin, (r.end() << 4) | ((r.full() ? 2 : 1) << 2)});
    }
    plan.items.reserve((size_t)H * M);
    for (int32_t h = 0; h < H; ++h) {
        const int c = tm->head_class[h];
        const ClassLists &cl = tm->walked(c);
        for (int32_t m = 0; m < M; ++m)
            plan.items.push_back({h, m, -1, 0, base[c] + (int32_t)cl.row_ptr[m], base[c] + (int32_t)cl.row_ptr[m + 1], cl.row_tiles[m], c | cl.compact[m] << 2});
    }
    std::sort(plan.items.begin(), plan.items.end(), [](const bs::PairItem &a, const bs::PairItem &b) {
        if (a.n_tiles != b.n_tiles) return a.n_tiles > b.n_tiles;
        if (a.tile_a != b.tile_a) return a.tile_a > b.tile_a;
        return a.head_a < b.head_a;
    });
    plan.epoch = tm->class_epoch;
}

// The units of the stacked tiles (see StackedTiles) of the text rows or of the others: a row sees the keys [lo(i), e(i)] of the dense
// mask, both ends grow with the position, so the rows of a tile share [lo(last), e(first)] and see [lo, e] of every run.  One walk
// over all rows, which makes the merged lists at once: this is host time of every new map (28K tokens in a window of 512, 883 units of a group
// of eight: the plan of a new map 275 -> 174 us, 158 without stacking).  Returns the steps of the units.
static int64_t build_stacked(const bs_tilemap *tm, int32_t G, bool text, bs::StackedTiles::Kind &out)
{
    const PromptGeometry &P = tm->geo;
    const int64_t n_rows = text ? P.n_text_rows() : P.n_other_rows(), n_slots = n_rows * G;
    out.n_tiles = (int32_t)((n_slots + P.bm - 1) / P.bm);
    if (out.n_tiles == 0) return 0;
    auto bounds = [&, window = tm->window, in_images = tm->bidir && !text](int32_t i, int32_t &first, int32_t &last) {
        int32_t unused_lo, unused_hi;
        if (in_images) return bs::row_bounds(tm, i, &first, &last, &unused_lo, &unused_hi);
        first = window > 0 ? std::max(0, i - window + 1) : 0;
        last = i;
    };
    std::vector<std::pair<int32_t, int32_t>> runs;   // of all rows
    P.row_runs(text, 0, (int32_t)n_rows, runs);
    size_t run = 0;        // the run that row t0 is in, ...
    int32_t before = 0;    // ... and the rows in front of it
    struct Piece { int32_t begin, end, state; };
    std::vector<Piece> lists[2];
    auto list_of = [&](int32_t j, std::vector<Piece> &list) {
        const int32_t t0 = (int32_t)((int64_t)j * P.bm / G), t1 = (int32_t)((std::min<int64_t>((int64_t)(j + 1) * P.bm, n_slots) - 1) / G);
        while (t0 - before >= runs[run].second - runs[run].first) before += runs[run].second - runs[run].first, ++run;
        size_t r = run;
        int32_t at = before;   // rows in front of run r
        while (t1 - at >= runs[r].second - runs[r].first) at += runs[r].second - runs[r].first, ++r;
        int32_t first, last;
        const size_t r_last = r;
        const int32_t p0 = runs[run].first + (t0 - before), p1 = runs[r_last].first + (t1 - at);
        bounds(p1, first, last);
        const int32_t full_from = (first + P.bn - 1) / P.bn;
        bounds(p0, first, last);
        const int32_t full_end = std::max(full_from, (last + 1) / P.bn);
        list.clear();
        auto emit = [&](int32_t b, int32_t e, int32_t state) { if (e > b) list.push_back({b, e, state}); };
        int32_t done = 0;   // tiles before this one are decided
        for (r = run; r <= r_last; ++r) {
            bounds(r == run ? p0 : runs[r].first, first, last);
            const int32_t b = std::max(done, first / P.bn);
            bounds(r == r_last ? p1 : runs[r].second - 1, first, last);
            const int32_t e = last / P.bn + 1;
            if (e <= b) continue;
            const int32_t f0 = std::min(std::max(full_from, b), e), f1 = std::min(std::max(full_end, f0), e);
            emit(b, f0, 1);
            emit(f0, f1, 2);
            emit(f1, e, 1);
            done = e;
        }
    };
    int64_t steps = 0;
    out.units.reserve((out.n_tiles + 1) / 2);
    for (int32_t j = 0; j < out.n_tiles; j += 2) {
        list_of(j, lists[0]);
        if (j + 1 < out.n_tiles) list_of(j + 1, lists[1]);
        else lists[1].clear();
        const Piece *a = lists[0].data(), *const a_end = a + lists[0].size(), *b = lists[1].data(), *const b_end = b + lists[1].size();
        const int32_t list_begin = (int32_t)out.ranges.size();
        int32_t tiles = 0;
        for (int32_t cur = 0; a < a_end || b < b_end;) {
            const bool in_a = a < a_end && a->begin <= cur, in_b = b < b_end && b->begin <= cur;
            int32_t next = INT32_MAX;   // boundary behind cur
            if (a < a_end) next = std::min(next, in_a ? a->end : a->begin);
            if (b < b_end) next = std::min(next, in_b ? b->end : b->begin);
            const int32_t states = (in_a ? a->state << 2 : 0) | (in_b ? b->state : 0);
            if (states != 0) {
                tiles += next - cur;
                const bool goes_on = (int32_t)out.ranges.size() > list_begin && out.ranges.back().end_states == (cur << 4 | states);
                if (goes_on) out.ranges.back().end_states = next << 4 | states;
                else out.ranges.push_back({cur, next << 4 | states});
            }
            cur = next;
            if (in_a && a->end == cur) ++a;
            if (in_b && b->end == cur) ++b;
        }
        out.units.push_back({list_begin, (int32_t)out.ranges.size(), tiles});
        steps += tiles;
    }
    return steps;
}

// Decides which rows are stacked in groups of G heads.  Without it two heads share a unit at the same 128 rows, and what is lost is
// the last, partly filled tile of every head and the keys that only some of the 128 rows see.  Text rows are few: 37 rows at the
// end of a 36K prompt are a tile of 577 steps for every pair of heads, stacked in groups of seven 1 unit instead of 3.5.
// A unit holds 256 rows either way, so groups of two gain nothing.  Stacked where that saves a thirtieth of the steps of these rows:
// below, units of two kinds side by side share fewer tiles.  (The kernel counts the rows of a group in 32 bits.)
// What lies around a unit is dearer with stacked rows, and in a short window a unit is ten steps long, but it has fewer of them: passes of
// three all-Dense layers, stacked / not: window of 512, 28 / 4 heads, 2.8K tokens 159 / 184 us, 40 / 8, 3.2K 209 / 240, 32 / 8 of d = 64, 2.8K
// 139 / 148, 16 / 2 (groups of eight, less than a unit a workgroup) 2.8K 126 / 129, 3.2K 134 / 130; window of 1024, 2.3K, 166 / 176, 218 / 225,
// 144 / 144, 134 / 139; none, 1.5K, 139 / 145, 157 / 165, 117 / 121, 121 / 123.
static void plan_stacked(bs_tilemap *tm, int32_t G, bool any_all_dense)
{
    bs::StackedTiles &st = tm->stacked;
    if (st.gqa_group != G) st = bs::StackedTiles();
    st.gqa_group = G;
    const PromptGeometry &P = tm->geo;
    if (G < 3 || (int64_t)G * (tm->L - tm->q_begin) >= INT32_MAX - P.bm) return;
    const int32_t m_other = P.regrouped ? P.m_img : tm->M;
    const std::vector<int32_t> &dense = tm->walked(BS_DENSE).row_tiles;
    auto decide = [&](bool text, bs::StackedTiles::Kind &kind) {   // once per map; of the other rows when a group is all Dense for the first time
        if (kind.decided) return;
        int64_t apart = 0;   // steps of one head; two heads walk them together
        for (int32_t m = text ? m_other : 0; m < (text ? tm->M : m_other); ++m) apart += dense[m];
        bs::StackedTiles::Kind made;   // (the map's own stays empty until this is whole: an allocation may fail)
        if (build_stacked(tm, G, text, made) * 60 <= apart * G * 29) kind = std::move(made);
        kind.decided = true;
    };
    if (P.regrouped) decide(true, st.text);
    if (any_all_dense) decide(false, st.other);
}

extern "C" int bs_tilemap_rebind(bs_tilemap *tm, const uint8_t *head_class, int32_t n_q_heads)
{
    if (!tm || !head_class || n_q_heads <= 0) return BS_EINVAL;
    for (int32_t h = 0; h < n_q_heads; ++h)
        if (head_class[h] > 3) return BS_EINVAL;
    if ((size_t)n_q_heads == tm->head_class.size() && std::equal(head_class, head_class + n_q_heads, tm->head_class.begin()))
        return BS_OK;   // same vector: the work units stay valid
    try {
        tm->head_class.assign(head_class, head_class + n_q_heads);
    } catch (const std::bad_alloc &) {
        return BS_ENOMEM;
    }
    tm->n_q_heads = n_q_heads;
    ++tm->class_epoch;
    return BS_OK;
}

// Pairing for the KV-sharing bf16 kernel.  Three rules, all exact (no approximation, only a
// different grouping of the same work), applied inside each KV group:
//   1. heads that carry the same class walk identical lists at the same query tile: pair them
//      two by two (no step is wasted);
//   2. heads left over with different classes may be paired at the same query tile: their lists
//      are merged and each run records the state for either item (a tile only one of them needs
//      is a SKIP step for the other).  Good when most query tiles mix text and image rows (then
//      both walk every causal tile anyway), bad when one class visits far more tiles;
//   3. a left-over head pairs its own query tiles 2j and 2j+1 the same way.
// A pair of left-over heads takes rule 2 or 3, whichever needs fewer steps, and the other one at the query tiles 2j and 2j+1
// where that is clearly shorter: in a window the lists of a Dense and of a sparse head differ on image rows and are the same
// on text rows, of which neighbouring tiles in turn share little.
void bs_plan_pairs(bs_tilemap *tm, int32_t G)
{
    bs::PairPlan &plan = tm->pairs;
    if (plan.gqa_group == G && plan.epoch == tm->class_epoch) return;
    plan.epoch = 0;   // (nobody's until it is whole: an allocation may fail)
    plan.ranges.clear();
    plan.items.clear();
    auto all_dense_group = [&](int32_t kv) {
        return std::all_of(tm->head_class.begin() + kv * G, tm->head_class.begin() + (kv + 1) * G, [](uint8_t c) { return c == BS_DENSE; });
    };
    bool any_all_dense = false;
    for (int32_t kv = 0; kv < tm->n_q_heads / G && !any_all_dense; ++kv) any_all_dense = all_dense_group(kv);
    plan_stacked(tm, G, any_all_dense);
    const bs::StackedTiles &st = tm->stacked;
    const int32_t n_text_tiles = st.text.n_tiles, H = tm->n_q_heads;
    const int32_t M = n_text_tiles > 0 ? tm->geo.m_img : tm->M;   // tiles that are walked head by head

    // merged list of (class ca, row ma) and (class cb, row mb); cb < 0: item A alone
    struct Span2 { int32_t begin, end, tiles; };
    bool count_only = false;
    auto merged = [&](int ca, int32_t ma, int cb, int32_t mb) {
        const ClassLists &la = tm->walked(ca);
        const ClassLists &lb = tm->walked(cb < 0 ? ca : cb);
        int64_t pa = la.row_ptr[ma], ea = la.row_ptr[ma + 1];
        int64_t pb = cb < 0 ? 0 : lb.row_ptr[mb], eb = cb < 0 ? 0 : lb.row_ptr[mb + 1];
        Span2 out{(int32_t)plan.ranges.size(), 0, 0};
        int32_t cur = 0, rb = -1, re = -1, rs = 0;
        auto emit = [&](int32_t b, int32_t e, int sa, int sb) {
            if (e <= b || (sa == 0 && sb == 0)) return;
            out.tiles += e - b;
            const int st = (sa << 2) | sb;
            if (count_only) return;
            if (rb >= 0 && b == re && st == rs) { re = e; return; }
            if (rb >= 0) plan.ranges.push_back({rb, (re << 4) | rs});
            rb = b; re = e; rs = st;
        };
        while (pa < ea || pb < eb) {
            while (pa < ea && la.ranges[pa].end() <= cur) ++pa;
            while (pb < eb && lb.ranges[pb].end() <= cur) ++pb;
            if (pa >= ea && pb >= eb) break;
            const bool in_a = pa < ea && la.ranges[pa].begin <= cur;
            const bool in_b = pb < eb && lb.ranges[pb].begin <= cur;
            int32_t nxt = INT32_MAX;  // next boundary after cur
            if (pa < ea) nxt = std::min(nxt, in_a ? la.ranges[pa].end() : la.ranges[pa].begin);
            if (pb < eb) nxt = std::min(nxt, in_b ? lb.ranges[pb].end() : lb.ranges[pb].begin);
            emit(cur, nxt, in_a ? (la.ranges[pa].full() ? 2 : 1) : 0, in_b ? (lb.ranges[pb].full() ? 2 : 1) : 0);
            cur = nxt;
        }
        if (rb >= 0) plan.ranges.push_back({rb, (re << 4) | rs});
        // Compact tiles first.  They begin with the prompt's first key, which takes most of the weight in many a row, and the
        // probabilities of the largest key of a row's first tile are 1 exactly: it is not rounded to bf16.  (Error of bf16
        // results against fp64 with the image's own tiles first: 4-8 % larger.)
        if (!count_only && tm->n_tiles > tm->N0) {
            size_t i = out.begin;
            while (i < plan.ranges.size() && plan.ranges[i].end_states >> 4 <= tm->N0) ++i;
            if (i < plan.ranges.size() && plan.ranges[i].begin < tm->N0) {   // a run that goes on from the prompt's tiles
                const bs::PairRange whole = plan.ranges[i];
                plan.ranges[i].end_states = (tm->N0 << 4) | (whole.end_states & 15);
                plan.ranges.insert(plan.ranges.begin() + ++i, {tm->N0, whole.end_states});
            }
            std::rotate(plan.ranges.begin() + out.begin, plan.ranges.begin() + i, plan.ranges.end());
        }
        out.end = (int32_t)plan.ranges.size();
        return out;
    };
    // lists shared by many units are made once: key (ca, cb or 4 for "alone"/same row pair kind, row)
    std::vector<Span2> cache_same[4], cache_cross[4][4], cache_rows[4], cache_alone[4];
    auto cached = [&](std::vector<Span2> &tab, int32_t idx, int32_t size, auto make) -> const Span2 & {
        if (tab.empty()) tab.assign(size, Span2{-1, -1, 0});
        if (tab[idx].begin < 0) tab[idx] = make();
        return tab[idx];
    };

    // steps of rule 3 for a class / of rule 2 for a class pair at query tiles 2j and 2j + 1
    const int32_t n_blocks = (M + 1) / 2;
    std::vector<int32_t> rows_steps[4], cross_steps[4][4];
    auto rows_at = [&](int c) -> const std::vector<int32_t> & {
        std::vector<int32_t> &v = rows_steps[c];
        if (v.empty()) {
            count_only = true;
            for (int32_t j = 0; j < n_blocks; ++j)
                v.push_back((2 * j + 1 < M) ? merged(c, 2 * j, c, 2 * j + 1).tiles : merged(c, 2 * j, -1, 0).tiles);
            count_only = false;
        }
        return v;
    };
    auto cross_at = [&](int ca, int cb) -> const std::vector<int32_t> & {
        std::vector<int32_t> &v = cross_steps[std::min(ca, cb)][std::max(ca, cb)];
        if (v.empty()) {
            count_only = true;
            for (int32_t j = 0; j < n_blocks; ++j) {
                int32_t t = merged(ca, 2 * j, cb, 2 * j).tiles;
                if (2 * j + 1 < M) t += merged(ca, 2 * j + 1, cb, 2 * j + 1).tiles;
                v.push_back(t);
            }
            count_only = false;
        }
        return v;
    };
    // Which rule a pair of heads takes: the one with fewer steps in all, and at a block of two query tiles the other one if
    // that saves an eighth there.  (The smaller of the two everywhere: chat_8k of the timed calls 1.5 % slower with 1 % fewer
    // steps, units of two kinds side by side share fewer tiles.)
    struct Pairing { int64_t saving = -1; std::vector<uint8_t> cross; };   // steps saved over rule 3 alone; rule 2 at block j
    Pairing pairing_of[4][4];
    auto pairing = [&](int ca, int cb) -> const Pairing & {
        Pairing &p = pairing_of[std::min(ca, cb)][std::max(ca, cb)];
        if (p.saving >= 0) return p;
        const std::vector<int32_t> &ra = rows_at(ca), &rb = rows_at(cb), &x = cross_at(ca, cb);
        int64_t total = 0;
        for (int32_t j = 0; j < n_blocks; ++j) total += ra[j] + rb[j] - x[j];
        p.saving = 0;
        p.cross.assign(n_blocks, 0);
        for (int32_t j = 0; j < n_blocks; ++j) {
            const int32_t rows = ra[j] + rb[j], saved = rows - x[j];
            p.cross[j] = total > 0 ? -8 * saved < x[j] : 8 * saved > rows;
            if (p.cross[j]) p.saving += saved;
        }
        p.saving = std::max<int64_t>(p.saving, 0);
        return p;
    };

    int32_t text_lists = -1, other_lists = -1;   // where the lists of stacked tiles begin
    auto push_stacked = [&](int32_t kv, const bs::StackedTiles::Kind &kind, int32_t first_id, int32_t &base) {
        if (base < 0) {
            base = (int32_t)plan.ranges.size();
            plan.ranges.insert(plan.ranges.end(), kind.ranges.begin(), kind.ranges.end());
        }
        for (int32_t j = 0; j < kind.n_tiles; j += 2) {   // neighbouring tiles in pairs
            const bs::StackedTiles::Unit &u = kind.units[j / 2];
            const bool pair = j + 1 < kind.n_tiles;
            plan.items.push_back({kv * G, first_id + j, pair ? kv * G : -1, pair ? first_id + j + 1 : 0, base + u.list_begin, base + u.list_end, u.n_tiles, 0});
        }
    };
    std::vector<int32_t> byclass[4], rest;
    for (int32_t kv = 0; kv < H / G; ++kv) {
        if (n_text_tiles > 0) push_stacked(kv, st.text, tm->M, text_lists);
        // (without stacked text rows these are among the tiles of every head)
        const bool all_dense = any_all_dense && all_dense_group(kv);
        if (all_dense && st.other.n_tiles > 0 && (n_text_tiles > 0 || !tm->geo.regrouped)) {
            push_stacked(kv, st.other, tm->M + n_text_tiles, other_lists);
            continue;
        }
        for (int c = 0; c < 4; ++c) byclass[c].clear();
        for (int32_t h = kv * G; h < (kv + 1) * G; ++h) byclass[tm->head_class[h]].push_back(h);
        rest.clear();
        for (int c = 0; c < 4; ++c) {
            size_t i = 0;
            for (; i + 1 < byclass[c].size(); i += 2)  // rule 1
                for (int32_t m = 0; m < M; ++m) {
                    const Span2 &sp = cached(cache_same[c], m, M, [&] { return merged(c, m, c, m); });
                    plan.items.push_back({byclass[c][i], m, byclass[c][i + 1], m, sp.begin, sp.end, sp.tiles, 0});
                }
            if (i < byclass[c].size()) rest.push_back(byclass[c][i]);
        }
        auto push_rows = [&](int32_t h, int32_t j) {   // rule 3
            const int c = tm->head_class[h];
            if (2 * j + 1 < M) {
                const Span2 &sp = cached(cache_rows[c], j, n_blocks, [&] { return merged(c, 2 * j, c, 2 * j + 1); });
                plan.items.push_back({h, 2 * j, h, 2 * j + 1, sp.begin, sp.end, sp.tiles, 0});
            } else {
                const Span2 &sp = cached(cache_alone[c], 0, 1, [&] { return merged(c, 2 * j, -1, 0); });
                plan.items.push_back({h, 2 * j, -1, 0, sp.begin, sp.end, sp.tiles, 0});
            }
        };
        // rule 2 where it saves steps over rule 3: repeatedly take the pair with the best saving
        while (rest.size() >= 2) {
            int64_t best = 0;
            size_t bi = 0, bj = 0;
            for (size_t i = 0; i < rest.size(); ++i)
                for (size_t j = i + 1; j < rest.size(); ++j) {
                    const int ca = tm->head_class[rest[i]], cb = tm->head_class[rest[j]];
                    const int64_t saving = pairing(ca, cb).saving;
                    if (saving > best) { best = saving; bi = i; bj = j; }
                }
            if (best <= 0) break;
            const int32_t ha = rest[bi], hb = rest[bj];
            const int ca = tm->head_class[ha], cb = tm->head_class[hb];
            for (int32_t j = 0; j < n_blocks; ++j) {
                if (!pairing(ca, cb).cross[j]) {
                    push_rows(ha, j);
                    push_rows(hb, j);
                    continue;
                }
                for (int32_t m = 2 * j; m < std::min(2 * j + 2, M); ++m) {
                    const Span2 &sp = cached(cache_cross[ca][cb], m, M, [&] { return merged(ca, m, cb, m); });
                    plan.items.push_back({ha, m, hb, m, sp.begin, sp.end, sp.tiles, 0});
                }
            }
            rest.erase(rest.begin() + bj);
            rest.erase(rest.begin() + bi);
        }
        for (int32_t h : rest)
            for (int32_t j = 0; j < n_blocks; ++j) push_rows(h, j);
    }
    // Queue order.  Heaviest units first (longest-processing-time rule), but in coarse cost
    // buckets inside which units of one KV head stay together, walking the same tiles at about
    // the same time.  The sorted list is then dealt to eight queues, one per XCD (each XCD has its
    // own L2), in blocks of kXcdBlock consecutive units: the units of a block run side by side on
    // one XCD and find each other's K / V^T tiles in its L2.  The kernel's workgroups take the
    // units of their XCD's queue in this order (plan.queue_off delimits the queues in plan.items).
    // Block size: 8 for a few thousand units (a bigger block costs load balance at the tail),
    // 16 for tens of thousands (measured on the 36K and 300K workloads).
    // Bucket width: 32 tiles for up to four KV heads.  With more KV heads a 32-tile bucket holds about one
    // block of each head, neighbours in a queue read different heads and the L2s share less: the width
    // grows with the square of the head count (measured: 16 KV heads at 300K tokens gain 2-3 % from 512-
    // 1024 tiles, 8 KV heads at 140K 0.3-1 % from 256-1024, 4 KV heads lose 0.2-0.5 % with anything above
    // 32), but never so wide that the heaviest-first order loses its grip on the tail (a workgroup's
    // share of the steps / 64; below 32 tiles on prompts of less than some 20K tokens, whose K and V the caches
    // hold anyway).
    // Blocks are dealt there and back, so that every queue gets heavy and light ones alike.  Dealt in turn, the first queue of a launch with
    // 16 / 28 rounds of blocks has 11-24 / 7-14 % more steps than the last, there and back 1-2 %: d = 64, 9K tokens, 1144 units, 779 -> 767 us, 8K
    // tokens, 912 units, 936 -> 931; single layers in turn / there and back, 16K of d = 64, 2021 units, 480.2 / 472.5, 11K, 1745 units,
    // 489.8 / 485.2, 16K, 1760, 660.5 / 659.2.  With more units the first queue still has 2-11 % more (41 rounds 1.04 and 1.11, 68 rounds 1.02 and
    // 1.06), but whoever has emptied its own helps on the next one, and neighbours in a queue meet less in L2 if it is dealt there and back: 16K,
    // 2520 units, 941.3 / 935.1, 24K, 2632, 1296 / 1296 and, all Dense, 3248 / 3243, 24K of d = 64, 3008, 918.9 / 917.5 and 2232 / 2249, 39.5K, 4333,
    // 3144 / 3147 and 8566 / 8561, 60K, 6572, 6917 / 6925; 281K of d = 64, 8 KV heads, 8800, 29.9 / 30.2 ms.  So the line lies where
    // the gain ends.  In a window the blocks of a bucket are alike (1430 / 1432).
    // In a window the cost says nothing about where a unit's keys lie: inside a bucket the units of a KV head stand in order
    // of their rows, and the buckets are 8 tiles wide (27K tokens, images of 256, window of 1024: 1624 -> 1603 us for three
    // layers, 4096: 3216 -> 3192, images of 1-5K 1388 -> 1364; 16 tiles the same, 64 tiles 2 % slower: the tail).
    constexpr int32_t kXcds = 8;
    int32_t cost_bucket = 32;
    {
        int64_t total = 0;
        for (const bs::PairItem &it : plan.items) total += it.n_tiles;
        const int64_t n_kv = std::max<int64_t>(1, (int64_t)tm->head_class.size() / std::max(G, 1));
        const int64_t for_locality = 32 * std::max<int64_t>(1, n_kv / 4) * std::max<int64_t>(1, n_kv / 4);
        const int64_t for_balance = total / 256 / 64;                     // 256 workgroups
        cost_bucket = (int32_t)std::max<int64_t>(1, for_balance < 32 ? for_balance : std::min(for_locality, for_balance) / 32 * 32);
    }
    if (tm->window > 0) cost_bucket = 8;
    const bool there_and_back = tm->window == 0 && plan.items.size() <= 2048;
    const int32_t kXcdBlock = std::min<int64_t>(16, std::max<int64_t>(8, (int64_t)plan.items.size() / 2048));
    {
        // Stable counting passes, a byte at a time, from the last field to the first: a sort that compares units took 50-70 ns each, more
        // than half of the planning that every rebinding pays (4336 units 358 -> 148 us; in a window, 4076 units, 511 -> 268).
        struct Place { uint32_t key; int32_t unit; };
        const size_t n = plan.items.size();
        std::vector<Place> order(n), moved(n);
        for (size_t i = 0; i < n; ++i) order[i].unit = (int32_t)i;
        auto by = [&](auto &&field) {
            uint32_t bits = 0;
            for (Place &p : order) bits |= p.key = (uint32_t)field(plan.items[p.unit]);
            for (int shift = 0; shift < 32 && bits >> shift != 0; shift += 8) {
                uint32_t at[257] = {0};
                for (const Place &p : order) ++at[(p.key >> shift & 255) + 1];
                for (int i = 0; i < 256; ++i) at[i + 1] += at[i];
                for (const Place &p : order) moved[at[p.key >> shift & 255]++] = p;
                order.swap(moved);
            }
        };
        int32_t longest = 0;
        for (const bs::PairItem &it : plan.items) longest = std::max(longest, it.n_tiles);
        if (tm->window > 0) by([](const bs::PairItem &it) { return it.tile_a; });
        else by([&](const bs::PairItem &it) { return longest - it.n_tiles; });
        by([&](const bs::PairItem &it) { return it.head_a / G; });
        by([&](const bs::PairItem &it) { return longest / cost_bucket - it.n_tiles / cost_bucket; });
        std::vector<bs::PairItem> queued;
        queued.reserve(n);
        for (int x = 0; x < kXcds; ++x) {
            plan.queue_off[x] = (int32_t)queued.size();
            for (size_t round = 0; round * kXcds * kXcdBlock < n; ++round) {
                const size_t block = (round * kXcds + (there_and_back && (round & 1) ? kXcds - 1 - x : x)) * kXcdBlock;
                for (size_t p = block; p < std::min(n, block + kXcdBlock); ++p) queued.push_back(plan.items[order[p].unit]);
            }
        }
        plan.queue_off[kXcds] = (int32_t)n;
        plan.back_block = there_and_back ? kXcdBlock : 0;
        plan.items.swap(queued);
    }
    auto item_class = [&](int32_t head, int32_t tile) { return tile >= tm->M ? BS_DENSE | 8 : tm->head_class[head] | tm->walked(tm->head_class[head]).compact[tile] << 2; };
    for (bs::PairItem &it : plan.items)
        it.classes = item_class(it.head_a, it.tile_a) | (it.head_b >= 0 ? item_class(it.head_b, it.tile_b) << 8 : 0);
    plan.gqa_group = G;
    plan.epoch = tm->class_epoch;
}

// Equal shares.  The queues balance a launch as long as there are many units per workgroup and none is long; with
// few units -- a short prompt, a chunk of a few hundred rows behind a long cache -- most of the chip waits for the
// longest one.  Here every workgroup gets units up to an equal share of the steps: first whole ones, longest first
// (neighbours in that order walk the same tiles side by side and share them in L2), then the room that is left is
// filled with parts of the units that found no place, cut along their key tiles.  A cut unit leaves partial results
// (unnormalised output, reference point, row sum) that a second kernel merges.  The time per step differs by up to
// 15 % between workgroups (which tiles they find in L2, partial tiles), so long shares keep back a part of the steps
// as short pieces that go to the queues, for whoever is done first.
// Costs are in key-tile steps: a unit or part costs its steps and kUnitCost around them, the merge kMergeCost for the launch.
// (The merge: 6 us, the gap in front of it, and the host's share of planning and launching it, of steps of 1.0 us at d = 64 and 1.7 at 128.
// 240 prompts of 0.6-4K tokens, passes with 6 / 7 / 8, the same plans for nearly all of them: 8 heads of d = 64, 970 tokens 71.2 / 71.9 / 77.5 us,
// 960 tokens 100 / 101 / 106; 32 heads, 990 tokens 83.9 / 84.1 / 88.3, 940 tokens 46.4 / 42.8 / 42.9, 1.4K tokens 55.3 / 54.5 / 52.2; 28
// heads of d = 128, 920 tokens 83.2 / 80.3 / 80.2; 32 heads, 890 tokens 90.5 / 90.4 / 93.6.)
// (By time stamps what lies around a unit takes 5 us against 1.7 us per step; 4 instead of 6: 4000 rows behind 30K 1426 -> 1410 us,
// 517 rows behind 36K 576 -> 572, but 300 rows behind 20K of d = 64 220 -> 225; 3 and 2: mixed, or slower.)
static void make_shares(const bs_tilemap *tm, const bs::PairPlan &plan, bool solo, int32_t G, int32_t n_wgs, bs::SharePlan &sp)
{
    sp.parts.clear(); sp.ranges.clear(); sp.share_off.clear(); sp.cut.clear();
    sp.n_slots = 0;
    std::fill(sp.queue_off, sp.queue_off + 9, 0);
    // the fp32 kernel's steps take 3.5-7 us
    const int64_t kUnitCost = solo ? 1 : 6, kMergeCost = solo ? 1 : 7, kMinPart = solo ? 1 : 4;
    // With more units than that the queues are better, although their longest workgroup has 5-6 % more steps than the mean on
    // prompts of 8-9K tokens (by the plan's steps; the time per step differs, and the queues make up for that, too).
    // Limit 8 instead of 3: 3 layers of 28 heads at 8.2K tokens (3.6 units) 1062 us, 1045 with 3; 32 heads of d = 64 at 9K
    // (4.5 units) 1008 and 971; the four runs of a 16K characterisation (6.9 units) 3655 and 3358.
    constexpr int64_t kMaxUnitsPerWg = 3;
    const int32_t n_units = (int32_t)std::min<size_t>(plan.items.size(), INT32_MAX);
    if (n_units > kMaxUnitsPerWg * n_wgs || n_wgs > 4096) return;
    int64_t total = 0, longest = 0;
    for (const bs::PairItem &it : plan.items) {
        total += it.n_tiles + kUnitCost;
        longest = std::max<int64_t>(longest, it.n_tiles + kUnitCost);
    }
    // a fresh share always takes a part: it is longer than two of the shortest
    const int64_t least = std::max<int64_t>((total + n_wgs - 1) / n_wgs, 2 * kMinPart + kUnitCost);
    if (n_units <= n_wgs && longest <= least + kMergeCost) return;

    // Longest first, in buckets of an eighth of a share inside which the units of a KV head stay together, in the order of the queues
    // as dealing in turn fills them: which units are cut, and so how the results are rounded, does not hang on how the queues are dealt.
    std::vector<int32_t> in_turn;
    if (plan.back_block > 0) {
        in_turn.reserve(n_units);
        for (int32_t x = 0; x < 8; ++x)
            for (int32_t round = 0; (round * 8 + x) * plan.back_block < n_units; ++round) {
                const int32_t first = plan.queue_off[round & 1 ? 7 - x : x] + round * plan.back_block;
                for (int32_t i = 0; i < std::min(plan.back_block, n_units - (round * 8 + x) * plan.back_block); ++i) in_turn.push_back(first + i);
            }
    }
    const int64_t bucket = std::max<int64_t>(1, least / 8);
    struct Unit { int32_t cost, unit; };   // (costs are below 2^28: n_tiles is)
    std::vector<Unit> order(n_units);
    {   // two stable counting passes: KV head, then bucket
        std::vector<int32_t> by_head(n_units), at;
        auto pass = [&](int64_t n_keys, auto &&unit, auto &&key, auto &&place) {
            at.assign(n_keys + 1, 0);
            for (int32_t i = 0; i < n_units; ++i) ++at[key(unit(i)) + 1];
            for (int64_t k = 0; k < n_keys; ++k) at[k + 1] += at[k];
            for (int32_t i = 0; i < n_units; ++i) place(at[key(unit(i))]++, unit(i));
        };
        pass((tm->n_q_heads + G - 1) / G, [&](int32_t i) { return in_turn.empty() ? i : in_turn[i]; }, [&](int32_t u) { return plan.items[u].head_a / G; },
             [&](int32_t i, int32_t u) { by_head[i] = u; });
        pass(longest / bucket + 1, [&](int32_t i) { return by_head[i]; },
             [&](int32_t u) { return (int32_t)(longest / bucket - plan.items[u].n_tiles / bucket); },
             [&](int32_t i, int32_t u) { order[i] = {plan.items[u].n_tiles + (int32_t)kUnitCost, u}; });
    }
    // Units in order to the least loaded workgroup (the first of several), if `accept` says so; no load passes `most`.  The
    // least load only grows, so the workgroups lie in a set per load.  (Planning is host time that every layer pays: 624
    // units of a windowed prompt of 5K tokens take 72 us; with a heap of pairs and a sort of them it was 300, three times the
    // kernels' time.)
    std::vector<int64_t> load(n_wgs);
    std::vector<uint64_t> sets;
    auto deal = [&](int64_t most, auto &&accept) {
        std::fill(load.begin(), load.end(), 0);
        int32_t w = 0, i = 0;          // first to the next workgroup that has nothing yet
        for (; i < n_units && w < n_wgs; ++i)
            if (accept(order[i], w, 0)) load[w++] = order[i].cost;
        if (i == n_units) return;
        const int32_t words = (n_wgs + 63) / 64;
        sets.assign((size_t)(most + 1) * words, 0);
        auto put = [&](int32_t w) { sets[(size_t)load[w] * words + (w >> 6)] |= (uint64_t)1 << (w & 63); };
        for (w = 0; w < n_wgs; ++w) put(w);
        for (size_t first = 0; i < n_units; ++i) {
            while (sets[first] == 0) ++first;
            w = (int32_t)(first % words) * 64 + __builtin_ctzll(sets[first]);
            if (!accept(order[i], w, load[w])) continue;
            sets[first] &= sets[first] - 1;
            load[w] += order[i].cost;
            put(w);                    // (behind this set: a unit costs something)
        }
    };
    int64_t queued = longest;   // what the queues need: heaviest first onto the workgroup that is free first
    if (n_units > n_wgs) {
        deal(total / n_wgs + longest, [](const Unit &, int32_t, int64_t) { return true; });
        for (int64_t l : load) queued = std::max(queued, l);
    }

    struct Piece { int32_t wg, unit, begin, steps; };
    std::vector<Piece> pieces;
    std::vector<int32_t> homeless;
    const int64_t kQueuedFrom = solo ? INT64_MAX : 600;   // shares from here on hand a sixth of the steps to the queues ...
    auto fill = [&](int64_t share) {       // false: units are left over
        const int64_t fixed = share >= kQueuedFrom ? share - share / 6 : share;
        const int64_t queue_piece = share / 24;   // ... in pieces of four to that sixth
        pieces.clear();
        homeless.clear();
        int64_t left_over = 0, room_left = 0;
        deal(fixed, [&](const Unit &o, int32_t w, int64_t load_w) {
            if (load_w + o.cost > fixed) {
                homeless.push_back(o.unit);
                left_over += o.cost;
                return false;
            }
            pieces.push_back({w, o.unit, 0, o.cost - (int32_t)kUnitCost});
            return true;
        });
        for (int64_t l : load) room_left += fixed - l;
        if (fixed == share && left_over > room_left) return false;
        int32_t w = 0;
        for (int32_t u : homeless) {
            int32_t done = 0;
            bool placed = false;   // (a unit without a key tile is a piece of its own: its rows are zeros, and somebody has to write them)
            for (int32_t left = plan.items[u].n_tiles; left > 0 || !placed;) {
                if (w == n_wgs && fixed == share) return false;
                const int64_t room = w == n_wgs ? queue_piece : fixed - load[w] - kUnitCost;
                // the rest of the unit, or a part as long as the room; neither it nor the rest too short
                const int64_t take = left <= room ? left : std::min<int64_t>(room, left - kMinPart);
                if (take >= std::min<int64_t>(left, kMinPart)) {
                    pieces.push_back({w, u, done, (int32_t)take});
                    if (w < n_wgs) load[w] += take + kUnitCost;
                    done += (int32_t)take;
                    left -= (int32_t)take;
                    placed = true;
                }
                if ((left > 0 || !placed) && w < n_wgs) ++w;
            }
        }
        return true;
    };
    // The first share with room for every unit and the cuts it takes (a part costs a unit's worth again); starting a
    // unit's worth above the mean instead left 20-40 of 256 workgroups without work on short prompts (28 heads, 1.3K
    // tokens: longest workgroup 15 steps, now 11; 243 -> 235 us a pass of four layers).
    auto has_room = [&](int64_t share) {
        int64_t need = 0;
        for (const bs::PairItem &it : plan.items)
            need += it.n_tiles + kUnitCost * (it.n_tiles <= share - kUnitCost ? 1 : (it.n_tiles + share - kUnitCost - 1) / (share - kUnitCost));
        return need <= share * n_wgs;
    };
    int64_t share = least;
    while (share + kMergeCost < queued && !(has_room(share) && fill(share))) share += std::max<int64_t>(1, share / 32);
    if (share + kMergeCost >= queued) return;   // no gain over the queues
    std::vector<int32_t> off(n_wgs + 2, 0);   // (the queued pieces count as those of workgroup n_wgs)
    for (const Piece &p : pieces) ++off[p.wg + 1];
    for (int32_t w = 0; w <= n_wgs; ++w) off[w + 1] += off[w];
    {   // by workgroup, the pieces of one in the order they were made
        std::vector<int32_t> at(off.begin(), off.end() - 1);
        std::vector<Piece> sorted(pieces.size());
        for (const Piece &p : pieces) sorted[at[p.wg]++] = p;
        pieces.swap(sorted);
    }
    off.pop_back();
    for (int q = 0; q <= 8; ++q) sp.queue_off[q] = (int32_t)(off[n_wgs] + (pieces.size() - off[n_wgs]) * q / 8);

    std::vector<int32_t> n_parts(n_units, 0), made(n_units, 0), slot0(n_units, -1);
    for (const Piece &p : pieces) ++n_parts[p.unit];
    sp.parts.reserve(pieces.size());
    for (const Piece &p : pieces) {
        const bs::PairItem &it = plan.items[p.unit];
        bs::PairItem part = it;
        int32_t slot = 0;
        if (n_parts[p.unit] > 1) {
            if (slot0[p.unit] < 0) {
                slot0[p.unit] = sp.n_slots;
                sp.n_slots += n_parts[p.unit];
                sp.cut.push_back({it.head_a, it.tile_a, slot0[p.unit], n_parts[p.unit] << 1});
                if (it.head_b >= 0) sp.cut.push_back({it.head_b, it.tile_b, slot0[p.unit], n_parts[p.unit] << 1 | 1});
            }
            slot = slot0[p.unit] + made[p.unit]++ + 1;
        }
        part.list_begin = (int32_t)sp.ranges.size();
        part.n_tiles = p.steps;
        int32_t skip = p.begin, left = p.steps;
        for (int32_t r = it.list_begin; r < it.list_end && left > 0; ++r) {
            const bs::PairRange &rg = plan.ranges[r];
            const int32_t len = (rg.end_states >> 4) - rg.begin;
            if (skip >= len) { skip -= len; continue; }
            const int32_t b = rg.begin + skip, e = std::min(rg.end_states >> 4, b + left);
            sp.ranges.push_back({b, (e << 4) | (rg.end_states & 15)});
            left -= e - b;
            skip = 0;
        }
        part.list_end = (int32_t)sp.ranges.size();
        part.classes = it.classes | slot << 16;
        sp.parts.push_back(part);
    }
    sp.share_off = off;
    if (sp.n_slots >= 32767) {   // the slot has 15 bits next to the classes
        sp.parts.clear(); sp.ranges.clear(); sp.share_off.clear(); sp.cut.clear();
        sp.n_slots = 0;
    }
}

void bs_plan_shares(bs_tilemap *tm, int32_t gqa_group, int32_t n_wgs)
{
    bs::SharePlan &sp = tm->shares;
    const bool solo = gqa_group == 0;
    if (solo) bs_plan_solo(tm);
    else bs_plan_pairs(tm, gqa_group);   // (also where the shares are there: the units may be those of another group size by now)
    if (sp.gqa_group == gqa_group && sp.epoch == tm->class_epoch && sp.n_wgs == n_wgs) return;
    sp.epoch = 0;   // (as for a plan of units)
    make_shares(tm, solo ? tm->solo : tm->pairs, solo, std::max(gqa_group, 1), n_wgs, sp);
    sp.gqa_group = gqa_group; sp.n_wgs = n_wgs; sp.epoch = tm->class_epoch;
}

extern "C" int bs_tilemap_pair_plan(bs_tilemap *tm, int32_t gqa_group, int64_t *n_units, int64_t *unit_tiles,
                                    int64_t *skip_steps)
{
    if (!tm || gqa_group <= 0 || tm->n_q_heads % gqa_group != 0) return BS_EINVAL;
    try {
        bs_plan_pairs(tm, gqa_group);
        // check the plan against the per-class lists it was derived from
        const bs::PairPlan &plan = tm->pairs;
        std::vector<uint8_t> want(tm->n_tiles), got_a(tm->n_tiles), got_b(tm->n_tiles);
        const bs::StackedTiles &st = tm->stacked;
        const int32_t M = tm->M + st.text.n_tiles + st.other.n_tiles;   // ids of query tiles
        std::vector<int32_t> seen((size_t)tm->n_q_heads * M, 0);
        // the states of an item: from the lists of its class, of a stacked tile from what its rows see one by one
        std::vector<std::vector<uint8_t>> stacked_states(M - tm->M);
        auto expected = [&](int32_t head, int32_t tile) {
            if (tile < tm->M) return expand_states(tm->walked(tm->head_class[head]), tile, want);
            std::vector<uint8_t> &states = stacked_states[tile - tm->M];
            if (states.empty()) {
                const bool text = tile - tm->M < st.text.n_tiles;
                const int32_t n_rows = text ? tm->geo.n_text_rows() : tm->geo.n_other_rows();
                const int64_t s0 = (int64_t)(tile - tm->M - (text ? 0 : st.text.n_tiles)) * tm->bm;
                std::vector<std::pair<int32_t, int32_t>> runs;
                tm->geo.row_runs(text, (int32_t)(s0 / gqa_group), (int32_t)std::min<int64_t>(n_rows, (s0 + tm->bm - 1) / gqa_group + 1), runs);
                states.assign(tm->n_tiles, 2);
                std::vector<uint8_t> any(tm->n_tiles, 0);
                for (const auto &r : runs)
                    for (int32_t i = r.first; i < r.second; ++i) {
                        int32_t lo, hi, unused_lo, unused_hi;
                        bs::row_bounds(tm, i, &lo, &hi, &unused_lo, &unused_hi);
                        for (int32_t n = 0; n < tm->n_tiles; ++n) {
                            const bool seen_some = n < tm->N0 && lo < (n + 1) * tm->bn && hi >= n * tm->bn;
                            any[n] |= (uint8_t)seen_some;
                            if (!seen_some || lo > n * tm->bn || hi < (n + 1) * tm->bn - 1) states[n] = 1;
                        }
                    }
                for (int32_t n = 0; n < tm->n_tiles; ++n) states[n] = any[n] ? states[n] : 0;
            }
            want = states;
        };
        int64_t tiles = 0, skips = 0;
        for (const bs::PairItem &it : plan.items) {
            if (it.head_a < 0 || it.head_a >= tm->n_q_heads || it.tile_a < 0 || it.tile_a >= M) return BS_EINVAL;
            if (it.head_b >= tm->n_q_heads || (it.head_b >= 0 && (it.tile_b < 0 || it.tile_b >= M))) return BS_EINVAL;
            if (it.head_b >= 0 && it.head_b / gqa_group != it.head_a / gqa_group) return BS_EINVAL;
            // (a stacked tile stands under the first head of its group; those of the other rows only if all its heads are Dense)
            for (int i = 0; i < 2; ++i) {
                const int32_t head = i ? it.head_b : it.head_a, tile = i ? it.tile_b : it.tile_a;
                if (head < 0 || tile < tm->M) continue;
                if (head % gqa_group != 0) return BS_EINVAL;
                for (int32_t h = head; h < head + gqa_group; ++h)
                    if (tile >= tm->M + st.text.n_tiles && tm->head_class[h] != BS_DENSE) return BS_EINVAL;
            }
            ++seen[(size_t)it.head_a * M + it.tile_a];
            if (it.head_b >= 0) ++seen[(size_t)it.head_b * M + it.tile_b];
            std::fill(got_a.begin(), got_a.end(), 0);
            std::fill(got_b.begin(), got_b.end(), 0);
            bool in_prompt = false;   // the compact tiles come first, then the prompt's, both in order
            int32_t prev_end = 0, n_tiles = 0;
            for (int32_t p = it.list_begin; p < it.list_end; ++p) {
                const bs::PairRange &r = plan.ranges[p];
                const int32_t e = r.end_states >> 4, sa = (r.end_states >> 2) & 3, sb = r.end_states & 3;
                if (r.begin < tm->N0 && !in_prompt) {
                    in_prompt = true;
                    prev_end = 0;
                }
                if (r.begin < prev_end || e <= r.begin || e > (in_prompt ? tm->N0 : tm->n_tiles) || (sa == 0 && sb == 0) || sa == 3 || sb == 3) return BS_EINVAL;
                for (int32_t n = r.begin; n < e; ++n) { got_a[n] = (uint8_t)sa; got_b[n] = (uint8_t)sb; }
                skips += (int64_t)(e - r.begin) * ((sa == 0) + (sb == 0 && it.head_b >= 0));
                n_tiles += e - r.begin;
                prev_end = e;
            }
            if (n_tiles != it.n_tiles) return BS_EINVAL;
            tiles += n_tiles;
            expected(it.head_a, it.tile_a);
            if (want != got_a) return BS_EINVAL;
            if (it.head_b >= 0) {
                expected(it.head_b, it.tile_b);
                if (want != got_b) return BS_EINVAL;
            }
        }
        // every row of every head exactly once: in its head's tile or in a stacked one of its group
        const int32_t m_text = tm->geo.regrouped ? tm->geo.m_img : tm->M;
        for (int32_t h = 0; h < tm->n_q_heads; ++h) {
            const int32_t *own = seen.data() + (size_t)h * M, *group = seen.data() + (size_t)(h - h % gqa_group) * M;
            auto once = [&](int32_t begin, int32_t end, int32_t stacked_begin, int32_t stacked_end) {
                const bool stacked = stacked_end > stacked_begin && group[stacked_begin] > 0;
                for (int32_t m = begin; m < end; ++m)
                    if (own[m] != (stacked ? 0 : 1)) return false;
                for (int32_t m = stacked_begin; m < stacked_end; ++m)
                    if (group[m] != (stacked ? 1 : 0) || (own != group && own[m] != 0)) return false;
                return true;
            };
            if (!once(m_text, tm->M, tm->M, tm->M + st.text.n_tiles) || !once(0, m_text, tm->M + st.text.n_tiles, M)) return BS_EINVAL;
        }
        if (n_units) *n_units = (int64_t)plan.items.size();
        if (unit_tiles) *unit_tiles = tiles;
        if (skip_steps) *skip_steps = skips;
    } catch (const std::bad_alloc &) {
        return BS_ENOMEM;
    }
    return BS_OK;
}

extern "C" int bs_tilemap_share_plan(bs_tilemap *tm, int32_t gqa_group, int32_t n_wgs, int64_t *n_parts, int64_t *n_cut_units,
                                     int64_t *n_queued)
{
    if (!tm || gqa_group < 0 || (gqa_group > 0 && tm->n_q_heads % gqa_group != 0) || n_wgs <= 0) return BS_EINVAL;
    try {
        bs_plan_shares(tm, gqa_group, n_wgs);
        const bs::PairPlan &plan = gqa_group == 0 ? tm->solo : tm->pairs;
        const bs::SharePlan &sp = tm->shares;
        const size_t n_units = plan.items.size();
        int64_t cut_units = 0;
        if (sp.share_off.empty()) {
            if (!sp.parts.empty() || !sp.cut.empty() || sp.n_slots != 0) return BS_EINVAL;
        } else {
            // every part is in the share of one workgroup or in one queue
            if (sp.share_off.size() != (size_t)n_wgs + 1 || sp.share_off[0] != 0 || sp.share_off[n_wgs] != sp.queue_off[0]) return BS_EINVAL;
            for (int32_t w = 0; w < n_wgs; ++w)
                if (sp.share_off[w + 1] < sp.share_off[w]) return BS_EINVAL;
            for (int q = 0; q < 8; ++q)
                if (sp.queue_off[q + 1] < sp.queue_off[q]) return BS_EINVAL;
            if ((size_t)sp.queue_off[8] != sp.parts.size()) return BS_EINVAL;

            // the parts of every unit
            const int32_t M = tm->M + (gqa_group > 0 ? tm->stacked.text.n_tiles + tm->stacked.other.n_tiles : 0);   // ids of query tiles
            std::vector<int32_t> unit_of((size_t)tm->n_q_heads * M, -1);
            for (size_t u = 0; u < n_units; ++u) unit_of[(size_t)plan.items[u].head_a * M + plan.items[u].tile_a] = (int32_t)u;
            std::vector<std::vector<int32_t>> parts_of(n_units);
            for (size_t i = 0; i < sp.parts.size(); ++i) {
                const bs::PairItem &p = sp.parts[i];
                if (p.head_a < 0 || p.head_a >= tm->n_q_heads || p.tile_a < 0 || p.tile_a >= M) return BS_EINVAL;
                const int32_t u = unit_of[(size_t)p.head_a * M + p.tile_a];
                if (u < 0) return BS_EINVAL;
                const bs::PairItem &it = plan.items[u];
                if (p.head_b != it.head_b || p.tile_b != it.tile_b || (p.classes & 0xffff) != it.classes) return BS_EINVAL;
                parts_of[u].push_back((int32_t)i);
            }
            std::vector<uint8_t> want(tm->n_tiles), got(tm->n_tiles), slot_used(sp.n_slots, 0);
            std::vector<bs::CutItem> cut;
            for (size_t u = 0; u < n_units; ++u) {
                const bs::PairItem &it = plan.items[u];
                if (parts_of[u].empty()) return BS_EINVAL;   // its rows would never be written
                const int32_t n = (int32_t)parts_of[u].size();
                // together the parts walk each of the unit's tiles once, in the unit's states
                std::fill(want.begin(), want.end(), 0);
                std::fill(got.begin(), got.end(), 0);
                for (int32_t r = it.list_begin; r < it.list_end; ++r)
                    for (int32_t t = plan.ranges[r].begin; t < plan.ranges[r].end_states >> 4; ++t)
                        want[t] = (uint8_t)(plan.ranges[r].end_states & 15);
                int32_t first_slot = INT32_MAX, last_slot = -1;
                for (int32_t i : parts_of[u]) {
                    const bs::PairItem &p = sp.parts[i];
                    int32_t steps = 0;
                    if (p.list_begin < 0 || p.list_end < p.list_begin || (size_t)p.list_end > sp.ranges.size()) return BS_EINVAL;
                    for (int32_t r = p.list_begin; r < p.list_end; ++r) {
                        const int32_t b = sp.ranges[r].begin, e = sp.ranges[r].end_states >> 4;
                        if (b < 0 || e <= b || e > tm->n_tiles) return BS_EINVAL;
                        for (int32_t t = b; t < e; ++t) {
                            if (got[t] != 0) return BS_EINVAL;
                            got[t] = (uint8_t)(sp.ranges[r].end_states & 15);
                        }
                        steps += e - b;
                    }
                    if (steps != p.n_tiles) return BS_EINVAL;
                    const int32_t slot = p.classes >> 16;   // slot + 1, 0: not a part
                    if ((slot > 0) != (n > 1) || slot > sp.n_slots) return BS_EINVAL;
                    if (slot > 0) {
                        if (slot_used[slot - 1]) return BS_EINVAL;
                        slot_used[slot - 1] = 1;
                        first_slot = std::min(first_slot, slot - 1);
                        last_slot = std::max(last_slot, slot - 1);
                    }
                }
                if (want != got) return BS_EINVAL;
                if (n > 1) {
                    if (last_slot - first_slot != n - 1) return BS_EINVAL;   // one behind the other: the merge walks them
                    ++cut_units;
                    cut.push_back({it.head_a, it.tile_a, first_slot, n << 1});
                    if (it.head_b >= 0) cut.push_back({it.head_b, it.tile_b, first_slot, n << 1 | 1});
                }
            }
            auto less = [](const bs::CutItem &a, const bs::CutItem &b) { return a.head != b.head ? a.head < b.head : a.tile < b.tile; };
            std::vector<bs::CutItem> have = sp.cut;
            std::sort(have.begin(), have.end(), less);
            std::sort(cut.begin(), cut.end(), less);
            if (have.size() != cut.size() || std::find(slot_used.begin(), slot_used.end(), 0) != slot_used.end()) return BS_EINVAL;
            for (size_t i = 0; i < cut.size(); ++i)
                if (have[i].head != cut[i].head || have[i].tile != cut[i].tile || have[i].first_slot != cut[i].first_slot ||
                    have[i].n_parts_item != cut[i].n_parts_item) return BS_EINVAL;
        }
        if (n_parts) *n_parts = (int64_t)sp.parts.size();
        if (n_cut_units) *n_cut_units = cut_units;
        if (n_queued) *n_queued = sp.share_off.empty() ? 0 : sp.queue_off[8] - sp.queue_off[0];
    } catch (const std::bad_alloc &) {
        return BS_ENOMEM;
    }
    return BS_OK;
}

extern "C" void bs_tilemap_destroy(bs_tilemap *tm)
{
    if (!tm) return;
    if (tm->dev && tm->dev_free) tm->dev_free(tm->dev);
    delete tm;
}

extern "C" int bs_tilemap_dims(const bs_tilemap *tm, int32_t *seq_len, int32_t *n_q_tiles,
                               int32_t *n_k_tiles, int32_t *n_q_heads)
{
    if (!tm) return BS_EINVAL;
    if (seq_len) *seq_len = tm->L;
    if (n_q_tiles) *n_q_tiles = tm->M;
    if (n_k_tiles) *n_k_tiles = tm->N;
    if (n_q_heads) *n_q_heads = tm->n_q_heads;
    return BS_OK;
}

extern "C" int bs_tilemap_row_order(const bs_tilemap *tm, int32_t *rows)
{
    if (!tm || !rows) return BS_EINVAL;
    std::vector<std::pair<int32_t, int32_t>> runs;
    try {
        for (int32_t m = 0; m < tm->M; ++m) {
            int32_t *r = rows + (size_t)m * tm->bm, *end = r + tm->bm;
            tm->geo.tile_runs(m, runs);
            for (const auto &x : runs)
                for (int32_t t = x.first; t < x.second; ++t) *r++ = t;
            std::fill(r, end, -1);
        }
    } catch (const std::bad_alloc &) {
        return BS_ENOMEM;
    }
    return BS_OK;
}

extern "C" int bs_tilemap_layout(const bs_tilemap *tm, int32_t *regrouped, int32_t *packed, int32_t *intra_compact)
{
    if (!tm) return BS_EINVAL;
    if (regrouped) *regrouped = tm->regrouped;
    if (packed) *packed = tm->packed;
    if (intra_compact) {
        try {
            published(tm, BS_INTRA);
        } catch (const std::bad_alloc &) {
            return BS_ENOMEM;
        }
        *intra_compact = tm->intra_compact;
    }
    return BS_OK;
}

extern "C" int bs_tilemap_key_order(const bs_tilemap *tm, int32_t *keys, int32_t *n_prompt_tiles)
{
    if (!tm) return BS_EINVAL;
    if (keys) {
        const int64_t n_slots = (int64_t)tm->N0 * tm->bn, n_compact = (int64_t)(tm->N - tm->N0) * tm->bn;
        for (int64_t s = 0; s < n_slots; ++s) keys[s] = s < tm->L ? (int32_t)s : -1;
        const int32_t n_free = tm->geo.n_free(tm->L);
        for (int64_t s = 0; s < n_compact; ++s) keys[n_slots + s] = s < n_free ? tm->geo.free_position((int32_t)s) : -1;
    }
    if (n_prompt_tiles) *n_prompt_tiles = tm->N0;
    return BS_OK;
}

extern "C" int bs_tilemap_tile_states(const bs_tilemap *tm, int32_t cls, int32_t q_tile_begin,
                                      int32_t q_tile_count, uint8_t *states)
{
    if (!tm || !states || cls < 0 || cls > 3 || q_tile_begin < 0 || q_tile_count < 0 ||
        (int64_t)q_tile_begin + q_tile_count > tm->M)
        return BS_EINVAL;
    try {
        const ClassLists &cl = published(tm, cls);
        std::vector<uint8_t> row(tm->N);
        for (int32_t r = 0; r < q_tile_count; ++r) {
            expand_states(cl, q_tile_begin + r, row);
            std::memcpy(states + (size_t)r * tm->N, row.data(), row.size());
        }
    } catch (const std::bad_alloc &) {
        return BS_ENOMEM;
    }
    return BS_OK;
}

extern "C" int bs_tilemap_walked(const bs_tilemap *tm, int32_t cls, int32_t q_tile, int32_t *n_tiles, uint8_t *states,
                                 int32_t *keys, int32_t *compact)
{
    if (!tm || cls < 0 || cls > 3 || q_tile < 0 || q_tile >= tm->M) return BS_EINVAL;
    const ClassLists &cl = tm->walked(cls);
    if (n_tiles) *n_tiles = tm->n_tiles;
    if (compact) *compact = cl.compact[q_tile];
    try {
        if (states) {
            std::vector<uint8_t> row(tm->n_tiles);
            expand_states(cl, q_tile, row);
            std::memcpy(states, row.data(), row.size());
        }
        if (keys) {
            const bs::PromptGeometry &P = tm->geo;
            const int64_t bn = tm->bn, n_free = P.n_free(tm->L), n_text = P.n_text(tm->L);
            for (int64_t s = 0; s < tm->n_tiles * bn; ++s) {
                const int64_t f = s - tm->N0 * bn, t = s - tm->text_tile0 * bn;
                if (f < 0) keys[s] = s < tm->L ? (int32_t)s : -1;
                else if (t < 0) keys[s] = f < n_free ? P.free_position((int32_t)f) : -1;
                else keys[s] = t < n_text ? P.text_position((int32_t)t) : -1;
            }
        }
    } catch (const std::bad_alloc &) {
        return BS_ENOMEM;
    }
    return BS_OK;
}

extern "C" int bs_tilemap_stats(const bs_tilemap *tm, int32_t cls, int64_t *visited, int64_t *full,
                                int64_t *partial, int64_t *allowed_pairs, int64_t *empty_rows,
                                int64_t *n_ranges)
{
    if (!tm || cls < 0 || cls > 3) return BS_EINVAL;
    if (allowed_pairs || empty_rows) {   // counted when first asked for; the lists do not need them
        std::lock_guard<std::mutex> lock(tm->lists_mutex);
        if (!tm->counted) count_pairs(tm->geo, tm->allowed_pairs, tm->empty_rows);
        tm->counted = true;
    }
    if (allowed_pairs) *allowed_pairs = tm->allowed_pairs[cls];
    if (empty_rows) *empty_rows = tm->empty_rows[cls];
    if (!visited && !full && !partial && !n_ranges) return BS_OK;
    try {
        const ClassLists &cl = published(tm, cls);
        if (visited) *visited = cl.visited;
        if (full) *full = cl.full;
        if (partial) *partial = cl.partial;
        if (n_ranges) *n_ranges = (int64_t)cl.ranges.size();
    } catch (const std::bad_alloc &) {
        return BS_ENOMEM;
    }
    return BS_OK;
}

extern "C" const char *bs_strerror(int code)
{
    switch (code) {
        case BS_OK: return "ok";
        case BS_EINVAL: return "invalid argument";
        case BS_EUNSUPPORTED: return "unsupported tile size, head_dim or dtype";
        case BS_ENOMEM: return "out of memory";
        case BS_EHIP: return "HIP runtime error";
        default: return "unknown error";
    }
}
