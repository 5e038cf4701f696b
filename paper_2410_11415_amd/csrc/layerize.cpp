// Host-side layerization and tensorization (paper Section 3.1 Eq. 2, Section 3.2, Alg. 2, Alg. 3).
#include "layerize.h"

#include <algorithm>
#include <climits>
#include <cmath>
#include <numeric>
#include <unordered_map>

namespace klay {

namespace {
// task size bounds (entries per wave task); overridable at compile time for tuning
#ifndef KLAY_TASK_MIN
#define KLAY_TASK_MIN 8
#endif
#ifndef KLAY_TASK_MAX
#define KLAY_TASK_MAX 32
#endif
#ifndef KLAY_TASK_DIV
#define KLAY_TASK_DIV 32768
#endif
constexpr int64_t kLatencyBoundEntries = 200000;     // see make_pass_plan
constexpr int64_t kTaskMin = KLAY_TASK_MIN, kTaskMax = KLAY_TASK_MAX, kTaskDiv = KLAY_TASK_DIV;
// Of the streaming kernel, whose waves read ahead: what they work on at one time is smaller and more of it is read a second time from the L2
// (3e6 nodes at B = 256, training step with at most 64 / 32 / 16 entries 3550 / 3538 / 3516 us).
constexpr int64_t kStreamTaskMax = 16;
// The persistent kernels' rows of more parents than this come first in their layer.  (8, 16, 64 and no such limit measured on
// 13 training steps: within 2%, 48 layers of 43000 nodes at B = 4 123.1 / 123.6 / 124.0 / 124.5 us)
constexpr int32_t kManyParents = 16;
enum : uint8_t { T_LIT = 0, T_AND = 1, T_OR = 2, T_TRUE = 3, T_FALSE = 4 };
constexpr int ST_OK = 0, ST_INVAL = 1, ST_CYCLE = 2;

// Segment length for a split row of k sources: about sqrt(k), so that the segment pass and the combine
// pass both see rows of that length, but at most kMaxSegment: a wave walks a segment 8 entries at a time
// and the launch lasts as long as the longest walk, while the combine pass gives a row with many partial
// rows a whole workgroup (combine_kernel).
constexpr int64_t kMaxSegment = 24;      // measured: 24 beats 12, 16, 20, 32, 48 and 64 on the power-law and the headline workload
int32_t segment_len(int64_t k, const Options& opt) {
    int64_t s = std::min<int64_t>(kMaxSegment, (int64_t)std::ceil(std::sqrt((double)k)));
    return (int32_t)std::max<int64_t>(s, std::max(1, opt.min_segment));
}
int64_t task_target(int64_t entries) { return std::min<int64_t>(kTaskMax, std::max<int64_t>(kTaskMin, entries / kTaskDiv)); }

// tasks over the rows r_begin .. r_end: close a task once it holds `target` entries (or 64 rows)
int32_t cut_tasks(const std::vector<int32_t>& ptr, int64_t r_begin, int64_t r_end, std::vector<int32_t>& tasks) {
    const int64_t target = task_target(ptr[(size_t)r_end] - ptr[(size_t)r_begin]);
    tasks.clear();
    int64_t r = r_begin;
    while (r < r_end) {
        tasks.push_back((int32_t)r);
        tasks.push_back(ptr[(size_t)r]);
        int64_t r1 = r;
        while (r1 < r_end && r1 - r < 64 && ptr[(size_t)r1] - ptr[(size_t)r] < target) ++r1;
        r = r1;
    }
    const int32_t count = (int32_t)(tasks.size() / 2);
    tasks.push_back((int32_t)r_end);
    tasks.push_back(ptr[(size_t)r_end]);
    return count;
}
}  // namespace

void make_pass_plan(int64_t n, const int32_t* ptr, const int32_t* idx_in, const Options& opt, PassPlan& out,
                    const uint32_t* flags_in, const uint32_t* row_bits, const uint8_t* skip) {
    // rows to leave out become empty rows of a CSR of their own, then one kSkipRow entry each, like split rows
    std::vector<int32_t> kept_ptr, kept_idx;
    std::vector<uint32_t> kept_flags;
    const int32_t* idx = idx_in;
    const uint32_t* flags = flags_in;
    if (skip) {
        kept_ptr.resize((size_t)n + 1);
        kept_ptr[0] = 0;
        for (int64_t r = 0; r < n; ++r) {
            if (!skip[(size_t)r])
                for (int32_t j = ptr[r]; j < ptr[r + 1]; ++j) {
                    kept_idx.push_back(idx_in[j]);
                    if (flags_in) kept_flags.push_back(flags_in[j]);
                }
            kept_ptr[(size_t)r + 1] = (int32_t)kept_idx.size();
        }
        ptr = kept_ptr.data();
        idx = kept_idx.data();
        if (flags_in) flags = kept_flags.data();
    }
    auto row_flag = [&](int64_t r) -> uint32_t { return row_bits && ((row_bits[(size_t)r >> 5] >> (r & 31)) & 1u) ? kRowFlag : 0u; };
    const int64_t e = ptr[n];
    out = PassPlan();
    if (flags)
        for (int64_t j = 0; j < e && !out.has_weighted; ++j) out.has_weighted = (flags[j] & kWeightedEdge) != 0;
    out.n_main = (int32_t)n;
    out.edges = e;
    int32_t heavy = std::max(1, opt.heavy_fan);
    {
        // A launch over the unsplit rows of a small pass lasts as long as its longest rows (a wave walks a row
        // 8 entries at a time).  Where rows are split anyway (so a lower threshold adds no launch), the unsplit
        // rows are few (the launch is bound by latency, not by what it moves) and rows longer than half the
        // threshold hold a tenth or more of their entries (power-law fan-ins), split from half the threshold on.
        // Measured at B = 64 on the two power-law workloads: 0.69 -> 0.64 ms and 0.75 -> 0.71 ms; the layered
        // workloads are 2-4% slower when every pass uses the lower threshold.
        const int32_t half = std::max(1, heavy / 2);
        int64_t light = 0, mid = 0;
        bool any_heavy = false;
        for (int64_t r = 0; r < n; ++r) {
            const int64_t k = ptr[r + 1] - ptr[r];
            if (k <= heavy) light += k;
            else any_heavy = true;
            if (k > half && k <= heavy) mid += k;
        }
        if (any_heavy && light < kLatencyBoundEntries && mid * 10 > light) heavy = half;
    }
    int64_t n_seg = 0, n_heavy = 0, heavy_edges = 0;
    for (int64_t r = 0; r < n; ++r) {
        int64_t k = ptr[r + 1] - ptr[r];
        if (k > heavy) {
            int32_t s = segment_len(k, opt);
            n_seg += (k + s - 1) / s;
            ++n_heavy;
            heavy_edges += k;
        }
    }
    out.n_seg = (int32_t)n_seg;
    out.n_heavy = (int32_t)n_heavy;
    out.ptr.resize((size_t)(n + n_seg + 1));
    int64_t n_skip = 0;
    if (skip)
        for (int64_t r = 0; r < n; ++r) n_skip += skip[(size_t)r] != 0;
    out.idx.assign((size_t)(e - heavy_edges + n_heavy + n_skip + heavy_edges + kIdxPad), 0u);
    out.seg_owner.resize((size_t)n_seg);
    out.comb_ptr.resize((size_t)(n_heavy + 1));
    out.comb_row.resize((size_t)n_heavy);
    // main rows keep their order and their entries come first; a split row is one kSkipRow entry
    int32_t w = 0;
    for (int64_t r = 0; r < n; ++r) {
        out.ptr[(size_t)r] = w;
        int64_t k = ptr[r + 1] - ptr[r];
        if (skip && skip[(size_t)r]) {
            out.idx[(size_t)w++] = kSkipRow;
        } else if (k <= heavy) {
            for (int64_t j = ptr[r]; j < ptr[r + 1]; ++j) out.idx[(size_t)w++] = (uint32_t)idx[j] | (flags ? flags[j] : 0u);
            if (k > 0) out.idx[(size_t)w - 1] |= kLastEdge | row_flag(r);
        } else {
            out.idx[(size_t)w++] = kSkipRow;
        }
    }
    out.ptr[(size_t)n] = w;
    out.n_tasks = cut_tasks(out.ptr, 0, n, out.tasks);
    if (n_heavy == 0) return;
    // Segments of all split rows, ordered by the first source they read: segments that read the
    // same stretch of source rows then run next to each other (and on the same XCD), so the
    // stretch is fetched once and served from L2 to the rest.
    struct Seg { int32_t owner, first_src; int64_t begin; int32_t len; };
    std::vector<Seg> segs;
    segs.reserve((size_t)n_seg);
    for (int64_t r = 0; r < n; ++r) {
        int64_t k = ptr[r + 1] - ptr[r];
        if (k <= heavy) continue;
        int32_t s = segment_len(k, opt);
        for (int64_t a = 0; a < k; a += s)
            segs.push_back(Seg{(int32_t)r, idx[ptr[r] + a], ptr[r] + a, (int32_t)std::min<int64_t>(s, k - a)});
    }
    std::stable_sort(segs.begin(), segs.end(), [](const Seg& a, const Seg& b) { return a.first_src < b.first_src; });
    // combine lists: scratch rows of each split row, in segment order
    std::vector<int32_t> per_owner_count((size_t)n, 0);
    for (const Seg& sg : segs) ++per_owner_count[(size_t)sg.owner];
    int64_t h = 0;
    std::vector<int32_t> owner_slot((size_t)n, -1);
    out.comb_ptr[0] = 0;
    // those of many partial rows first: they take a workgroup each (combine_kernel)
    for (const bool many : {true, false}) {
        for (int64_t r = 0; r < n; ++r)
            if (per_owner_count[(size_t)r] > 0 && (per_owner_count[(size_t)r] > kCombineWave) == many) {
                owner_slot[(size_t)r] = (int32_t)h;
                out.comb_row[(size_t)h] = (int32_t)r;
                out.comb_ptr[(size_t)h + 1] = out.comb_ptr[(size_t)h] + per_owner_count[(size_t)r];
                ++h;
            }
        if (many) out.n_comb_many = (int32_t)h;
    }
    out.comb_idx.assign((size_t)n_seg + kIdxPad, 0u);
    std::vector<int32_t> fill(out.comb_ptr.begin(), out.comb_ptr.end() - 1);
    for (size_t sidx = 0; sidx < segs.size(); ++sidx) {
        const Seg& sg = segs[sidx];
        for (int64_t j = sg.begin; j < sg.begin + sg.len; ++j) out.idx[(size_t)w++] = (uint32_t)idx[j] | (flags ? flags[j] : 0u);
        out.idx[(size_t)w - 1] |= kLastEdge;
        out.seg_owner[sidx] = sg.owner;
        out.ptr[(size_t)n + sidx + 1] = w;
        out.comb_idx[(size_t)fill[(size_t)owner_slot[(size_t)sg.owner]]++] = (uint32_t)sidx;
    }
    for (int64_t hh = 0; hh < n_heavy; ++hh)
        out.comb_idx[(size_t)out.comb_ptr[(size_t)hh + 1] - 1] |= row_flag(out.comb_row[(size_t)hh]);
    out.n_seg_tasks = cut_tasks(out.ptr, n, n + n_seg, out.seg_tasks);
}

std::vector<int32_t> stream_tasks(const PassPlan& p, int64_t from, int64_t to) {
    const int64_t target = std::min(kStreamTaskMax, task_target(p.ptr[(size_t)to] - p.ptr[(size_t)from]));
    std::vector<int32_t> tasks;
    auto skipped = [&](int64_t r) { return p.ptr[(size_t)r + 1] == p.ptr[(size_t)r] + 1 && p.idx[(size_t)p.ptr[(size_t)r]] == kSkipRow; };
    for (int64_t r = from; r < to;) {
        if (skipped(r)) { ++r; continue; }
        int64_t end = r;
        while (end < to && end - r < 64 && p.ptr[(size_t)end] - p.ptr[(size_t)r] < target && !skipped(end)) ++end;
        for (int64_t x : {r, (int64_t)p.ptr[(size_t)r], end, (int64_t)p.ptr[(size_t)end]}) tasks.push_back((int32_t)x);
        for (int i = 0; i < kTaskWords - kTaskHead; ++i) tasks.push_back((int32_t)p.idx[(size_t)p.ptr[(size_t)r] + (size_t)i]);      // (padded)
        r = end;
    }
    return tasks;
}

void compact_pass(const PassPlan& in, PassPlan& out, std::vector<int32_t>& out_row, std::vector<int32_t>& entry_row) {
    out = in;
    out.ptr.assign(1, 0);
    out.idx.clear();
    out_row.clear();
    entry_row.clear();
    for (int32_t r = 0; r < in.n_main; ++r) {
        const int32_t from = in.ptr[(size_t)r], to = in.ptr[(size_t)r + 1];
        if (to == from + 1 && in.idx[(size_t)from] == kSkipRow) continue;
        out_row.push_back(r);
        out.idx.insert(out.idx.end(), in.idx.begin() + from, in.idx.begin() + to);
        entry_row.insert(entry_row.end(), (size_t)(to - from), r);
        out.ptr.push_back((int32_t)out.idx.size());
    }
    out.n_main = (int32_t)out_row.size();
    const int32_t shift = in.ptr[(size_t)in.n_main] - (int32_t)out.idx.size();
    out.idx.insert(out.idx.end(), in.idx.begin() + in.ptr[(size_t)in.n_main], in.idx.end());       // segments and padding
    for (int32_t i = 1; i <= in.n_seg; ++i) out.ptr.push_back(in.ptr[(size_t)in.n_main + (size_t)i] - shift);
    entry_row.insert(entry_row.end(), (size_t)kIdxPad, 0);
    out.tasks.clear();
    out.seg_tasks.clear();
    out.n_tasks = out.n_seg_tasks = 0;
}

void make_cols(int64_t n, const int32_t* ptr, const int32_t* idx, const uint32_t* flags, const uint32_t* row_bits,
               int waves, int pad, ColStep step, ColPlan& out) {
    out = ColPlan();
    // Cycles of a wave with 15 others beside it, fitted to the times of the waves of both sweeps of a circuit of 85000 nodes
    // (per wave and layer, 640 samples, to within 10%): a chunk of kind 0, 1, 2, a unit of kind 3 or 4, a line of it, a
    // step of its butterfly, and what a run costs before its first row.
    struct Cost { int64_t chunk[3], unit, line, fly, run; };
    static const Cost kCosts[4] = {{{120, 140, 195}, 600, 65, 5, 550}, {{200, 370, 380}, 300, 350, 60, 620},
                                   {{255, 335, 350}, 60, 470, 45, 790}, {{210, 360, 560}, 670, 890, 10, 540}};
    const Cost& cost = kCosts[step];
    struct Piece { int64_t row, rows, cost; int kind, k; int32_t blocks; };
    // longest[k][r]: the longest row among the 64 >> k rows from r on
    std::vector<int32_t> longest[7];
    longest[6].resize((size_t)n);
    for (int64_t r = 0; r < n; ++r) longest[6][(size_t)r] = ptr[r + 1] - ptr[r];
    for (int k = 5; k >= 0; --k) {
        longest[k] = longest[k + 1];
        const int64_t half = 64 >> (k + 1);
        for (int64_t r = 0; r + half < n; ++r) longest[k][(size_t)r] = std::max(longest[k][(size_t)r], longest[k + 1][(size_t)(r + half)]);
    }
    // cheapest cut, then again without pieces that take longer than a wave's share of it
    std::vector<int64_t> best((size_t)n + 1, 0);
    std::vector<Piece> pick((size_t)n);
    int64_t cap = INT64_MAX;
    for (int turn = 0; turn < 2; ++turn) {
        for (int64_t r = n - 1; r >= 0; --r) {
            Piece b{}, least{};
            int64_t total = INT64_MAX;
            least.cost = INT64_MAX;
            auto consider = [&](int kind, int k, int32_t blocks, int64_t cost) {
                const Piece u{r, std::min<int64_t>(64 >> k, n - r), cost, kind, k, blocks};
                if (cost < least.cost) least = u;
                if (cost <= cap && cost + best[(size_t)(r + u.rows)] < total) { total = cost + best[(size_t)(r + u.rows)]; b = u; }
            };
            const int32_t most = longest[0][(size_t)r];
            if (most <= 4) {
                const int kind = most <= 1 ? 0 : most <= 2 ? 1 : 2;
                consider(kind, 0, 1, cost.chunk[kind]);
            }
            for (int k = 0; k <= 6; ++k) {
                const int32_t e = std::max(1, (longest[k][(size_t)r] + (1 << k) - 1) >> k), blocks = (e + 15) / 16;
                if (blocks > kColBlocksMax) continue;
                consider(e <= 8 ? 4 : 3, k, blocks, cost.unit + (e + 7) / 8 * cost.line + k * cost.fly);
            }
            if (total == INT64_MAX) { b = least; total = b.cost + best[(size_t)(r + b.rows)]; }
            best[(size_t)r] = total;
            pick[(size_t)r] = b;
        }
        cap = std::max<int64_t>(best[0] / waves, cost.unit + cost.line + 6 * cost.fly);
    }
    std::vector<Piece> pieces;
    for (int64_t r = 0; r < n; r += pick[(size_t)r].rows) pieces.push_back(pick[(size_t)r]);
    // contiguous shares: the smallest bound (in steps of a thirty-second) under which they number at most `waves`; a share
    // pays for each of its runs
    auto joins = [](const Piece& a, const Piece& b) { return a.kind == b.kind && a.k == b.k && a.blocks == b.blocks; };
    auto share_end = [&](size_t from, int64_t bound) {
        int64_t load = 0;
        size_t i = from;
        for (; i < pieces.size(); ++i) {
            const int64_t more = pieces[i].cost + (i > from && joins(pieces[i - 1], pieces[i]) ? 0 : cost.run);
            if (i > from && load + more > bound) break;
            load += more;
        }
        return i;
    };
    int64_t bound = best[0] / waves + 1;
    for (const Piece& u : pieces) bound = std::max(bound, u.cost + cost.run);
    for (;; bound += bound / 32 + 1) {
        size_t at = 0;
        int used = 0;
        for (; at < pieces.size() && used < waves; ++used) at = share_end(at, bound);
        if (at == pieces.size()) break;
    }
    out.share = bound;
    const uint32_t pads = (uint32_t)pad | (uint32_t)pad << 16;
    size_t next = 0;
    for (int w = 0; w < kColWaves; ++w) {
        out.block_at[w] = (int32_t)(out.blocks.size() / kBlockWords);
        out.table_at[w] = (int32_t)(out.tables.size() / (kDescTable * kDescWords));
        const size_t end = share_end(next, bound);
        int in_table = 0;
        auto describe = [&](uint32_t a, uint32_t b) {
            out.tables.push_back(a);
            out.tables.push_back(b);
            ++in_table;
        };
        while (next < end) {
            // the longest run of pieces that go on as the first one does
            const Piece& u = pieces[next];
            size_t stop = next + 1;
            int64_t rows = u.rows;
            while (stop < end && joins(u, pieces[stop])) rows += pieces[stop++].rows;
            if (in_table == kDescTable - 1) { describe(1u, 0u); in_table = 0; }
            describe((uint32_t)(kColSlots + u.row) | (uint32_t)u.blocks << 15, (uint32_t)rows | (uint32_t)u.k << 16 | (uint32_t)u.kind << 20);
            const size_t at = out.blocks.size();
            const int64_t per_block = u.kind < 3 ? 1024 >> u.kind : 64 >> u.k;
            out.blocks.resize(at + (size_t)((rows + per_block - 1) / per_block * u.blocks) * kBlockWords, pads);
            // entry e (0 .. 15) of a lane in block i of the run
            auto put = [&](int64_t i, int lane, int e, uint32_t entry) {
                uint32_t& word = out.blocks[at + (size_t)i * kBlockWords + (size_t)(e / 8) * kLineWords + (size_t)lane * 4 + (size_t)((e & 7) / 2)];
                word = (e & 1) ? (word & 0xFFFFu) | entry << 16 : (word & 0xFFFF0000u) | entry;
            };
            auto entry_of = [&](int64_t r, int64_t j) -> uint32_t {       // entry j of row r, or padding
                const bool flagged = row_bits && ((row_bits[(size_t)r >> 5] >> (r & 31)) & 1u);
                uint32_t x = (uint32_t)pad;
                if (ptr[r] + j < ptr[r + 1])
                    x = (uint32_t)(kColSlots + idx[ptr[r] + j]) | (flags && (flags[ptr[r] + j] & kWeightedEdge) ? 0x8000u : 0u);
                return flagged ? x | 0x8000u : x;
            };
            for (int64_t r = 0; r < rows; ++r) {
                if (u.kind < 3) {
                    const int64_t chunk = r / 64;
                    for (int e = 0; e < (1 << u.kind); ++e)
                        put(r / per_block, (int)(r & 63), (int)((chunk << u.kind) & 15) + e, entry_of(u.row + r, e));
                } else {
                    const int per_line = u.kind == 4 ? 8 : 16;
                    for (int sub = 0; sub < (1 << u.k); ++sub)
                        for (int64_t e = 0; e < (int64_t)per_line * u.blocks; ++e)
                            put(r / per_block * u.blocks + e / per_line, (int)((r % per_block) << u.k) + sub, (int)(e % per_line),
                                entry_of(u.row + r, sub + (e << u.k)));
                }
            }
            next = stop;
        }
        describe(0u, 0u);
        while (out.tables.size() % (kDescTable * kDescWords)) out.tables.push_back(0u);
    }
    out.block_at[kColWaves] = (int32_t)(out.blocks.size() / kBlockWords);
    out.table_at[kColWaves] = (int32_t)(out.tables.size() / (kDescTable * kDescWords));
    make_units(n, ptr, idx, flags, row_bits, pad, kNarrowUnits, out.units);
}

void make_units(int64_t n, const int32_t* ptr, const int32_t* idx, const uint32_t* flags, const uint32_t* row_bits, int pad, int most,
                std::vector<uint32_t>& units) {
    units.clear();
    // rows by class: 2^k lanes, from the most down to one, then the short ones
    std::vector<int32_t> by_class[8];
    int64_t lanes = 0;
    for (int64_t r = 0; r < n; ++r) {
        const int64_t fan = ptr[r + 1] - ptr[r];
        int k = 0;
        while (((int64_t)kUnitEntries << k) < fan) ++k;
        lanes += (int64_t)1 << std::min(k, 6);
        if (k > 6 || lanes > (int64_t)most * 64) return;
        by_class[fan <= kUnitEntries / 2 ? 7 : 6 - k].push_back((int32_t)r);
    }
    units.resize((size_t)((lanes + 63) / 64) * kUnitWords);
    for (size_t i = 0; i < units.size(); ++i) units[i] = i % 4 ? (uint32_t)pad | (uint32_t)pad << 16 : (uint32_t)kUnitIdleSlot;
    int64_t at = 0;
    for (int c = 0; c < 8; ++c)
        for (int32_t r : by_class[c]) {
            const int k = c < 7 ? 6 - c : 0;
            const bool flagged = row_bits && ((row_bits[(size_t)r >> 5] >> (r & 31)) & 1u);
            for (int64_t sub = 0; sub < (int64_t)1 << k; ++sub) {
                uint32_t* lane = units.data() + (size_t)(at + sub) * 4;
                lane[0] = (uint32_t)(kColSlots + r) | (uint32_t)k << kUnitLanesAt | (flagged ? kUnitRow : 0u);
                for (int64_t i = 0; i < kUnitEntries; ++i) {
                    const int64_t j = ptr[r] + sub + (i << k);
                    if (j >= ptr[r + 1]) break;
                    const uint32_t entry = (uint32_t)(kColSlots + idx[j]) | (flags && (flags[j] & kWeightedEdge) ? 0x8000u : 0u);
                    uint32_t& word = lane[1 + i / 2];
                    word = i & 1 ? (word & 0xFFFFu) | entry << 16 : (word & 0xFFFF0000u) | entry;
                }
            }
            // (classes in falling order keep a row's lanes together and aligned)
            if (c == 7 && at % 64 == 0) units[(size_t)at * 4] |= kUnitShort;
            at += (int64_t)1 << k;
        }
}

int layerize(int32_t V, int64_t N, const uint8_t* node_type, const int32_t* node_lit,
             const int64_t* child_ptr, const int32_t* child_idx_in, int32_t R, const int32_t* roots_in,
             const Options& opt, CircuitPlan& plan, std::string& err) {
    plan = CircuitPlan();
    const int32_t* child_idx = child_idx_in;
    const int32_t* roots = roots_in;
    // ---------------------------------------------------------------- validation
    if (V < 0 || N <= 0 || R <= 0 || !node_type || !node_lit || !child_ptr || !roots) {
        err = "klay_build: null array or non-positive size";
        return ST_INVAL;
    }
    if (N >= INT32_MAX) { err = "klay_build: more than 2^31-1 nodes"; return ST_INVAL; }
    if (child_ptr[0] != 0) { err = "klay_build: child_ptr[0] must be 0"; return ST_INVAL; }
    for (int64_t i = 0; i < N; ++i)
        if (child_ptr[i + 1] < child_ptr[i]) { err = "klay_build: child_ptr is not monotone"; return ST_INVAL; }
    const int64_t E = child_ptr[N];
    if (E > 0 && !child_idx) { err = "klay_build: child_idx is null"; return ST_INVAL; }
    for (int64_t i = 0; i < N; ++i) {
        const int64_t k = child_ptr[i + 1] - child_ptr[i];
        switch (node_type[i]) {
        case T_LIT: {
            int64_t l = node_lit[i];
            if (l == 0 || std::llabs(l) > V) {
                err = "klay_build: literal of node " + std::to_string(i) + " out of range";
                return ST_INVAL;
            }
        }   // fallthrough
        case T_TRUE:
        case T_FALSE:
            if (k != 0) { err = "klay_build: leaf node " + std::to_string(i) + " has children"; return ST_INVAL; }
            break;
        case T_AND:
        case T_OR:
            if (k == 0) { err = "klay_build: gate " + std::to_string(i) + " has no children"; return ST_INVAL; }
            break;
        default:
            err = "klay_build: unknown node type at node " + std::to_string(i);
            return ST_INVAL;
        }
    }
    for (int64_t j = 0; j < E; ++j)
        if (child_idx[j] < 0 || child_idx[j] >= N) { err = "klay_build: child index out of range"; return ST_INVAL; }
    for (int32_t r = 0; r < R; ++r)
        if (roots[r] < 0 || roots[r] >= N) { err = "klay_build: root index out of range"; return ST_INVAL; }

    // Leaves that carry the same literal (or the same constant) are one node: every reference is
    // redirected to the first of them (the leaf case of the node identification of Section 3.2).
    std::vector<int32_t> cidx((size_t)E), croots((size_t)R);
    {
        std::vector<int32_t> first_lit((size_t)2 * V + 2, -1), canon((size_t)N);
        for (int64_t i = 0; i < N; ++i) {
            canon[(size_t)i] = (int32_t)i;
            int64_t slot = -1;
            if (node_type[i] == T_LIT) slot = 2 * (std::llabs((int64_t)node_lit[i]) - 1) + (node_lit[i] < 0 ? 1 : 0);
            else if (node_type[i] == T_TRUE) slot = 2 * (int64_t)V;
            else if (node_type[i] == T_FALSE) slot = 2 * (int64_t)V + 1;
            if (slot >= 0) {
                if (first_lit[(size_t)slot] < 0) first_lit[(size_t)slot] = (int32_t)i;
                canon[(size_t)i] = first_lit[(size_t)slot];
            }
        }
        for (int64_t j = 0; j < E; ++j) cidx[(size_t)j] = canon[(size_t)child_idx[j]];
        for (int32_t r = 0; r < R; ++r) croots[(size_t)r] = canon[(size_t)roots[r]];
        child_idx = cidx.data();
        roots = croots.data();
    }

    // ---------------------------------------------------------------- parents of every node
    std::vector<int64_t> par_ptr((size_t)N + 1, 0);
    for (int64_t j = 0; j < E; ++j) ++par_ptr[(size_t)child_idx[j] + 1];
    for (int64_t i = 0; i < N; ++i) par_ptr[(size_t)i + 1] += par_ptr[(size_t)i];
    std::vector<int32_t> par_idx((size_t)E);
    {
        std::vector<int64_t> fill(par_ptr.begin(), par_ptr.end() - 1);
        for (int64_t i = 0; i < N; ++i)
            for (int64_t j = child_ptr[i]; j < child_ptr[i + 1]; ++j) par_idx[(size_t)fill[(size_t)child_idx[j]]++] = (int32_t)i;
    }

    // ---------------------------------------------------------------- heights, children first (Eq. 2)
    // h = 0 for leaves, 1 + max over children otherwise; a gate whose parity disagrees with its
    // type (AND must sit on an odd layer, OR on an even one) is lifted by one layer.
    std::vector<int32_t> h((size_t)N, 0);
    std::vector<int32_t> topo;                  // every node, children before parents
    topo.reserve((size_t)N);
    {
        std::vector<int64_t> pending((size_t)N);
        std::vector<int32_t> ready;
        ready.reserve((size_t)N);
        for (int64_t i = 0; i < N; ++i) {
            pending[(size_t)i] = child_ptr[i + 1] - child_ptr[i];
            if (pending[(size_t)i] == 0) ready.push_back((int32_t)i);
        }
        int64_t done = 0;
        while (!ready.empty()) {
            int32_t n = ready.back();
            ready.pop_back();
            ++done;
            topo.push_back(n);
            if (node_type[n] == T_AND || node_type[n] == T_OR) {
                int32_t m = 0;
                for (int64_t j = child_ptr[n]; j < child_ptr[n + 1]; ++j) m = std::max(m, h[(size_t)child_idx[j]]);
                int32_t hn = m + 1;
                const bool odd = (hn & 1) != 0;
                if ((node_type[n] == T_AND) != odd) ++hn;
                h[(size_t)n] = hn;
            }
            for (int64_t j = par_ptr[(size_t)n]; j < par_ptr[(size_t)n + 1]; ++j)
                if (--pending[(size_t)par_idx[(size_t)j]] == 0) ready.push_back(par_idx[(size_t)j]);
        }
        if (done != N) { err = "klay_build: the node graph has a cycle"; return ST_CYCLE; }
    }

    // ---------------------------------------------------------------- identical sub-circuits (Section 3.2, Eq. 3, Theorem 1)
    // Bottom-up, a gate is identified by its type and the multiset of its (already identified)
    // children.  The hash is a permutation-invariant sum of mixed child ids; on a hash hit the child
    // lists are compared, so a collision can never merge different gates.  Identical gates have
    // identical heights, so the layers computed above stay valid.
    if (!opt.no_merge) {
        auto mix = [](uint64_t x) {
            x += 0x9E3779B97F4A7C15ull;
            x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
            x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
            return x ^ (x >> 31);
        };
        std::vector<int32_t> rep((size_t)N);
        std::iota(rep.begin(), rep.end(), 0);
        std::unordered_map<uint64_t, int32_t> head;
        head.reserve((size_t)N);
        std::vector<int32_t> next_same((size_t)N, -1);
        for (int32_t n : topo) {
            if (node_type[n] != T_AND && node_type[n] != T_OR) continue;
            const int64_t a = child_ptr[n], b = child_ptr[n + 1];
            for (int64_t j = a; j < b; ++j) cidx[(size_t)j] = rep[(size_t)cidx[(size_t)j]];
            std::sort(cidx.begin() + a, cidx.begin() + b);
            uint64_t hsh = mix((uint64_t)node_type[n] * 0x51ED27ull + (uint64_t)(b - a));
            for (int64_t j = a; j < b; ++j) hsh += mix((uint64_t)cidx[(size_t)j]);
            auto it = head.find(hsh);
            int32_t found = -1;
            if (it != head.end()) {
                for (int32_t m = it->second; m >= 0; m = next_same[(size_t)m]) {
                    const int64_t ma = child_ptr[m], mb = child_ptr[m + 1];
                    if (node_type[m] == node_type[n] && mb - ma == b - a &&
                        std::equal(cidx.begin() + a, cidx.begin() + b, cidx.begin() + ma)) { found = m; break; }
                }
            }
            if (found >= 0) {
                rep[(size_t)n] = found;
                ++plan.num_merged;
            } else if (it != head.end()) {
                next_same[(size_t)n] = it->second;
                it->second = n;
            } else {
                head.emplace(hsh, n);
            }
        }
        for (int32_t r = 0; r < R; ++r) croots[(size_t)r] = rep[(size_t)croots[(size_t)r]];
    }

    // ---------------------------------------------------------------- reachability from the roots
    std::vector<uint8_t> reach((size_t)N, 0);
    {
        std::vector<int32_t> stack;
        for (int32_t r = 0; r < R; ++r)
            if (!reach[(size_t)roots[r]]) { reach[(size_t)roots[r]] = 1; stack.push_back(roots[r]); }
        while (!stack.empty()) {
            int32_t n = stack.back();
            stack.pop_back();
            for (int64_t j = child_ptr[n]; j < child_ptr[n + 1]; ++j) {
                int32_t c = child_idx[j];
                if (!reach[(size_t)c]) { reach[(size_t)c] = 1; stack.push_back(c); }
            }
        }
    }
    // A gate that is part of the circuit must not name the same input node twice (the children of a
    // gate are a set, Eq. 1).  Checked on the ids as given: two different leaf nodes that carry the same
    // literal, or two gates that turn out identical, are two children and count twice, as in Eq. 1.
    {
        std::vector<int32_t> stamp((size_t)N, -1);
        for (int64_t i = 0; i < N; ++i) {
            if (!reach[(size_t)i]) continue;
            for (int64_t j = child_ptr[i]; j < child_ptr[i + 1]; ++j) {
                const int32_t c = child_idx_in[j];
                if (stamp[(size_t)c] == (int32_t)i) { err = "klay_build: gate " + std::to_string(i) + " lists a child twice"; return ST_INVAL; }
                stamp[(size_t)c] = (int32_t)i;
            }
        }
    }
    int32_t L = 0;
    for (int32_t r = 0; r < R; ++r) L = std::max(L, h[(size_t)roots[r]]);

    // ---------------------------------------------------------------- unary chains (Section 3.1; one per (child, layer))
    // need[c] = highest layer at which a stand-in for c is read: parent height - 1, or L for roots.
    std::vector<int32_t> need(h);
    std::vector<int32_t> max_fan((size_t)L + 1, 0);       // largest fan-in among the gates of a layer
    for (int64_t p = 0; p < N; ++p) {
        if (!reach[(size_t)p]) continue;
        plan.dag_nodes++;
        plan.dag_edges += child_ptr[p + 1] - child_ptr[p];
        max_fan[(size_t)h[(size_t)p]] = (int32_t)std::max<int64_t>(max_fan[(size_t)h[(size_t)p]], child_ptr[p + 1] - child_ptr[p]);
        for (int64_t j = child_ptr[p]; j < child_ptr[p + 1]; ++j) {
            int32_t c = child_idx[j];
            need[(size_t)c] = std::max(need[(size_t)c], h[(size_t)p] - 1);
        }
    }
    for (int32_t r = 0; r < R; ++r) need[(size_t)roots[r]] = L;

    // Padding-free lower part (Options::alias_chains): the layers 1 .. B0 (B0 = plan.alias_top) hold no
    // stand-ins except that layer B0 is complete: it holds a stand-in for every node that a layer above
    // reads.  The edges of the layers up to B0 name the child's own row in the whole activation buffer,
    // wherever it lives; from layer B0 + 1 on every edge goes to the layer directly below, as in the
    // paper.  B0 is chosen so that the layers above it are exactly the narrow top of the circuit that the
    // persistent kernels can take (they need complete layers); B0 = 0 is the paper's layerization, B0 = L
    // has no chain nodes at all except the stand-ins that bring every root to the top layer.
    const int64_t rows_cap = opt.tail_rows_cap > 0 ? std::min<int64_t>(opt.tail_rows_cap, kTailRowsCap) : kTailRowsCap;
    int32_t B0 = 0, top_first = 0;
    {
        std::vector<int64_t> full((size_t)L + 1, 0);       // layer sizes with all chain nodes
        std::vector<int64_t> edges((size_t)L + 1, 0);      // and their edges
        for (int64_t c = 0; c < N; ++c)
            if (reach[(size_t)c]) {
                edges[(size_t)h[(size_t)c]] += child_ptr[c + 1] - child_ptr[c];
                for (int32_t l = h[(size_t)c]; l <= need[(size_t)c]; ++l) {
                    ++full[(size_t)l];
                    edges[(size_t)l] += l > h[(size_t)c];
                }
            }
        if (opt.alias_chains) {
            B0 = L;
            if (!opt.no_tail) {
                int32_t t = L + 1;
                while (t - 1 >= 1 && full[(size_t)t - 1] <= rows_cap && full[(size_t)t - 2] <= rows_cap &&
                       max_fan[(size_t)t - 1] <= kTailFanCap)
                    --t;
                if (L - t + 1 >= 2) B0 = t - 1;            // a persistent kernel takes two layers or more
                // further down rows are long (or a layer wide): the plan for those (TopPlan)
                t = L + 1;
                while (t - 1 >= 1 && full[(size_t)t - 1] <= rows_cap && full[(size_t)t - 2] <= rows_cap && edges[(size_t)t - 1] <= kTopEdges) --t;
                int64_t stand_ins = 0;                      // of leaves
                for (int64_t c = 0; c < N; ++c)
                    if (reach[(size_t)c] && h[(size_t)c] == 0) stand_ins += need[(size_t)c];
                if (t == 1 && stand_ins > kTopLeafStandIns) t = 2;
                if (L - t + 1 >= 2 && t <= B0) top_first = t;
            }
        }
    }
    plan.alias_top = B0;
    plan.alias = B0 > 0;
    // lowest level at which c has a stand-in (none if that is above need[c])
    auto lo = [&](int64_t c) { return std::max(h[(size_t)c] + 1, B0); };

    // Fused AND rows (see LayerPlan): AND nodes of the padding-free part whose value nothing has to read.
    std::vector<uint8_t> fused((size_t)N, 0);
    if (B0 > 0 && !opt.no_fusion) {
        // a row is split when it has more entries than heavy_fan, or than half of it (make_pass_plan): the rows that
        // read through fused rows stay at or below that, so that no group of entries is cut by a segment boundary
        const int64_t row_max = std::min<int64_t>(kFusedRowMax, std::max(1, opt.heavy_fan / 2));
        std::vector<uint8_t> cand((size_t)N, 0);
        for (int64_t c = 0; c < N; ++c) {
            if (!reach[(size_t)c] || !(h[(size_t)c] & 1) || h[(size_t)c] >= B0 || need[(size_t)c] >= B0) continue;
            const int64_t fi = child_ptr[c + 1] - child_ptr[c];
            int64_t gates = 0;
            for (int64_t j = child_ptr[c]; j < child_ptr[c + 1]; ++j) gates += h[(size_t)child_idx[j]] > 0;
            cand[(size_t)c] = fi >= 1 && gates <= 1 && fi <= row_max;
            // (a TopPlan from layer f on reads the nodes below f that are read from f - 1 or above: with fused rows that are read
            // from the next layer only, those are the ones of layer f - 1, see klay_forward)
            if (top_first > 0 && need[(size_t)c] >= top_first - 1 && need[(size_t)c] > h[(size_t)c]) cand[(size_t)c] = 0;
        }
        // every parent has to be an OR row that stays short when it reads the children of its fused children
        for (int64_t p = 0; p < N; ++p) {
            if (!reach[(size_t)p] || h[(size_t)p] == 0) continue;
            int64_t len = 0;
            bool any = false;
            for (int64_t j = child_ptr[p]; j < child_ptr[p + 1]; ++j) {
                const int32_t c = child_idx[j];
                any = any || (cand[(size_t)c] & 1);
                len += (cand[(size_t)c] & 1) ? child_ptr[c + 1] - child_ptr[c] : 1;
            }
            if (!any || ((h[(size_t)p] & 1) == 0 && len <= row_max)) continue;
            for (int64_t j = child_ptr[p]; j < child_ptr[p + 1]; ++j) cand[(size_t)child_idx[j]] |= 2;      // not through this parent
        }
        // In the layers that a TopPlan may take, fused rows are for the batches that leave them to the launches; there a layer has to be wide and
        // mostly fused.  (kTopFusedRows, kTopFusedShare; forward, us, no fused rows there / without the two limits / with: 41000 nodes in
        // 24 layers, fan-ins up to 400, B = 1300 276 / 290 / 273, B = 2500 386 / 364 / 363; 24000 in 16 layers, up to 100, B = 1300
        // 169 / 187 / 168; 58000 in 20 layers, up to 300, B = 1600 293 / 259 / 267; 51000 in 14 layers, up to 1952, 1 in 60 fused, B = 400
        // 176 / 180 / 176.)
        std::vector<int64_t> rows((size_t)L + 1, 0), rows_fused((size_t)L + 1, 0);
        for (int64_t c = 0; c < N; ++c)
            if (reach[(size_t)c]) {
                ++rows[(size_t)h[(size_t)c]];
                rows_fused[(size_t)h[(size_t)c]] += cand[(size_t)c] == 1;
            }
        for (int64_t c = 0; c < N; ++c) {
            if (cand[(size_t)c] != 1) continue;
            const size_t l = (size_t)h[(size_t)c];
            if (top_first > 0 && need[(size_t)c] >= top_first - 1 && (rows[l] < kTopFusedRows || rows_fused[l] * kTopFusedShare < rows[l])) continue;
            fused[(size_t)c] = 1;
            ++plan.num_fused;
        }
    }

    std::vector<int64_t> count((size_t)L + 1, 0);
    std::vector<int64_t> pad_base((size_t)N + 1, 0);
    for (int64_t c = 0; c < N; ++c) {
        pad_base[(size_t)c + 1] = pad_base[(size_t)c];
        if (!reach[(size_t)c]) continue;
        ++count[(size_t)h[(size_t)c]];
        const int32_t pads = std::max(0, need[(size_t)c] - lo(c) + 1);
        pad_base[(size_t)c + 1] += pads;
        for (int32_t l = lo(c); l <= need[(size_t)c]; ++l) ++count[(size_t)l];
    }
    plan.num_pad_nodes = pad_base[(size_t)N];
    for (int32_t l = 0; l <= L; ++l)
        if (count[(size_t)l] >= INT32_MAX) { err = "klay_build: a layer has more than 2^31-1 nodes"; return ST_INVAL; }

    // slot of every node within its layer before ordering: real nodes by id, then chain nodes by id
    std::vector<int32_t> pos_real((size_t)N, -1);
    std::vector<int32_t> pos_pad((size_t)plan.num_pad_nodes, -1);
    plan.layers.resize((size_t)L + 1);
    {
        std::vector<int64_t> fill((size_t)L + 1, 0);
        for (int32_t l = 0; l <= L; ++l) {
            plan.layers[(size_t)l].n = count[(size_t)l];
            plan.layers[(size_t)l].origin.resize((size_t)count[(size_t)l]);
            plan.layers[(size_t)l].is_pad.assign((size_t)count[(size_t)l], 0);
        }
        for (int64_t c = 0; c < N; ++c)
            if (reach[(size_t)c]) {
                int32_t l = h[(size_t)c];
                pos_real[(size_t)c] = (int32_t)fill[(size_t)l];
                plan.layers[(size_t)l].origin[(size_t)fill[(size_t)l]++] = (int32_t)c;
            }
        for (int64_t c = 0; c < N; ++c)
            if (reach[(size_t)c])
                for (int32_t l = lo(c); l <= need[(size_t)c]; ++l) {
                    pos_pad[(size_t)(pad_base[(size_t)c] + l - lo(c))] = (int32_t)fill[(size_t)l];
                    plan.layers[(size_t)l].origin[(size_t)fill[(size_t)l]] = (int32_t)c;
                    plan.layers[(size_t)l].is_pad[(size_t)fill[(size_t)l]++] = 1;
                }
    }
    plan.row0.assign((size_t)L + 2, 0);
    for (int32_t l = 0; l <= L; ++l) plan.row0[(size_t)l + 1] = plan.row0[(size_t)l] + count[(size_t)l];
    if (plan.row0[(size_t)L + 1] + R >= kMaxRows) { err = "klay_build: more than 2^29 rows"; return ST_INVAL; }
    // position, within layer `level`, of node c or of its stand-in there (c is present at that level)
    auto at = [&](int32_t c, int32_t level) -> int32_t {
        return level == h[(size_t)c] ? pos_real[(size_t)c] : pos_pad[(size_t)(pad_base[(size_t)c] + level - lo(c))];
    };
    // what an edge from layer level + 1 down to c holds: below B0 the row of c itself in the whole
    // activation buffer, from B0 on the position of c (or of its stand-in) in layer `level`
    auto src_at = [&](int32_t c, int32_t level) -> int32_t {
        if (level < B0) return (int32_t)(plan.row0[(size_t)h[(size_t)c]] + pos_real[(size_t)c]);
        return at(c, level);
    };
    // ordering key of a child: its position in the layer below, or (below the boundary layer) its relative
    // position within its own layer scaled to the width of the layer below
    auto child_key = [&](int32_t c, int32_t level) -> double {
        if (level >= B0) return (double)at(c, level);
        const int32_t hc = h[(size_t)c];
        return (double)pos_real[(size_t)c] / (double)std::max<int64_t>(1, count[(size_t)hc]) * (double)count[(size_t)level];
    };
    auto set_at = [&](int32_t c, int32_t level, int32_t p) {
        if (level == h[(size_t)c]) pos_real[(size_t)c] = p;
        else pos_pad[(size_t)(pad_base[(size_t)c] + level - lo(c))] = p;
    };

    // ---------------------------------------------------------------- node order within layers (Section 4: arbitrary)
    // Layer 0: by variable, positive literal first, then constants.  Higher layers: by the smallest
    // position among a node's children in the layer below (one bottom-up sweep; ties keep slot
    // order): every row of the layer below is then first read in storage order, a sequential
    // stream, and only the remaining reads of a row are scattered.  (Measured on the headline
    // circuit: 12% faster than input order, 2% faster than ordering by the mean child position.)
    // AND layers are then re-ordered by their first parent (see below).
    auto apply_order = [&](int32_t l, const std::vector<int32_t>& order /* new position -> old slot */) {
        LayerPlan& lay = plan.layers[(size_t)l];
        std::vector<int32_t> origin(lay.origin.size());
        std::vector<uint8_t> is_pad(lay.is_pad.size());
        for (size_t p = 0; p < order.size(); ++p) {
            origin[p] = lay.origin[(size_t)order[p]];
            is_pad[p] = lay.is_pad[(size_t)order[p]];
            set_at(origin[p], l, (int32_t)p);
        }
        lay.origin.swap(origin);
        lay.is_pad.swap(is_pad);
    };
    {
        LayerPlan& l0 = plan.layers[0];
        std::vector<int32_t> order((size_t)l0.n);
        std::iota(order.begin(), order.end(), 0);
        auto key = [&](int32_t slot) -> int64_t {
            int32_t c = l0.origin[(size_t)slot];
            if (node_type[c] == T_LIT) {
                int64_t lit = node_lit[c];
                return 2 * (std::llabs(lit) - 1) + (lit < 0 ? 1 : 0);
            }
            return 2 * (int64_t)V + (node_type[c] == T_TRUE ? 0 : 1);
        };
        std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return key(a) < key(b); });
        apply_order(0, order);
    }
    if (!opt.no_reorder) {
        auto order_by_children = [&](int32_t l) {
            LayerPlan& lay = plan.layers[(size_t)l];
            std::vector<double> key((size_t)lay.n);
            for (int64_t s = 0; s < lay.n; ++s) {
                int32_t c = lay.origin[(size_t)s];
                if (lay.is_pad[(size_t)s]) key[(size_t)s] = child_key(c, l - 1);
                else {
                    double acc = 1e300;
                    for (int64_t j = child_ptr[c]; j < child_ptr[c + 1]; ++j) acc = std::min(acc, child_key(child_idx[j], l - 1));
                    key[(size_t)s] = acc;
                }
            }
            std::vector<int32_t> order((size_t)lay.n);
            std::iota(order.begin(), order.end(), 0);
            std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return key[(size_t)a] < key[(size_t)b]; });
            if (lay.n <= rows_cap && l >= B0 && !opt.no_tail) {
                // A layer small enough for the persistent top-of-circuit kernels: there a thread walks a whole
                // row and a wave waits for its longest one, while locality is irrelevant (the layer sits in
                // LDS).  Group rows by fan-in (powers of two) and order each group by fan-out, so that the 64
                // rows of a wave have similar lengths in the forward and in the reverse sweep.  The few rows of
                // many parents come first, so that they do not stretch the chunks of the others.
                std::vector<int32_t> fan_in((size_t)lay.n), fan_out((size_t)lay.n, 0);
                for (int64_t s2 = 0; s2 < lay.n; ++s2) {
                    const int32_t c = lay.origin[(size_t)s2];
                    fan_in[(size_t)s2] = lay.is_pad[(size_t)s2] ? 1 : (int32_t)(child_ptr[c + 1] - child_ptr[c]);
                }
                if (l < L) {
                    const LayerPlan& up = plan.layers[(size_t)l + 1];
                    for (int64_t s2 = 0; s2 < up.n; ++s2) {
                        const int32_t c = up.origin[(size_t)s2];
                        if (up.is_pad[(size_t)s2]) ++fan_out[(size_t)at(c, l)];
                        else
                            for (int64_t j = child_ptr[c]; j < child_ptr[c + 1]; ++j) ++fan_out[(size_t)at(child_idx[j], l)];
                    }
                }
                auto bucket = [](int32_t k) { int b = 0; while ((1 << b) < k) ++b; return b; };
                std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) {
                    const bool ma = fan_out[(size_t)a] > kManyParents, mb = fan_out[(size_t)b] > kManyParents;
                    if (ma != mb) return ma;
                    const int ba = bucket(fan_in[(size_t)a]), bb = bucket(fan_in[(size_t)b]);
                    if (!ma && ba != bb) return ba > bb;
                    return fan_out[(size_t)a] > fan_out[(size_t)b];
                });
            }
            apply_order(l, order);
        };
        for (int32_t l = 1; l <= L; ++l) order_by_children(l);
        // Second sweep, from the top, over the AND layers only: a row moves next to the first of its
        // parents, so the children of an OR node sit together.  The reverse sweep of an OR layer reads two
        // rows per edge (adjoint and value of the parent) against one in every other pass, so that pass
        // gets the locality: its gathers of a parent's rows then hit in L2 for the siblings.  (Measured on
        // the headline circuit: 2.4% of the step; doing the same for the OR layers, or iterating the two
        // sweeps, gains nothing more.)
        auto order_by_parents = [&](int32_t l) {
            LayerPlan& lay = plan.layers[(size_t)l];
            if (lay.n <= rows_cap && !opt.no_tail) return;       // keep the fan-sorted order of small layers
            const LayerPlan& up = plan.layers[(size_t)l + 1];
            std::vector<int32_t> key((size_t)lay.n, INT32_MAX);
            for (int64_t p2 = 0; p2 < up.n; ++p2) {
                const int32_t c = up.origin[(size_t)p2];
                if (up.is_pad[(size_t)p2]) { int32_t& k2 = key[(size_t)at(c, l)]; k2 = std::min<int32_t>(k2, (int32_t)p2); }
                else
                    for (int64_t j = child_ptr[c]; j < child_ptr[c + 1]; ++j) {
                        int32_t& k2 = key[(size_t)at(child_idx[j], l)];
                        k2 = std::min<int32_t>(k2, (int32_t)p2);
                    }
            }
            std::vector<int32_t> order((size_t)lay.n);
            std::iota(order.begin(), order.end(), 0);
            std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return key[(size_t)a] < key[(size_t)b]; });
            apply_order(l, order);
        };
        // (layers from B0 on: their parents sit in the layer directly above)
        for (int32_t l = L - 1; l >= std::max(B0, 1); --l)
            if (l & 1) order_by_parents(l);
        if (B0 > 0) {
            // the same idea for the layers below B0, whose parents sit in any higher layer up to B0: one sweep
            // from the top keeps, per node, the smallest relative position among its parents seen so far
            std::vector<double> pkey((size_t)N, 2.0);
            for (int32_t l = B0; l >= 1; --l) {
                LayerPlan& lay = plan.layers[(size_t)l];
                if ((l & 1) && l < B0) {
                    std::vector<int32_t> order((size_t)lay.n);
                    std::iota(order.begin(), order.end(), 0);
                    std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) {
                        return pkey[(size_t)lay.origin[(size_t)a]] < pkey[(size_t)lay.origin[(size_t)b]];
                    });
                    apply_order(l, order);
                }
                for (int64_t s2 = 0; s2 < lay.n; ++s2) {
                    const int32_t c = lay.origin[(size_t)s2];
                    const double rel = ((double)s2 + 0.5) / (double)lay.n;
                    if (lay.is_pad[(size_t)s2]) { pkey[(size_t)c] = std::min(pkey[(size_t)c], rel); continue; }
                    for (int64_t j = child_ptr[c]; j < child_ptr[c + 1]; ++j) pkey[(size_t)child_idx[j]] = std::min(pkey[(size_t)child_idx[j]], rel);
                }
            }
        }
    }

    // the row of node x in the whole activation buffer (the padding-free part)
    auto own_row = [&](int32_t x) -> int32_t { return (int32_t)(plan.row0[(size_t)h[(size_t)x]] + pos_real[(size_t)x]); };

    // ---------------------------------------------------------------- index vectors per layer (Alg. 3), CSR by parent
    Options popt = opt;
    for (int32_t l = 1; l <= L; ++l) {
        LayerPlan& lay = plan.layers[(size_t)l];
        int64_t e = 0;
        for (int64_t p = 0; p < lay.n; ++p)
            e += lay.is_pad[(size_t)p] ? 1 : child_ptr[lay.origin[(size_t)p] + 1] - child_ptr[lay.origin[(size_t)p]];
        if (e + lay.n >= INT32_MAX - 64) { err = "klay_build: a layer has more than 2^31 edges"; return ST_INVAL; }
        lay.e = e;
        lay.row_ptr.resize((size_t)lay.n + 1);
        lay.child.resize((size_t)e);
        int32_t w = 0;
        for (int64_t p = 0; p < lay.n; ++p) {
            lay.row_ptr[(size_t)p] = w;
            int32_t c = lay.origin[(size_t)p];
            if (lay.is_pad[(size_t)p]) lay.child[(size_t)w++] = src_at(c, l - 1);
            else {
                const int32_t w0 = w;
                for (int64_t j = child_ptr[c]; j < child_ptr[c + 1]; ++j) lay.child[(size_t)w++] = src_at(child_idx[j], l - 1);
                std::sort(lay.child.begin() + w0, lay.child.begin() + w);
            }
            plan.max_fan_in = std::max<int64_t>(plan.max_fan_in, w - lay.row_ptr[(size_t)p]);
        }
        lay.row_ptr[(size_t)lay.n] = w;
        lay.multi.assign((size_t)(lay.n + 31) / 32, 0u);
        for (int64_t p = 0; p < lay.n; ++p)
            if (lay.row_ptr[(size_t)p + 1] - lay.row_ptr[(size_t)p] > 1) lay.multi[(size_t)p >> 5] |= 1u << (p & 31);
        make_pass_plan(lay.n, lay.row_ptr.data(), lay.child.data(), popt, lay.fwd);
        if ((l & 1) && l < B0 && plan.num_fused > 0) {
            std::vector<uint8_t> skip((size_t)lay.n, 0);
            for (int64_t p = 0; p < lay.n; ++p) {
                skip[(size_t)p] = fused[(size_t)lay.origin[(size_t)p]];
                lay.n_fused += skip[(size_t)p];
            }
            if (lay.n_fused > 0 && lay.n_fused < lay.n)
                make_pass_plan(lay.n, lay.row_ptr.data(), lay.child.data(), popt, lay.fwd_kept, nullptr, nullptr, skip.data());
        }
        if ((l & 1) == 0 && l <= B0 && plan.num_fused > 0) {
            // fwd2: every child of an OR row as a group of entries; a fused AND child is replaced by its children
            bool reads_fused = false;
            std::vector<int32_t> ptr2((size_t)lay.n + 1, 0), idx2;
            std::vector<uint32_t> flag2;
            idx2.reserve((size_t)e * 2);
            flag2.reserve((size_t)e * 2);
            std::vector<std::pair<int32_t, int32_t>> kids;       // (row, node) of a row's children, by row
            std::vector<int32_t> grp;
            for (int64_t p = 0; p < lay.n; ++p) {
                const int32_t c = lay.origin[(size_t)p];
                if (lay.is_pad[(size_t)p]) {
                    idx2.push_back(lay.child[(size_t)lay.row_ptr[(size_t)p]]);
                    flag2.push_back(kGroupEnd);
                } else {
                    kids.clear();
                    for (int64_t j = child_ptr[c]; j < child_ptr[c + 1]; ++j) kids.emplace_back(own_row(child_idx[j]), child_idx[j]);
                    std::sort(kids.begin(), kids.end());
                    for (const auto& kid : kids) {
                        if (!fused[(size_t)kid.second]) {
                            idx2.push_back(kid.first);
                            flag2.push_back(kGroupEnd);
                            continue;
                        }
                        reads_fused = true;
                        const int32_t a = kid.second;
                        grp.clear();
                        for (int64_t j = child_ptr[a]; j < child_ptr[a + 1]; ++j) grp.push_back(own_row(child_idx[j]));
                        std::sort(grp.begin(), grp.end());
                        for (size_t g = 0; g < grp.size(); ++g) {
                            idx2.push_back(grp[g]);
                            flag2.push_back(g + 1 == grp.size() ? kGroupEnd : 0u);
                        }
                    }
                }
                if (idx2.size() >= (size_t)INT32_MAX - 64) { err = "klay_build: a layer has more than 2^31 edges"; return ST_INVAL; }
                ptr2[(size_t)p + 1] = (int32_t)idx2.size();
            }
            if (reads_fused) {
                make_pass_plan(lay.n, ptr2.data(), idx2.data(), popt, lay.fwd2, flag2.data());
                plan.max_fwd_seg = std::max<int64_t>(plan.max_fwd_seg, lay.fwd2.n_seg);
            }
        }

        plan.num_edges += e;
        plan.num_split_rows += lay.fwd.n_heavy;
        plan.max_fwd_seg = std::max<int64_t>(plan.max_fwd_seg, lay.fwd.n_seg);
        if (l <= B0) continue;             // their reverse plans are built below, over the whole lower part

        // by child (for the reverse sweep): rows = nodes of layer l-1, sources = parents in layer l;
        // an edge is weighted when its parent is an OR node with more than one child
        const int64_t nc = plan.layers[(size_t)l - 1].n;
        std::vector<int32_t> cptr((size_t)nc + 1, 0), cpar((size_t)e);
        std::vector<uint32_t> cflag((size_t)e, 0u);
        for (int64_t j = 0; j < e; ++j) ++cptr[(size_t)lay.child[(size_t)j] + 1];
        for (int64_t i = 0; i < nc; ++i) {
            plan.max_fan_out = std::max<int64_t>(plan.max_fan_out, cptr[(size_t)i + 1]);
            cptr[(size_t)i + 1] += cptr[(size_t)i];
        }
        {
            std::vector<int32_t> fill(cptr.begin(), cptr.end() - 1);
            for (int64_t p = 0; p < lay.n; ++p)
                for (int32_t j = lay.row_ptr[(size_t)p]; j < lay.row_ptr[(size_t)p + 1]; ++j) {
                    const int32_t slot = fill[(size_t)lay.child[(size_t)j]]++;
                    cpar[(size_t)slot] = (int32_t)p;
                    if ((l & 1) == 0 && lay.row_ptr[(size_t)p + 1] - lay.row_ptr[(size_t)p] > 1) cflag[(size_t)slot] = kWeightedEdge;
                }
        }
        // the rows of this pass are the nodes of layer l - 1: below an AND layer they are OR nodes, and those
        // with more than one child are flagged (their adjoints are stored in the one-gather form)
        make_pass_plan(nc, cptr.data(), cpar.data(), popt, lay.bwd, cflag.data(),
                       (l & 1) && l >= 3 ? plan.layers[(size_t)l - 1].multi.data() : nullptr);
        if (!opt.no_tail && lay.n <= rows_cap && nc <= rows_cap) {
            int64_t fan_in = 0, fan_out = 0;
            for (int64_t i = 0; i < lay.n; ++i) fan_in = std::max<int64_t>(fan_in, lay.row_ptr[(size_t)i + 1] - lay.row_ptr[(size_t)i]);
            for (int64_t i = 0; i < nc; ++i) fan_out = std::max<int64_t>(fan_out, cptr[(size_t)i + 1] - cptr[(size_t)i]);
            if (fan_in <= kTailFanCap && fan_out <= kColRowEntries) {
                lay.tail_ok = true;
                const bool is_and = (l & 1) != 0;
                make_cols(lay.n, lay.row_ptr.data(), lay.child.data(), nullptr, nullptr, kColFwdWaves,
                          is_and ? kColPadAnd : kColPadOr, is_and ? kColFwdAnd : kColFwdOr, lay.col_fwd);
                make_cols(nc, cptr.data(), cpar.data(), cflag.data(), is_and && l >= 3 ? plan.layers[(size_t)l - 1].multi.data() : nullptr,
                          kColBwdWaves, kColPadAnd, is_and ? kColBwdAnd : kColBwdOr, lay.col_bwd);
            }
        }
        plan.num_split_rows += lay.bwd.n_heavy;
        plan.max_bwd_seg = std::max<int64_t>(plan.max_bwd_seg, lay.bwd.n_seg);
    }
    if (B0 > 0) {
        // Reverse-sweep sources of every row below layer B0: its parents, which are rows of any higher
        // layer up to B0 (adjoint rows are numbered like the rows of the activation buffer).
        const int64_t NR = plan.row0[(size_t)B0];
        std::vector<int32_t> gptr((size_t)NR + 1, 0);
        for (int32_t l = 1; l <= B0; ++l)
            for (int32_t ch : plan.layers[(size_t)l].child) ++gptr[(size_t)ch + 1];
        for (int64_t i = 0; i < NR; ++i) {
            plan.max_fan_out = std::max<int64_t>(plan.max_fan_out, gptr[(size_t)i + 1]);
            if ((int64_t)gptr[(size_t)i] + gptr[(size_t)i + 1] >= INT32_MAX - 64) { err = "klay_build: more than 2^31 edges"; return ST_INVAL; }
            gptr[(size_t)i + 1] += gptr[(size_t)i];
        }
        std::vector<int32_t> gsrc((size_t)gptr[(size_t)NR]);
        std::vector<uint32_t> gflag((size_t)gptr[(size_t)NR], 0u);
        {
            std::vector<int32_t> fill(gptr.begin(), gptr.end() - 1);
            for (int32_t l = 1; l <= B0; ++l) {
                const LayerPlan& lay = plan.layers[(size_t)l];
                for (int64_t p = 0; p < lay.n; ++p) {
                    const bool weighted = (l & 1) == 0 && lay.row_ptr[(size_t)p + 1] - lay.row_ptr[(size_t)p] > 1;
                    for (int32_t j = lay.row_ptr[(size_t)p]; j < lay.row_ptr[(size_t)p + 1]; ++j) {
                        const int32_t slot = fill[(size_t)lay.child[(size_t)j]]++;
                        gsrc[(size_t)slot] = (int32_t)(plan.row0[(size_t)l] + p);
                        if (weighted) gflag[(size_t)slot] = kWeightedEdge;
                    }
                }
            }
        }
        for (int32_t l = 0; l < B0; ++l) {
            // rows of layer l: a CSR slice rebased to start at 0
            const int64_t a = plan.row0[(size_t)l], n = plan.layers[(size_t)l].n;
            std::vector<int32_t> lptr((size_t)n + 1);
            for (int64_t i = 0; i <= n; ++i) lptr[(size_t)i] = gptr[(size_t)(a + i)] - gptr[(size_t)a];
            PassPlan& dst = plan.layers[(size_t)l + 1].bwd;
            // rows that are OR nodes with more than one child are flagged, as in the layer-by-layer plans
            make_pass_plan(n, lptr.data(), gsrc.data() + gptr[(size_t)a], popt, dst, gflag.data() + gptr[(size_t)a],
                           (l & 1) == 0 && l >= 2 ? plan.layers[(size_t)l].multi.data() : nullptr);
            plan.num_split_rows += dst.n_heavy;
            plan.max_bwd_seg = std::max<int64_t>(plan.max_bwd_seg, dst.n_seg);
        }
    }
    for (int32_t l = 0; l <= L; ++l) {
        plan.num_nodes += plan.layers[(size_t)l].n;
        plan.max_layer_nodes = std::max(plan.max_layer_nodes, plan.layers[(size_t)l].n);
    }

    // the narrow top: the longest suffix of candidate layers
    plan.tail_first = 0;
    if (!opt.no_tail) {
        int32_t t = L + 1;
        while (t - 1 >= 1 && plan.layers[(size_t)t - 1].tail_ok) --t;
        if (t <= L) plan.tail_first = t;
        for (--t; t >= 1; --t) plan.layers[(size_t)t].col_fwd = plan.layers[(size_t)t].col_bwd = ColPlan();      // candidates below a layer that is none
    }
    plan.col_off.assign((size_t)L + 1, -1);
    if (plan.tail_first > 0) {
        for (int32_t l = plan.tail_first; l <= L; ++l) { plan.col_off[(size_t)l] = plan.col_rows; plan.col_rows += plan.layers[(size_t)l].n; }
        plan.col_off[(size_t)plan.tail_first - 1] = plan.col_rows;
    }

    // ---------------------------------------------------------------- leaf layer and roots
    plan.num_vars = V;
    plan.num_roots = R;
    plan.num_layers = L;
    plan.pos_row.assign((size_t)V, -1);
    plan.neg_row.assign((size_t)V, -1);
    plan.leaf_code.resize((size_t)plan.layers[0].n);
    for (int64_t p = 0; p < plan.layers[0].n; ++p) {
        int32_t c = plan.layers[0].origin[(size_t)p];
        if (node_type[c] == T_LIT) {
            int32_t lit = node_lit[c];
            plan.leaf_code[(size_t)p] = lit;
            (lit > 0 ? plan.pos_row : plan.neg_row)[(size_t)(std::abs(lit) - 1)] = (int32_t)p;
        } else {
            plan.leaf_code[(size_t)p] = node_type[c] == T_TRUE ? INT32_MAX : INT32_MIN;
        }
    }
    plan.root_pos.resize((size_t)R);
    for (int32_t r = 0; r < R; ++r) plan.root_pos[(size_t)r] = at(roots[r], L);
    // the roots that read each of the nt nodes of the top layer
    auto roots_by_node = [&](int64_t nt, const std::vector<int32_t>& root_pos, std::vector<int32_t>& ptr, std::vector<int32_t>& root) {
        ptr.assign((size_t)nt + 1, 0);
        root.resize((size_t)R);
        for (int32_t r = 0; r < R; ++r) ++ptr[(size_t)root_pos[(size_t)r] + 1];
        for (int64_t i = 0; i < nt; ++i) ptr[(size_t)i + 1] += ptr[(size_t)i];
        std::vector<int32_t> fill(ptr.begin(), ptr.end() - 1);
        for (int32_t r = 0; r < R; ++r) root[(size_t)fill[(size_t)root_pos[(size_t)r]]++] = r;
    };
    roots_by_node(plan.layers[(size_t)L].n, plan.root_pos, plan.top_ptr, plan.top_root);
    if (top_first > 0) {
        // ------------------------------------------------------------ the narrow top with its chain nodes (TopPlan)
        TopPlan& top = plan.top;
        top.first = top_first;
        top.levels.resize((size_t)(L - top_first + 2));
        // slots: pos[base[c] + l] = position of node c (or of its stand-in) in level l
        std::vector<int64_t> base((size_t)N, 0);
        int64_t slots = 0;
        for (int64_t c = 0; c < N; ++c)
            if (reach[(size_t)c] && need[(size_t)c] >= top_first - 1) {
                const int32_t low = std::max(h[(size_t)c], top_first - 1);
                base[(size_t)c] = slots - low;
                slots += need[(size_t)c] - low + 1;
            }
        std::vector<int32_t> pos((size_t)slots, -1);
        auto slot = [&](int32_t c, int32_t l) -> int32_t& { return pos[(size_t)(base[(size_t)c] + l)]; };
        std::vector<std::vector<int32_t>> nodes((size_t)L + 1);      // of each level, by id
        for (int64_t c = 0; c < N; ++c)
            if (reach[(size_t)c])
                for (int32_t l = std::max(h[(size_t)c], top_first - 1); l <= need[(size_t)c]; ++l) nodes[(size_t)l].push_back((int32_t)c);
        // f(child) for every child of c (of its stand-in) in level l
        auto children = [&](int32_t c, int32_t l, auto f) {
            if (l > h[(size_t)c]) f(c);
            else for (int64_t j = child_ptr[c]; j < child_ptr[c + 1]; ++j) f(child_idx[j]);
        };
        auto fan_in = [&](int32_t c, int32_t l) -> int64_t { return l > h[(size_t)c] ? 1 : child_ptr[c + 1] - child_ptr[c]; };
        auto bucket = [](int64_t k) { int b = 0; while ((int64_t)1 << b < k) ++b; return b; };
        std::vector<int32_t> fan_out((size_t)N, 0);
        for (int32_t l = top_first - 1; l <= L; ++l) {
            TopPlan::Level& lev = top.level(l);
            std::vector<int32_t>& order = nodes[(size_t)l];
            // Rows that the reverse sweep leaves out come last.  Level 0 and the level below the plan are in the order of their
            // activation rows; the others by length, as in the layers above alias_top.
            auto left_out = [&](int32_t c) { return l < B0 && top_first > 1 && h[(size_t)c] < top_first; };
            if (l < top_first) {
                std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return own_row(a) < own_row(b); });
            } else {
                if (l < L)
                    for (int32_t p : nodes[(size_t)l + 1]) children(p, l + 1, [&](int32_t c) { ++fan_out[(size_t)c]; });
                std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) {
                    if (left_out(a) != left_out(b)) return left_out(b);
                    const bool ma = fan_out[(size_t)a] > kManyParents, mb = fan_out[(size_t)b] > kManyParents;
                    if (ma != mb) return ma;
                    const int ba = bucket(fan_in(a, l)), bb = bucket(fan_in(b, l));
                    if (!ma && ba != bb) return ba > bb;
                    return fan_out[(size_t)a] > fan_out[(size_t)b];
                });
                if (l < L)
                    for (int32_t p : nodes[(size_t)l + 1]) children(p, l + 1, [&](int32_t c) { fan_out[(size_t)c] = 0; });
            }
            lev.n = (int64_t)order.size();
            lev.at = top.rows;
            for (int64_t r = 0; r < lev.n; ++r) {
                const int32_t c = order[(size_t)r];
                slot(c, l) = (int32_t)r;
                lev.own.push_back(own_row(c));
                lev.e += fan_in(c, l);
                if (l < top_first || left_out(c)) continue;
                ++lev.kept;
                top.act_row.push_back(l >= B0 ? (int32_t)plan.row0[(size_t)l] + at(c, l) : l == h[(size_t)c] ? own_row(c) : -1);
            }
            if (l < top_first) {
                lev.kept = lev.n;
                continue;
            }
            top.rows += lev.kept;
            lev.launches = plan.layers[(size_t)l].fwd.n_heavy > 0 ? 2 : 1;
            // index vectors by parent, and by child over the kept rows of both levels
            const TopPlan::Level& low = top.level(l - 1);
            const bool is_and = (l & 1) != 0, down = l > top_first || top_first == 1;
            std::vector<int32_t> fptr((size_t)lev.n + 1, 0), fsrc, bptr((size_t)low.kept + 1, 0);
            fsrc.reserve((size_t)lev.e);
            for (int64_t r = 0; r < lev.n; ++r) {
                const size_t from = fsrc.size();
                children(order[(size_t)r], l, [&](int32_t c) { fsrc.push_back(slot(c, l - 1)); });
                std::sort(fsrc.begin() + (int64_t)from, fsrc.end());
                fptr[(size_t)r + 1] = (int32_t)fsrc.size();
            }
            make_cols(lev.n, fptr.data(), fsrc.data(), nullptr, nullptr, kColFwdWaves, is_and ? kColPadAnd : kColPadOr,
                      is_and ? kColFwdAnd : kColFwdOr, lev.fwd);
            if (!down) continue;
            for (int32_t s : fsrc)
                if (s < low.kept) ++bptr[(size_t)s + 1];
            for (int64_t i = 0; i < low.kept; ++i) bptr[(size_t)i + 1] += bptr[(size_t)i];
            std::vector<int32_t> bsrc((size_t)bptr[(size_t)low.kept]), fill(bptr.begin(), bptr.end() - 1);
            std::vector<uint32_t> flag(bsrc.size(), 0u), multi((size_t)(low.n + 31) / 32, 0u);
            for (int64_t r = 0; r < lev.n; ++r)
                for (int32_t j = fptr[(size_t)r]; j < fptr[(size_t)r + 1]; ++j) {
                    const int32_t s = fsrc[(size_t)j];
                    if (s >= low.kept) continue;
                    flag[(size_t)fill[(size_t)s]] = !is_and && fptr[(size_t)r + 1] - fptr[(size_t)r] > 1 ? kWeightedEdge : 0u;
                    bsrc[(size_t)fill[(size_t)s]++] = (int32_t)r;
                }
            if (is_and && l >= 3)
                for (int64_t r = 0; r < low.n; ++r)
                    if (fan_in(nodes[(size_t)l - 1][(size_t)r], l - 1) > 1) multi[(size_t)r >> 5] |= 1u << (r & 31);
            make_cols(low.kept, bptr.data(), bsrc.data(), flag.data(), is_and && l >= 3 ? multi.data() : nullptr, kTopBwdWaves, kColPadAnd,
                      is_and ? kColBwdAnd : kColBwdOr, lev.bwd);
        }
        const std::vector<int32_t>& last = nodes[(size_t)L];
        top.multi.assign((last.size() + 31) / 32, 0u);
        for (size_t r = 0; r < last.size(); ++r)
            if (fan_in(last[r], L) > 1) top.multi[r >> 5] |= 1u << (r & 31);
        top.root_pos.resize((size_t)R);
        for (int32_t r = 0; r < R; ++r) top.root_pos[(size_t)r] = slot(roots[r], L);
        roots_by_node((int64_t)last.size(), top.root_pos, top.top_ptr, top.top_root);
    }
    return ST_OK;
}

}  // namespace klay
