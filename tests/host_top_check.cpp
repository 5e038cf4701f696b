// Host check of the plan for the narrow top of circuits with long rows (TopPlan), with no GPU: random circuits are layerized, the
// streams of every level are walked as the persistent kernels walk them, and a reverse sweep over integers that takes the levels
// and then the launches' plans below them is compared with the sweep over the launches' plans alone.  Compiled
// with -fsanitize=address,undefined by tests/test_host_top.py.
#include <climits>
#include <random>

#include "host_col_walk.h"

struct Dag {
    int32_t vars = 0;
    std::vector<uint8_t> type;
    std::vector<int32_t> lit, idx, roots;
    std::vector<int64_t> ptr{0};
};

// layers of gates over the nodes of a few layers below, some rows of hundreds of children
static Dag random_dag(std::mt19937_64& rng) {
    Dag d;
    d.vars = 3 + (int)(rng() % 30);
    auto node = [&](uint8_t type, int32_t lit) { d.type.push_back(type); d.lit.push_back(lit); d.ptr.push_back((int64_t)d.idx.size()); };
    for (int v = 1; v <= d.vars; ++v) { node(0, v); node(0, -v); }
    if (rng() % 2) node(3, 0);
    const int layers = 2 + (int)(rng() % 9);
    int width = 50 + (int)(rng() % 400);
    std::vector<int> from{0};
    for (int l = 1; l <= layers; ++l, width = std::max(3, width * 3 / 4)) {
        const int low = from[(size_t)std::max(0, l - 1 - (int)(rng() % 4))], high = (int)d.type.size();
        from.push_back(high);
        const bool heavy = rng() % 3 == 0;
        for (int g = 0; g < width; ++g) {
            const int k = heavy && rng() % 6 == 0 ? 65 + (int)(rng() % 300) : 1 + (int)(rng() % 4);
            std::vector<uint8_t> seen((size_t)high, 0);
            for (int j = 0; j < k; ++j) {
                const int c = rng() % 5 == 0 ? (int)(rng() % (uint64_t)high) : low + (int)(rng() % (uint64_t)(high - low));
                if (!seen[(size_t)c]) { seen[(size_t)c] = 1; d.idx.push_back(c); }
            }
            node(l & 1 ? 1 : 2, 0);
        }
    }
    const int n = (int)d.type.size();
    for (int r = 1 + (int)(rng() % 40); r > 0; --r) d.roots.push_back(rng() % 4 ? from.back() + (int)(rng() % (uint64_t)(n - from.back())) : (int)(rng() % (uint64_t)n));
    return d;
}

int main(int argc, char** argv) {
    const int trials = argc > 1 ? std::atoi(argv[1]) : 150;
    std::mt19937_64 rng(4321);
    ColSeen cols;
    long whole = 0, partial = 0, over_tail = 0, left_out = 0, none = 0;
    for (int trial = 0; trial < trials; ++trial) {
        const Dag d = random_dag(rng);
        klay::Options o;
        o.alias_chains = true;
        o.no_merge = rng() % 2;
        o.no_reorder = rng() % 4 == 0;
        o.tail_rows_cap = rng() % 4 == 0 ? 0 : 100 + (int)(rng() % 400);
        klay::CircuitPlan p;
        std::string err;
        const int st = klay::layerize(d.vars, (int64_t)d.type.size(), d.type.data(), d.lit.data(), d.ptr.data(), d.idx.data(), (int32_t)d.roots.size(), d.roots.data(), o, p, err);
        CHECK(st == 0, "layerize: %s", err.c_str());
        const klay::TopPlan& top = p.top;
        const int L = p.num_layers, B0 = p.alias_top, t = top.first;
        if (t == 0) { ++none; continue; }
        CHECK(t >= 1 && t <= B0 && t < L && (int)top.levels.size() == L - t + 2, "place of the plan");
        (t == 1 ? whole : partial) += 1;
        over_tail += p.tail_first > 0;
        // nodes and children by activation row
        const int64_t rows = p.row0[(size_t)L + 1];
        std::vector<int32_t> layer((size_t)rows), node_row((size_t)rows);           // the row of the node that a row stands for
        std::vector<int32_t> row_of(d.type.size(), -1);
        for (int l = 0; l <= L; ++l)
            for (int64_t r = 0; r < p.layers[(size_t)l].n; ++r)
                if (!p.layers[(size_t)l].is_pad[(size_t)r]) row_of[(size_t)p.layers[(size_t)l].origin[(size_t)r]] = (int32_t)(p.row0[(size_t)l] + r);
        std::vector<std::vector<int32_t>> kids((size_t)rows);                       // of the nodes' own rows: own rows of the children
        for (int l = 0; l <= L; ++l)
            for (int64_t r = 0; r < p.layers[(size_t)l].n; ++r) {
                const klay::LayerPlan& lay = p.layers[(size_t)l];
                const size_t row = (size_t)(p.row0[(size_t)l] + r);
                layer[row] = l;
                node_row[row] = row_of[(size_t)lay.origin[(size_t)r]];
                if (l > 0)
                    for (int j = lay.row_ptr[(size_t)r]; j < lay.row_ptr[(size_t)r + 1]; ++j)
                        kids[row].push_back(node_row[(size_t)(lay.child[(size_t)j] + (l > B0 ? p.row0[(size_t)l - 1] : 0))]);
            }
        // the launches' reverse sweep: an integer per row, every edge times a weight of its parent
        auto weight = [&](int32_t own) { return mix((u64)own) | 1u; };
        std::vector<u64> G((size_t)rows, 0);
        for (size_t r = 0; r < p.root_pos.size(); ++r) G[(size_t)(p.row0[(size_t)L] + p.root_pos[r])] += r + 1;
        for (int l = L; l >= 1; --l) {
            const klay::LayerPlan& lay = p.layers[(size_t)l];
            for (int64_t r = 0; r < lay.n; ++r) {
                const size_t row = (size_t)(p.row0[(size_t)l] + r);
                const u64 w = lay.is_pad[(size_t)r] ? 1 : weight((int32_t)row);
                for (int j = lay.row_ptr[(size_t)r]; j < lay.row_ptr[(size_t)r + 1]; ++j)
                    G[(size_t)(lay.child[(size_t)j] + (l > B0 ? p.row0[(size_t)l - 1] : 0))] += w * G[row];
            }
        }
        // the levels
        std::vector<std::vector<u64>> adj((size_t)L + 1);
        std::vector<std::vector<int64_t>> fsrc((size_t)L + 1);
        int64_t at = 0;
        for (int l = t - 1; l <= L; ++l) {
            const klay::TopPlan::Level& lev = top.level(l);
            CHECK((int64_t)lev.own.size() == lev.n && lev.kept <= lev.n && lev.n <= klay::kTailRowsCap, "sizes");
            if (o.tail_rows_cap > 0) CHECK(lev.n <= o.tail_rows_cap, "row cap");
            if (l == 0)
                for (int64_t r = 0; r < lev.n; ++r) CHECK(lev.own[(size_t)r] == r && lev.n == p.layers[0].n, "order of the leaves");
            if (l < t) continue;
            CHECK(lev.at == at && lev.e <= klay::kTopEdges, "place of a level");
            at += lev.kept;
            const klay::TopPlan::Level& low = top.level(l - 1);
            std::vector<int32_t> pos((size_t)rows, -1);
            for (int64_t s = 0; s < low.n; ++s) { CHECK(pos[(size_t)low.own[(size_t)s]] == -1, "a node twice"); pos[(size_t)low.own[(size_t)s]] = (int32_t)s; }
            const bool is_and = l & 1, down = l > t || t == 1;
            std::vector<u64> fwd((size_t)lev.n, 0), bwd((size_t)low.kept, 0);
            std::vector<uint32_t> multi((size_t)(low.n + 31) / 32, 0u);
            for (int64_t s = 0; s < low.n; ++s)
                if (layer[(size_t)low.own[(size_t)s]] == l - 1 && kids[(size_t)low.own[(size_t)s]].size() > 1) multi[(size_t)s >> 5] |= 1u << (s & 31);
            for (int64_t r = 0; r < lev.n; ++r) {
                const int32_t own = lev.own[(size_t)r];
                CHECK(layer[(size_t)own] <= l && node_row[(size_t)own] == own, "a row's node");
                const bool pad = layer[(size_t)own] < l;
                const std::vector<int32_t> stand{own}, &below = pad ? stand : kids[(size_t)own];
                for (int32_t c : below) {
                    const int32_t s = pos[(size_t)c];
                    CHECK(s >= 0, "a child that is not in the level below");
                    fwd[(size_t)r] += mix((u64)s);
                    if (s < low.kept) {
                        if (down) CHECK(r < lev.kept, "a kept row under one that is not");
                        bwd[(size_t)s] += mix((u64)r) * (!is_and && below.size() > 1 ? 3u : 1u);
                    }
                }
                // what the row is outside: its own, a stand-in of the complete layers, or nothing
                const int32_t want = l >= B0 ? -2 : pad ? -1 : own;
                if (r < lev.kept) {
                    const int32_t act = top.act_row[(size_t)(lev.at + r)];
                    if (want == -2) CHECK(layer[(size_t)act] == l && node_row[(size_t)act] == own, "row of a complete layer");
                    else CHECK(act == want, "activation row");
                } else {
                    CHECK(l < B0 && pad && layer[(size_t)own] < t && t > 1, "a row left out");
                    ++left_out;
                }
            }
            walk_cols(lev.fwd, lev.n, low.n, klay::kColFwdWaves, is_and ? klay::kColPadAnd : klay::kColPadOr, false, nullptr, fwd, nullptr, "forward", cols);
            if (down)
                walk_cols(lev.bwd, low.kept, lev.kept, klay::kTopBwdWaves, klay::kColPadAnd, !is_and, is_and && l >= 3 ? &multi : nullptr, bwd, nullptr, "reverse", cols);
            else
                CHECK(lev.bwd.blocks.empty(), "a step that nothing takes");
        }
        CHECK(at == top.rows && (int64_t)top.act_row.size() == at, "rows of a column");
        // the sweep over the levels down to any first one, then the launches
        for (int first = t; first <= std::min(B0, L - 1); ++first) {
            std::vector<u64> H((size_t)rows, 0);
            for (int l = t - 1; l <= L; ++l) adj[(size_t)l].assign((size_t)top.level(l).n, 0);
            for (size_t r = 0; r < top.root_pos.size(); ++r) adj[(size_t)L][(size_t)top.root_pos[r]] += r + 1;
            for (int l = L; l >= first; --l) {
                const klay::TopPlan::Level& lev = top.level(l);
                for (int64_t r = 0; r < lev.kept && l <= B0; ++r)
                    if (const int32_t act = top.act_row[(size_t)(lev.at + r)]; act >= 0) H[(size_t)act] = adj[(size_t)l][(size_t)r];
                if (l == first) break;
                const klay::TopPlan::Level& low = top.level(l - 1);
                std::vector<int32_t> pos((size_t)rows, -1);
                for (int64_t s = 0; s < low.kept; ++s) pos[(size_t)low.own[(size_t)s]] = (int32_t)s;
                for (int64_t r = 0; r < lev.n; ++r) {
                    const int32_t own = lev.own[(size_t)r];
                    const bool pad = layer[(size_t)own] < l;
                    const std::vector<int32_t> stand{own}, &below = pad ? stand : kids[(size_t)own];
                    for (int32_t c : below)
                        if (pos[(size_t)c] >= 0) adj[(size_t)l - 1][(size_t)pos[(size_t)c]] += (pad ? 1 : weight(own)) * adj[(size_t)l][(size_t)r];
                }
            }
            for (int l = first - 1; l >= 0; --l) {
                const klay::PassPlan& bp = p.layers[(size_t)l + 1].bwd;
                const int64_t row0 = p.row0[(size_t)l];
                for (int64_t r = 0; r < bp.n_main + bp.n_seg; ++r) {
                    const int64_t owner = r < bp.n_main ? r : bp.seg_owner[(size_t)(r - bp.n_main)];
                    for (int j = bp.ptr[(size_t)r]; j < bp.ptr[(size_t)r + 1]; ++j) {
                        if (bp.idx[(size_t)j] == klay::kSkipRow) continue;
                        const int32_t parent = (int32_t)(bp.idx[(size_t)j] & (klay::kRowFlag - 1u));
                        H[(size_t)(row0 + owner)] += (node_row[(size_t)parent] == parent ? weight(parent) : 1) * H[(size_t)parent];
                    }
                }
            }
            for (int64_t r = 0; r < p.row0[(size_t)std::min(B0, L - 1) + 1]; ++r) CHECK(H[(size_t)r] == G[(size_t)r], "adjoint of row %lld, first %d of %d", (long long)r, first, L);
        }
        for (size_t i = 0; i + 1 < top.top_ptr.size(); ++i)
            for (int j = top.top_ptr[i]; j < top.top_ptr[i + 1]; ++j) CHECK(top.root_pos[(size_t)top.top_root[(size_t)j]] == (int32_t)i, "roots of a node");
        CHECK(top.top_ptr.back() == (int32_t)top.root_pos.size(), "roots");
    }
    CHECK(whole > 5 && partial > 10 && over_tail > 5 && left_out > 100 && none > 0, "cases seen: %ld %ld %ld %ld %ld", whole, partial, over_tail, left_out, none);
    std::printf("ok: %ld whole, %ld partial, %ld over layers of the plan itself, %ld rows left out, %ld without\n", whole, partial, over_tail, left_out, none);
    return 0;
}
