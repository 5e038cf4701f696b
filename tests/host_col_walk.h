// The walk of the persistent kernels over a ColPlan, executed on the host on integer "values": the waves take their runs,
// tables and blocks in order, 2^k lanes work for a row, padding is known by its name.  Shared by host_col_check.cpp and
// host_plan_check.cpp.
#pragma once

#include <cstdio>
#include <cstdlib>
#include <string>
#include <vector>

#include "../paper_2410_11415_amd/csrc/layerize.h"

using u64 = unsigned long long;
static u64 mix(u64 x) { x += 0x9E3779B97F4A7C15ull; x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull; x = (x ^ (x >> 27)) * 0x94D049BB133111EBull; return x ^ (x >> 31); }
#define CHECK(cond, ...) do { if (!(cond)) { std::printf("FAILED %s:%d: ", __FILE__, __LINE__); std::printf(__VA_ARGS__); std::printf("\n"); std::exit(1); } } while (0)

// what the plans walked so far contained
struct ColSeen {
    long runs = 0, wide = 0, tables = 0, kinds[5] = {0, 0, 0, 0, 0};
    long full_blocks[3] = {0, 0, 0};       // blocks of 1024 >> kind rows
    int most_blocks = 0;                   // of a unit
};

// Walks `p` (n rows over n_src sources) and compares: want[r] = sum of mix(source), three times where the edge is weighted;
// entries[r] = how many (or null).  weighted: bit 15 of an entry marks its edge; row_bits (or null): it marks the row.
static void walk_cols(const klay::ColPlan& p, int64_t n, int64_t n_src, int waves, int pad, bool weighted, const std::vector<uint32_t>* row_bits,
                      const std::vector<u64>& want, const std::vector<int64_t>* entries, const char* what, ColSeen& seen_of) {
    CHECK((size_t)p.block_at[klay::kColWaves] * klay::kBlockWords == p.blocks.size(), "%s: blocks", what);
    CHECK((size_t)p.table_at[klay::kColWaves] * klay::kDescTable * klay::kDescWords == p.tables.size(), "%s: tables", what);
    std::vector<int> written((size_t)n, 0);
    for (int w = 0; w < klay::kColWaves; ++w) {
        int64_t q = p.block_at[w], t = p.table_at[w];
        CHECK(p.table_at[w + 1] > t, "%s: a wave without a table", what);
        for (int i = 0;;) {
            const uint32_t* ds = p.tables.data() + ((size_t)t * klay::kDescTable + (size_t)i) * klay::kDescWords;
            const int64_t rows = ds[1] & 0xFFFFu;
            if (rows == 0) {
                if (ds[0] == 0) break;
                CHECK(i == klay::kDescTable - 1 && t + 1 < p.table_at[w + 1], "%s: another table", what);
                ++t;
                i = 0;
                ++seen_of.tables;
                continue;
            }
            CHECK(++i < klay::kDescTable, "%s: a table without an end", what);
            const int64_t first = (int64_t)(ds[0] & 0x7FFFu) - klay::kColSlots;
            const int k = (ds[1] >> 16) & 15, kind = (ds[1] >> 20) & 15, blocks = (int)(ds[0] >> 15);
            CHECK(w < waves, "%s: a run for a wave that does not take part", what);
            CHECK(blocks >= 1 && k <= 6 && kind <= 4 && first >= 0 && first + rows <= n, "%s: shape", what);
            CHECK(kind == 3 || blocks == 1, "%s: blocks of a unit", what);
            CHECK(kind >= 3 || k == 0, "%s: lanes of a row", what);
            const int64_t per = kind < 3 ? 1024 >> kind : 64 >> k;        // rows of a unit of blocks
            ++seen_of.runs; seen_of.wide += k > 0; ++seen_of.kinds[kind];
            if (kind < 3) seen_of.full_blocks[kind] += rows / per;
            if (blocks > seen_of.most_blocks) seen_of.most_blocks = blocks;
            std::vector<u64> acc((size_t)rows, 0);
            std::vector<int64_t> count((size_t)rows, 0);
            for (int64_t unit = 0; unit * per < rows; ++unit)
                for (int b = 0; b < blocks; ++b, ++q)
                    for (int lane = 0; lane < 64; ++lane)
                        for (int e = 0; e < 16; ++e) {
                            const uint32_t word = p.blocks[(size_t)q * klay::kBlockWords + (size_t)(e / 8) * klay::kLineWords + (size_t)lane * 4 + (size_t)((e & 7) / 2)];
                            uint32_t x = e & 1 ? word >> 16 : word & 0xFFFFu;
                            if (kind == 4 && e >= 8) { CHECK((int)x == pad, "%s: second line of a unit of kind 4", what); continue; }
                            const int64_t r = unit * per + (kind >= 3 ? lane >> k : 64 * (e >> kind) + lane);
                            const bool real_row = r < rows;
                            if (row_bits) {
                                const bool f = real_row && (((*row_bits)[(size_t)(first + r) >> 5] >> ((first + r) & 31)) & 1u);
                                CHECK(((x & 0x8000u) != 0) == f, "%s: row flag", what);
                                x &= 0x7FFFu;
                            }
                            const bool marked = weighted && (x & 0x8000u);
                            if (weighted) x &= 0x7FFFu;
                            if ((int)x == pad) { CHECK(!marked, "%s: flag on padding", what); continue; }
                            CHECK(real_row, "%s: entry in an idle place", what);
                            const int64_t src = (int64_t)x - klay::kColSlots;
                            CHECK(src >= 0 && src < n_src, "%s: source out of range", what);
                            acc[(size_t)r] += mix((u64)src) * (marked ? 3u : 1u);
                            ++count[(size_t)r];
                        }
            for (int64_t j = 0; j < rows; ++j) {
                CHECK(acc[(size_t)j] == want[(size_t)(first + j)], "%s: value of row %lld", what, (long long)(first + j));
                if (entries) CHECK(count[(size_t)j] == (*entries)[(size_t)(first + j)], "%s: entries of row %lld", what, (long long)(first + j));
                ++written[(size_t)(first + j)];
            }
        }
        CHECK(q == p.block_at[w + 1] && t + 1 == p.table_at[w + 1], "%s: blocks of wave %d", what, w);
    }
    for (int64_t r = 0; r < n; ++r) CHECK(written[(size_t)r] == 1, "%s: row %lld written %d times", what, (long long)r, written[(size_t)r]);
}
