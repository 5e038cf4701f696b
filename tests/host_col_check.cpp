// Host check of the persistent kernels' streams (ColPlan), with no GPU: random index vectors with long (up to 300000
// entries, more than 255 blocks of a unit) and short rows are cut into runs, blocks and tables, and the walk of the kernels over them (16 waves, blocks
// taken in order, 2^k lanes per row, padding by name) is executed here on integer "values".
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "../paper_2410_11415_amd/csrc/layerize.h"

using u64 = unsigned long long;
static u64 mix(u64 x) { x += 0x9E3779B97F4A7C15ull; x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull; x = (x ^ (x >> 27)) * 0x94D049BB133111EBull; return x ^ (x >> 31); }
#define CHECK(cond, ...) do { if (!(cond)) { std::printf("FAILED %s:%d: ", __FILE__, __LINE__); std::printf(__VA_ARGS__); std::printf("\n"); std::exit(1); } } while (0)

int main() {
    std::mt19937_64 rng(7);
    const int64_t sizes[] = {1, 2, 3, 63, 64, 65, 127, 128, 129, 1000, 1024, 1025, 5000, 20000};
    int most_blocks = 0;
    long wide = 0, runs = 0, tables = 0, kinds[5] = {0, 0, 0, 0, 0};
    for (int64_t n : sizes)
        for (int shape = 0; shape < (n == 3 || n == 1000 ? 8 : 7); ++shape) {
            const int64_t n_src = 1 + (int64_t)(rng() % 20000);
            std::vector<int32_t> ptr{0}, idx;
            std::vector<uint32_t> flags;
            for (int64_t r = 0; r < n; ++r) {
                int64_t k = 1;
                switch (shape) {
                case 0: k = 1; break;
                case 1: k = 1 + (int64_t)(rng() % 4); break;
                case 2: k = 1 + (int64_t)(rng() % 64); break;
                case 3: k = r % 97 == 0 ? 700 + (int64_t)(rng() % 3000) : 1 + (int64_t)(rng() % 3); break;
                case 6: k = (r / 64) % 2 ? 1 + (int64_t)(rng() % 2) : 5 + (int64_t)((r / 128) % 5) * 9; break;
                case 4: k = r == n / 2 ? 20000 : 2; break;
                case 7: k = r == n / 2 ? 300000 : 1 + (int64_t)(rng() % 3); break;
                default: k = 1 + (int64_t)(2.0 / (1e-3 + (double)(rng() % 1000) / 1000.0)); break;
                }
                for (int64_t j = 0; j < k; ++j) { idx.push_back((int32_t)(rng() % (u64)n_src)); flags.push_back(rng() % 3 == 0 ? klay::kWeightedEdge : 0u); }
                ptr.push_back((int32_t)idx.size());
            }
            std::vector<uint32_t> bits((size_t)(n + 31) / 32, 0u);
            for (int64_t r = 0; r < n; ++r) if (rng() % 2) bits[(size_t)r >> 5] |= 1u << (r & 31);
            for (int mode = 0; mode < 3; ++mode) {                        // forward, weighted edges, row flags
                const int pad = mode == 0 && (rng() & 1) ? klay::kColPadOr : klay::kColPadAnd;
                const int waves = rng() & 1 ? klay::kColFwdWaves : klay::kColBwdWaves;
                klay::ColPlan p;
                klay::make_cols(n, ptr.data(), idx.data(), mode == 1 ? flags.data() : nullptr, mode == 2 ? bits.data() : nullptr, waves,
                                pad, (klay::ColStep)(rng() % 4), p);
                CHECK((size_t)p.block_at[klay::kSlabWaves] * klay::kBlockWords == p.blocks.size(), "blocks");
                CHECK((size_t)p.table_at[klay::kSlabWaves] * klay::kDescTable * klay::kDescWords == p.tables.size(), "tables");
                std::vector<int> written((size_t)n, 0);
                for (int w = 0; w < klay::kSlabWaves; ++w) {
                    int64_t q = p.block_at[w], t = p.table_at[w];
                    CHECK(p.table_at[w + 1] > t, "a wave without a table");
                    for (int i = 0;;) {
                        const uint32_t* ds = p.tables.data() + ((size_t)t * klay::kDescTable + (size_t)i) * klay::kDescWords;
                        const int64_t rows = ds[1] & 0xFFFFu;
                        if (rows == 0) {
                            if (ds[0] == 0) break;
                            CHECK(i == klay::kDescTable - 1 && t + 1 < p.table_at[w + 1], "another table");
                            ++t;
                            i = 0;
                            ++tables;
                            continue;
                        }
                        CHECK(++i < klay::kDescTable, "a table without an end");
                        const int64_t first = (int64_t)(ds[0] & 0x7FFFu) - klay::kColSlots;
                        const int k = (ds[1] >> 16) & 15, kind = (ds[1] >> 20) & 15, blocks = (int)(ds[0] >> 15);
                        if (blocks > most_blocks) most_blocks = blocks;
                        CHECK(w < waves, "a run for a wave that does not take part");
                        CHECK(blocks >= 1 && k <= 6 && kind <= 4 && first >= 0 && first + rows <= n, "shape");
                        CHECK(kind == 3 || blocks == 1, "blocks of a unit");
                        CHECK(kind >= 3 || k == 0, "lanes of a row");
                        ++runs; wide += k > 0; ++kinds[kind];
                        std::vector<u64> acc((size_t)rows, 0);
                        std::vector<int> seen((size_t)rows, 0);
                        const int64_t per = kind < 3 ? 1024 >> kind : 64 >> k;        // rows of a unit of blocks
                        for (int64_t unit = 0; unit * per < rows; ++unit)
                            for (int b = 0; b < blocks; ++b, ++q)
                                for (int lane = 0; lane < 64; ++lane)
                                    for (int e = 0; e < 16; ++e) {
                                        const uint32_t word = p.blocks[(size_t)q * klay::kBlockWords + (size_t)(e / 8) * klay::kLineWords + (size_t)lane * 4 + (size_t)((e & 7) / 2)];
                                        uint32_t x = e & 1 ? word >> 16 : word & 0xFFFFu;
                                        if (kind == 4 && e >= 8) { CHECK((int)x == pad, "second line of a unit of kind 4"); continue; }
                                        const int64_t r = unit * per + (kind >= 3 ? lane >> k : 64 * (e >> kind) + lane);
                                        const bool real_row = r < rows;
                                        if (mode == 2) {
                                            const bool f = real_row && ((bits[(size_t)(first + r) >> 5] >> ((first + r) & 31)) & 1u);
                                            CHECK(((x & 0x8000u) != 0) == f, "row flag");
                                            x &= 0x7FFFu;
                                        }
                                        const bool weighted = mode == 1 && (x & 0x8000u);
                                        x &= 0x7FFFu;
                                        if ((int)x == pad) { CHECK(!weighted, "flag on padding"); continue; }
                                        CHECK(real_row, "entry in an idle place");
                                        const int64_t src = (int64_t)x - klay::kColSlots;
                                        CHECK(src >= 0 && src < n_src, "source out of range");
                                        acc[(size_t)r] += mix((u64)src) * (weighted ? 3u : 1u);
                                        ++seen[(size_t)r];
                                    }
                        for (int64_t j = 0; j < rows; ++j) {
                            const int64_t r = first + j;
                            u64 want = 0;
                            for (int32_t x = ptr[(size_t)r]; x < ptr[(size_t)r + 1]; ++x)
                                want += mix((u64)idx[(size_t)x]) * (mode == 1 && (flags[(size_t)x] & klay::kWeightedEdge) ? 3u : 1u);
                            CHECK(acc[(size_t)j] == want && seen[(size_t)j] == ptr[(size_t)r + 1] - ptr[(size_t)r], "value of row %lld", (long long)r);
                            ++written[(size_t)r];
                        }
                    }
                    CHECK(q == p.block_at[w + 1] && t + 1 == p.table_at[w + 1], "blocks of wave %d", w);
                }
                for (int64_t r = 0; r < n; ++r) CHECK(written[(size_t)r] == 1, "row %lld written %d times", (long long)r, written[(size_t)r]);
            }
        }
    CHECK(most_blocks > 255, "units of many blocks");
    CHECK(wide > 0 && tables > 0 && kinds[0] > 0 && kinds[1] > 0 && kinds[2] > 0 && kinds[3] > 0 && kinds[4] > 0, "kinds of runs seen");
    std::printf("ok: %ld runs (%ld with several lanes per row, %ld tables more)\n", runs, wide, tables);
    return 0;
}
