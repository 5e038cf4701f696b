// Host check of the persistent kernels' streams (ColPlan), with no GPU: random index vectors with long (up to 300000
// entries, more than 255 blocks of a unit) and short rows are cut into runs, blocks and tables, and the walk of the kernels over them (16 waves, blocks
// taken in order, 2^k lanes per row, padding by name) is executed here on integer "values".
#include <random>

#include "host_col_walk.h"

int main() {
    std::mt19937_64 rng(7);
    const int64_t sizes[] = {1, 2, 3, 63, 64, 65, 127, 128, 129, 1000, 1024, 1025, 5000, 20000};
    ColSeen seen;
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
                std::vector<u64> want((size_t)n, 0);
                std::vector<int64_t> entries((size_t)n);
                for (int64_t r = 0; r < n; ++r) {
                    entries[(size_t)r] = ptr[(size_t)r + 1] - ptr[(size_t)r];
                    for (int32_t x = ptr[(size_t)r]; x < ptr[(size_t)r + 1]; ++x)
                        want[(size_t)r] += mix((u64)idx[(size_t)x]) * (mode == 1 && (flags[(size_t)x] & klay::kWeightedEdge) ? 3u : 1u);
                }
                walk_cols(p, n, n_src, waves, pad, mode == 1, mode == 2 ? &bits : nullptr, want, &entries, "random rows", seen);
            }
        }
    CHECK(seen.most_blocks > 255, "units of many blocks");
    CHECK(seen.wide > 0 && seen.tables > 0, "several lanes per row, several tables");
    for (int kind = 0; kind < 5; ++kind) CHECK(seen.kinds[kind] > 0 && (kind > 2 || seen.full_blocks[kind] > 0), "kind %d", kind);
    std::printf("ok: %ld runs (%ld with several lanes per row, %ld tables more)\n", seen.runs, seen.wide, seen.tables);
    return 0;
}
