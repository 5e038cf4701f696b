// Host check of the units of narrow layers (make_units), with no GPU: random index vectors around the edges of lanes, units and the
// limits of rows and layers; every row has to be there once, whole, within one unit and aligned, in falling order of lanes.
#include <random>

#include "host_col_walk.h"

int main() {
    std::mt19937_64 rng(5);
    constexpr int kMost = klay::kNarrowUnits;
    const int64_t sizes[] = {1, 2, 3, 31, 32, 33, 63, 64, 65, 128, 129, 1000, 64 * kMost - 1, 64 * kMost, 64 * kMost + 1, 20000};
    long walked = 0, refused = 0, shorts = 0, lanes_seen[7] = {0, 0, 0, 0, 0, 0, 0};
    for (int64_t n : sizes)
        for (int shape = 0; shape < 6; ++shape) {
            const int64_t n_src = 1 + (int64_t)(rng() % 20000);
            std::vector<int32_t> ptr{0}, idx;
            std::vector<uint32_t> flags;
            bool too_long = false;
            int64_t lanes = 0;
            for (int64_t r = 0; r < n; ++r) {
                int64_t k = 1;
                switch (shape) {
                case 0: k = 1 + (int64_t)(rng() % 3); break;
                case 1: k = (int64_t)(rng() % 8); break;                                   // (rows without entries as well)
                case 2: k = ((int64_t)klay::kUnitEntries << (rng() % 4)) + (int64_t)(rng() % 2); break;
                case 3: k = r == n / 2 ? (int64_t)klay::kUnitEntries * 64 : 2; break;
                case 4: k = r == n / 2 ? (int64_t)klay::kUnitEntries * 64 + 1 : 2; break;
                default: k = 1 + (int64_t)(2.0 / (1e-2 + (double)(rng() % 1000) / 1000.0)); break;
                }
                int64_t of_row = 1;
                while (of_row * klay::kUnitEntries < k) of_row *= 2;
                too_long |= of_row > 64;
                lanes += of_row;
                for (int64_t j = 0; j < k; ++j) { idx.push_back((int32_t)(rng() % (u64)n_src)); flags.push_back(rng() % 3 == 0 ? klay::kWeightedEdge : 0u); }
                ptr.push_back((int32_t)idx.size());
            }
            std::vector<uint32_t> bits((size_t)(n + 31) / 32, 0u), units;
            for (int64_t r = 0; r < n; ++r) if (rng() % 2) bits[(size_t)r >> 5] |= 1u << (r & 31);
            const int pad = shape & 1 ? klay::kColPadOr : klay::kColPadAnd;
            klay::make_units(n, ptr.data(), idx.data(), flags.data(), bits.data(), pad, kMost, units);
            if (too_long || lanes > 64 * kMost) { CHECK(units.empty(), "a layer that is none"); ++refused; continue; }
            CHECK((int64_t)units.size() == (lanes + 63) / 64 * klay::kUnitWords, "units of %lld lanes", (long long)lanes);
            std::vector<int> written((size_t)n, 0);
            int before = 6;
            for (int64_t at = 0; at < (int64_t)units.size() / 4;) {
                const uint32_t* lane = units.data() + (size_t)at * 4;
                const uint32_t head = units[(size_t)(at / 64) * klay::kUnitWords];
                const int k = (lane[0] >> klay::kUnitLanesAt) & 7, slot = (int)(lane[0] & klay::kUnitSlot);
                CHECK(((head >> klay::kUnitLanesAt) & 7) >= (uint32_t)k, "the first lane has the most");
                CHECK((lane[0] & ~(klay::kUnitSlot | 7u << klay::kUnitLanesAt | klay::kUnitRow | klay::kUnitShort)) == 0, "bits of the streams");
                CHECK(!(lane[0] & klay::kUnitShort) || at % 64 == 0, "short unit");
                if (slot == klay::kUnitIdleSlot) {
                    CHECK(at >= lanes && k == 0, "an idle lane");
                    for (int i = 1; i < 4; ++i) CHECK(lane[i] == ((uint32_t)pad | (uint32_t)pad << 16), "entries of an idle lane");
                    ++at;
                    continue;
                }
                CHECK(k <= before && at % (1 << k) == 0, "order");
                before = k;
                const int64_t r = slot - klay::kColSlots;
                CHECK(r >= 0 && r < n, "row");
                CHECK(((lane[0] & klay::kUnitRow) != 0) == ((bits[(size_t)r >> 5] >> (r & 31)) & 1u), "row flag");
                u64 sum = 0, want = 0;
                int64_t count = 0;
                for (int sub = 0; sub < 1 << k; ++sub)
                    for (int i = 0; i < klay::kUnitEntries; ++i) {
                        CHECK((lane[4 * sub] & (klay::kUnitSlot | 7u << klay::kUnitLanesAt)) == (lane[0] & (klay::kUnitSlot | 7u << klay::kUnitLanesAt)), "lanes of a row");
                        const uint32_t x = (lane[4 * sub + 1 + i / 2] >> (i & 1 ? 16 : 0)) & 0xFFFFu;
                        if ((int)x == pad) continue;
                        CHECK(!(head & klay::kUnitShort) || i < klay::kUnitEntries / 2, "entries of a short unit");
                        const int64_t src = (int64_t)(x & 0x7FFFu) - klay::kColSlots;
                        CHECK(src >= 0 && src < n_src, "source");
                        sum += mix((u64)src) * (x & 0x8000u ? 3u : 1u);
                        ++count;
                    }
                for (int32_t j = ptr[(size_t)r]; j < ptr[(size_t)r + 1]; ++j) want += mix((u64)idx[(size_t)j]) * (flags[(size_t)j] ? 3u : 1u);
                CHECK(sum == want && count == ptr[(size_t)r + 1] - ptr[(size_t)r], "value of row %lld", (long long)r);
                shorts += head & klay::kUnitShort ? 1 : 0;
                ++lanes_seen[k];
                ++written[(size_t)r];
                at += 1 << k;
            }
            for (int64_t r = 0; r < n; ++r) CHECK(written[(size_t)r] == 1, "row %lld written %d times", (long long)r, written[(size_t)r]);
            ++walked;
        }
    CHECK(walked > 50 && refused > 5 && shorts > 0, "layers of both kinds");
    for (int k = 0; k < 7; ++k) CHECK(lanes_seen[k] > 0, "rows of %d lanes", 1 << k);
    std::printf("ok: %ld layers, %ld that are none\n", walked, refused);
    return 0;
}
