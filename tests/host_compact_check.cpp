// Host check of compact_pass, with no GPU: plans of random index vectors with left-out and split rows, with those rows' entries taken
// out; every other row has to be there with its entries, its number and the tasks over it, and the segments as they were.
#include <random>

#include "host_col_walk.h"

int main() {
    std::mt19937_64 rng(11);
    long rows_out = 0, split = 0;
    for (int64_t n : {1, 2, 7, 63, 64, 65, 1000, 5000})
        for (int share = 0; share < 4; ++share) {
            std::vector<int32_t> ptr{0}, idx;
            std::vector<uint8_t> skip((size_t)n);
            for (int64_t r = 0; r < n; ++r) {
                const int64_t k = rng() % 50 == 0 ? 49 + (int64_t)(rng() % 900) : 1 + (int64_t)(rng() % 4);
                for (int64_t j = 0; j < k; ++j) idx.push_back((int32_t)(rng() % 100000));
                ptr.push_back((int32_t)idx.size());
                skip[(size_t)r] = share == 3 ? 1 : (int)(rng() % 3) < share;
            }
            klay::PassPlan in, out;
            std::vector<int32_t> out_row, entry_row;
            klay::make_pass_plan(n, ptr.data(), idx.data(), klay::Options(), in, nullptr, nullptr, skip.data());
            klay::compact_pass(in, out, out_row, entry_row);
            CHECK(out.n_main == (int32_t)out_row.size() && out.n_seg == in.n_seg && out.n_heavy == in.n_heavy && out.comb_row == in.comb_row, "shape");
            CHECK(out.ptr.size() == (size_t)(out.n_main + out.n_seg + 1) && out.idx.size() >= (size_t)out.ptr.back() + klay::kIdxPad, "padding");
            CHECK(entry_row.size() == (size_t)out.ptr[(size_t)out.n_main] + klay::kIdxPad, "padding of the rows of entries");
            int32_t at = 0;
            for (int64_t r = 0; r < n; ++r) {
                const int32_t from = in.ptr[(size_t)r], k = in.ptr[(size_t)r + 1] - from;
                if (k == 1 && in.idx[(size_t)from] == klay::kSkipRow) { ++split; continue; }
                CHECK(at < out.n_main && out_row[(size_t)at] == r && out.ptr[(size_t)at + 1] - out.ptr[(size_t)at] == k, "row %lld", (long long)r);
                for (int32_t j = 0; j < k; ++j)
                    CHECK(out.idx[(size_t)(out.ptr[(size_t)at] + j)] == in.idx[(size_t)(from + j)] && entry_row[(size_t)(out.ptr[(size_t)at] + j)] == r, "entry of row %lld", (long long)r);
                ++at;
                ++rows_out;
            }
            CHECK(at == out.n_main, "rows");
            for (int32_t i = 0; i < in.n_seg; ++i) {
                const int32_t a = in.ptr[(size_t)(in.n_main + i)], b = out.ptr[(size_t)(out.n_main + i)], k = in.ptr[(size_t)(in.n_main + i) + 1] - a;
                CHECK(out.ptr[(size_t)(out.n_main + i) + 1] - b == k, "segment");
                for (int32_t j = 0; j < k; ++j) CHECK(out.idx[(size_t)(b + j)] == in.idx[(size_t)(a + j)], "entry of a segment");
            }
            for (int part = 0; part < 2; ++part) {
                const std::vector<int32_t>& t = part ? out.seg_tasks : out.tasks;
                const int32_t count = part ? out.n_seg_tasks : out.n_tasks, lo = part ? out.n_main : 0, hi = part ? out.n_main + out.n_seg : out.n_main;
                if (part && out.n_seg == 0) continue;
                CHECK(t.size() == (size_t)(2 * (count + 1)) && t[0] == lo && t[2 * (size_t)count] == hi, "tasks");
                for (int32_t i = 0; i <= count; ++i) CHECK(t[2 * (size_t)i + 1] == out.ptr[(size_t)t[2 * (size_t)i]] && (i == 0 || t[2 * (size_t)i] > t[2 * (size_t)i - 2]), "task");
            }
        }
    // the streaming kernel's tasks: every row that is no skip entry in one of them, in order, and bounded
    for (int64_t n : {1, 2, 50, 4000, 300000}) {
        klay::PassPlan p;
        std::vector<int32_t> ptr{0}, idx;
        for (int64_t r = 0; r < n; ++r) {
            for (int64_t k = rng() % 40 == 0 ? 60 : 1 + (int64_t)(rng() % 5); k > 0; --k) idx.push_back((int32_t)(rng() % 1000));
            ptr.push_back((int32_t)idx.size());
        }
        klay::make_pass_plan(n, ptr.data(), idx.data(), klay::Options(), p);
        for (int part = 0; part < 2; ++part) {
            const int64_t from = part ? n : 0, to = part ? n + p.n_seg : n;
            const std::vector<int32_t> t = klay::stream_tasks(p, from, to);
            int64_t row = from;
            auto skipped = [&](int64_t r) { return p.idx[(size_t)p.ptr[(size_t)r]] == klay::kSkipRow; };
            for (size_t i = 0; i < t.size(); i += klay::kTaskWords) {
                for (int e = klay::kTaskHead; e < klay::kTaskWords; ++e) CHECK((uint32_t)t[i + (size_t)e] == p.idx[(size_t)t[i + 1] + (size_t)(e - klay::kTaskHead)], "entry of a task");
                for (; row < t[i]; ++row) CHECK(skipped(row), "row %lld in no task", (long long)row);
                CHECK(t[i] == row && t[i + 2] > t[i] && t[i + 2] <= to && t[i + 1] == p.ptr[(size_t)t[i]] && t[i + 3] == p.ptr[(size_t)t[i + 2]], "task");
                CHECK(t[i + 3] > t[i + 1] && p.ptr[(size_t)t[i + 2] - 1] - t[i + 1] < 16, "entries of a task before its last row");
                for (; row < t[i + 2]; ++row) CHECK(!skipped(row), "a skip entry in a task");
            }
            for (; row < to; ++row) CHECK(skipped(row), "row %lld in no task", (long long)row);
        }
    }
    CHECK(rows_out > 1000 && split > 1000, "rows of both kinds");
    std::printf("ok: %ld rows, %ld without entries\n", rows_out, split);
    return 0;
}
