// Host check of compact_pass, with no GPU: plans of random index vectors with left-out and split rows, with those rows' entries taken
// out; every other row has to be there with its entries, its number and the tasks over it, and the segments as they were; and what the streaming
// kernel reads of its tasks has to be inside the arrays.
#include <random>

#include "host_col_walk.h"

// The streaming kernel's tasks over the rows from .. to: every row that is no skip entry in one of them, in order, and bounded.
static std::vector<int32_t> checked_tasks(const klay::PassPlan& p, int64_t from, int64_t to) {
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
    return t;
}

// What a wave reads of every task of a plan without its left-out rows, main rows and segments, is inside the arrays.  Returns the tasks
// that are segments.
static long check_reads(const klay::PassPlan& out, const std::vector<int32_t>& entry_row) {
    long segments = 0;
    for (int part = 0; part < 2; ++part) {
        const std::vector<int32_t> t = checked_tasks(out, part ? out.n_main : 0, part ? out.n_main + out.n_seg : out.n_main);
        for (size_t i = 0; i < t.size(); i += klay::kTaskWords) {
            const int64_t first = t[i + 1], reads = klay::stream_reads(t[i + 3] - t[i + 1]);
            CHECK(first + reads <= (int64_t)out.idx.size(), "entries read past their end");
            const char* rows = static_cast<const char*>(klay::task_entry_rows(out.idx.data(), entry_row.data(), t[i + 1], part == 1));
            auto inside = [&](const void* array, size_t n) { return rows >= static_cast<const char*>(array) && rows + 4 * reads <= static_cast<const char*>(array) + 4 * n; };
            CHECK(inside(entry_row.data(), entry_row.size()) || inside(out.idx.data(), out.idx.size()),
                  "%s task at entry %lld reads the rows of %lld entries past the end of their %zu", part ? "segment" : "main", (long long)first, (long long)reads, entry_row.size());
            if (!part)
                for (int64_t j = first; j < t[i + 3]; ++j) CHECK(reinterpret_cast<const int32_t*>(rows)[j - first] == entry_row[(size_t)j], "row of an entry");
            segments += part;
        }
    }
    return segments;
}

int main() {
    std::mt19937_64 rng(11);
    long rows_out = 0, split = 0, segments = 0;
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
            segments += check_reads(out, entry_row);
            checked_tasks(in, 0, n);
            checked_tasks(in, n, n + in.n_seg);
        }
    // whole plans
    for (int64_t n : {1, 2, 50, 4000, 300000}) {
        klay::PassPlan p;
        std::vector<int32_t> ptr{0}, idx;
        for (int64_t r = 0; r < n; ++r) {
            for (int64_t k = rng() % 40 == 0 ? 60 : 1 + (int64_t)(rng() % 5); k > 0; --k) idx.push_back((int32_t)(rng() % 1000));
            ptr.push_back((int32_t)idx.size());
        }
        klay::make_pass_plan(n, ptr.data(), idx.data(), klay::Options(), p);
        checked_tasks(p, 0, n);
        checked_tasks(p, n, n + p.n_seg);
    }
    // nearly all entries in segments: a layer of 300 rows of 20000 entries and 4000 that are left out
    {
        klay::PassPlan in, out;
        std::vector<int32_t> ptr{0}, idx, out_row, entry_row;
        std::vector<uint8_t> skip;
        for (int r = 0; r < 4300; ++r) {
            for (int64_t k = r < 300 ? 20000 : 2; k > 0; --k) idx.push_back((int32_t)(rng() % 30000));
            ptr.push_back((int32_t)idx.size());
            skip.push_back(r >= 300);
        }
        klay::make_pass_plan(4300, ptr.data(), idx.data(), klay::Options(), in, nullptr, nullptr, skip.data());
        klay::compact_pass(in, out, out_row, entry_row);
        CHECK(out.n_main == 0 && out.n_seg > 100000, "segments alone");
        segments += check_reads(out, entry_row);
    }
    CHECK(rows_out > 1000 && split > 1000 && segments > 1000, "rows of all kinds");
    std::printf("ok: %ld rows, %ld without entries\n", rows_out, split);
    return 0;
}
