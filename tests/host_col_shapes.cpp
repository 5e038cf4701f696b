// Prints the runs of the persistent kernels' streams of a circuit: one line "direction is_and kind lanes rows blocks" per run
// (direction 0: forward, 1: the reverse step out of the layer), after a line with the widths of the layers.  Input file:
// V N R E as int32, then node types (uint8), literals (int32), child offsets (int64), children (int32), roots (int32).
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "../paper_2410_11415_amd/csrc/layerize.h"

template <class T>
static std::vector<T> read(FILE* f, size_t n) {
    std::vector<T> v(n);
    if (n && std::fread(v.data(), sizeof(T), n, f) != n) { std::puts("short file"); std::exit(1); }
    return v;
}

int main(int argc, char** argv) {
    FILE* f = argc > 1 ? std::fopen(argv[1], "rb") : nullptr;
    if (!f) return 1;
    const std::vector<int32_t> head = read<int32_t>(f, 4);
    const std::vector<uint8_t> type = read<uint8_t>(f, (size_t)head[1]);
    const std::vector<int32_t> lit = read<int32_t>(f, (size_t)head[1]);
    const std::vector<int64_t> ptr = read<int64_t>(f, (size_t)head[1] + 1);
    const std::vector<int32_t> idx = read<int32_t>(f, (size_t)head[3]), roots = read<int32_t>(f, (size_t)head[2]);
    std::fclose(f);
    klay::Options o;
    o.alias_chains = true;
    o.no_merge = true;
    klay::CircuitPlan plan;
    std::string err;
    if (klay::layerize(head[0], head[1], type.data(), lit.data(), ptr.data(), idx.data(), head[2], roots.data(), o, plan, err) != 0) {
        std::puts(err.c_str());
        return 1;
    }
    for (const klay::LayerPlan& lay : plan.layers) std::printf("%lld ", (long long)lay.n);
    std::printf("\n");
    for (int l = plan.tail_first > 0 ? plan.tail_first : plan.num_layers + 1; l <= plan.num_layers; ++l)
        for (int direction = 0; direction < 2; ++direction) {
            const klay::ColPlan& p = direction ? plan.layers[(size_t)l].col_bwd : plan.layers[(size_t)l].col_fwd;
            for (size_t i = 0; i < p.tables.size(); i += klay::kDescWords) {
                const uint32_t a = p.tables[i], b = p.tables[i + 1];
                if ((b & 0xFFFFu) == 0) continue;
                std::printf("%d %d %u %u %u %u\n", direction, l & 1, (b >> 20) & 15u, (b >> 16) & 15u, b & 0xFFFFu, a >> 15);
            }
        }
    return 0;
}
