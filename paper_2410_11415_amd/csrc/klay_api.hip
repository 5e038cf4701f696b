// C ABI of the layered circuit evaluator (see include/klay.h): handle management, workspace,
// and the launch sequences of the forward sweep (paper Section 4, Alg. 1 / Appendix C, Alg. 4)
// and of the reverse sweep that yields the derivative with respect to the leaf weights.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "../../include/klay.h"
#include "klay_kernels.hip.h"
#include "klay_kernels_f64.hip.h"
#include "layerize.h"

// Workspace of klay_forward_static, the entry point that allocates nothing: a fixed array in device
// memory.  Every GPU the library runs on holds its own copy at its own address until the process
// ends.  In host code the name below is only a handle for hipGetSymbolAddress; the kernels get the
// address that call returned (kept per device in g_static_ws).
constexpr size_t kStaticWorkspaceBytes = KLAY_STATIC_WORKSPACE_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticWorkspaceBytes];

// Layers with split rows and at most this many index entries run main rows and segments in one generic
// launch and the combine rows in another; larger ones the segments first, then main rows and combine rows.
// (32 < B <= 64.  us, together throughout / this rule: 1e6 nodes with power-law fan-ins, training step at B = 50 914 / 882; 290000 nodes, 1e7
// edges, forward at B = 64 375 / 384.  The line looks at a layer's size alone, and is 2% off where the segments are most of a large layer.)
constexpr int64_t kSmallPassEntries = 100000;
constexpr size_t kTailLdsMax = 160 * 1024;     // LDS of a gfx950 compute unit: the most a workgroup of the persistent kernels gets

namespace {

thread_local std::string g_err;

constexpr int kMaxDevices = 64;
std::mutex g_static_mu;
float* g_static_ws[kMaxDevices] = {};      // device address of `scratch` on each device

// Looks the array's address up once per device; `device` must be the current device.
hipError_t static_workspace(int device, float** out) {
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_static_mu);
    if (!g_static_ws[device]) {
        void* ptr = nullptr;
        hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_static_ws[device] = static_cast<float*>(ptr);
    }
    *out = g_static_ws[device];
    return hipSuccess;
}

klay_status fail(klay_status s, const std::string& msg) {
    g_err = msg;
    return s;
}

#define KLAY_HIP(call)                                                                         \
    do {                                                                                       \
        hipError_t e__ = (call);                                                               \
        if (e__ != hipSuccess)                                                                 \
            return fail(KLAY_EHIP, std::string(#call) + ": " + hipGetErrorString(e__));        \
    } while (0)

// Roots that one wave of the persistent forward kernel reads at the end; more are read by all, which then stay until then.
constexpr int32_t kRootsOneWave = 256;

constexpr size_t kAlignInts = 64;   // 256-byte alignment of every uploaded array

struct DevPass {
    const int32_t *ptr = nullptr, *seg_owner = nullptr, *comb_ptr = nullptr, *comb_row = nullptr, *tasks = nullptr,
                  *seg_tasks = nullptr;
    const uint32_t *idx = nullptr, *comb_idx = nullptr;
    const int32_t *out_row = nullptr, *entry_row = nullptr;      // of a plan without left-out rows (compact_pass)
    const int32_t *stream_tasks = nullptr, *stream_seg_tasks = nullptr;      // of the streaming kernel
    int32_t n_stream_tasks = 0, n_stream_seg_tasks = 0;
    int32_t n_light = 0;                         // main rows that are evaluated as such
    int32_t n_main = 0, n_seg = 0, n_heavy = 0, n_tasks = 0, n_seg_tasks = 0;
    int32_t longest_comb = 0;                    // partial rows of the split row with most of them
    int32_t longest_seg = 0;                     // entries of the longest segment
    int32_t n_comb_many = 0;                     // see PassPlan
    bool has_weighted = false;
    int64_t edges = 0;
    int64_t main_entries = 0, seg_entries = 0;   // index entries of light main rows / of segments
    int64_t n_src = 0;                           // distinct source rows the pass reads
};

// Log-semiring reverse sweep: adjoints of OR layers travel in the one-gather form (off: the two-gather step).
constexpr bool kOneGather = true;

struct DevLayer {
    int64_t n = 0, e = 0;
    int64_t row0 = 0;        // first row of this layer in the activation buffer
    DevPass fwd, bwd;
    // the fused plans (LayerPlan::fwd_kept, fwd2), where the layerizer built them
    DevPass fwd_kept, fwd2;
    bool has_fwd2 = false;
    int64_t n_fused = 0;     // AND layers: so many rows are fused (their values are not written when the fused plans run)
    bool has_fwd_kept = false;
    const uint32_t* multi = nullptr;   // OR layers: bit r = node r has more than one child
    bool has_multi = false;
};

// The layers that the persistent kernels may run, first .. L: those of the circuit plan itself (klay_circuit::tail) or of its
// TopPlan.
struct ColTail {
    int32_t first = 0;                   // lowest one (0: none)
    std::vector<int64_t> n, kept, at;    // by layer from first - 1 on (index l): rows, rows kept for the reverse sweep, first entry in a column
    std::vector<int64_t> e, words[2];    // edges; words of the streams, forward and reverse
    int64_t rows = 0;                    // kept rows of the layers first .. L
    const klay::ColLayer* layers = nullptr;    // where the streams of the layers first .. L start
    const klay::Line* blocks[2] = {nullptr, nullptr};
    int32_t n_blocks[2] = {0, 0};
    const klay::Desc* tables = nullptr;
    const klay::Line* units[2] = {nullptr, nullptr};
    int32_t n_units[2] = {0, 0};
    int32_t narrow[2] = {0, 0};          // forward: the layers from this one on are narrow (L + 1: none); reverse: the steps from the layers down to this one
    const int32_t *root_pos = nullptr, *top_ptr = nullptr, *top_root = nullptr;
    std::vector<int32_t> launches;       // what the layers take otherwise
    std::vector<int64_t> share;          // ColPlan::share of the forward streams
    // TopPlan only: activation row of every row (of level l from own_at[l] on), of every kept row; flags of the top level (null: no
    // layer of OR nodes)
    const int32_t *own = nullptr, *act_row = nullptr;
    std::vector<int64_t> own_at;
    const uint32_t* multi = nullptr;
};

struct Geometry {            // how a batch of B columns is mapped onto lanes
    int vec = 1, w = 64, ld = 0, tiles = 1;
};

Geometry geometry(int B) {
    Geometry g;
    if (B > 128) { g.vec = 4; g.w = 64; }
    else if (B > 64) { g.vec = 2; g.w = 64; }
    else if (B > 32) { g.vec = 1; g.w = 64; }
    else {
        g.vec = 1;
        g.w = 1;
        while (g.w < B) g.w *= 2;
    }
    g.ld = B > 32 ? (B + 3) / 4 * 4 : B;        // rows of wave-wide batches are float4-aligned
    const int tile = g.w * g.vec;
    g.tiles = (B + tile - 1) / tile;
    return g;
}

size_t align_floats(size_t n) { return (n + 63) / 64 * 64; }

struct Workspace {
    size_t act = 0, wT = 0, seg_rows = 0, g0 = 0, g1 = 0, g2 = 0, tb = 0, stage = 0, flags = 0, total = 0;   // offsets in floats
    size_t top_tb = 0, top_g = 0;            // TopPlan: values and adjoints of its levels
    size_t top_stage = 0, top_stage_n = 0;   // and the level below its first one, for the forward kernel to read (0 floats: it reads rows)
};

struct EventRec {
    int cls;
    hipEvent_t start, stop;
    double bytes, min_bytes;
};

}  // namespace

struct klay_circuit {
    klay::CircuitPlan plan;
    int device = -1;
    bool small_batch_edges = false;      // klay_options.small_batch_edges
    bool one_gather = false;             // the log reverse sweep may use the one-gather form (see upload)
    std::vector<DevLayer> dl;
    int32_t* d_index = nullptr;          // one allocation holding every index array
    size_t index_bytes = 0;
    const int32_t* d_leaf_list = nullptr;      // see leaf_list, of n_leaf_list variables (0: there is none)
    int32_t n_leaf_list = 0;
    const int32_t *d_pos_row = nullptr, *d_neg_row = nullptr, *d_root_pos = nullptr, *d_top_ptr = nullptr,
                  *d_top_root = nullptr;
    int32_t true_row = -1, false_row = -1;
    ColTail tail, top;                         // what the persistent kernels may run: layers of the plan, and of its TopPlan
    size_t tail_lds_bytes = 0;                 // LDS a workgroup of the persistent kernels may use (0: kernels unusable)
    int64_t tail_rows = 0;                     // T: rows of all tail candidate layers (one column of the tail buffer)
    int32_t last_tail_first = 0;               // first layer the last forward ran in the persistent kernel (0: none)
    int32_t last_top_first = 0;                // the same, from the TopPlan
    int32_t last_tail_T = 0;                   // floats in a column of its value buffer
    bool last_tail_staged = false;             // the layer below it is part of that buffer
    // real-semiring reverse sweep (built at its first use): per AND layer the plain by-parent index
    // vectors (for prod_parent_kernel); for the layers below alias_top also the by-child pass over the
    // parents in all higher layers up to alias_top, whose entries tell AND parents from plain adjoint rows
    struct RealLayer { const int32_t* ptr = nullptr; const int32_t* child = nullptr; DevPass by_child; };
    std::vector<RealLayer> real_layers;
    int32_t* d_real_index = nullptr;
    const int32_t *d_real_ptr = nullptr, *d_real_child = nullptr;      // persistent kernel: offsets in it by depth under the top layer (null: too large)
    void* ws_own = nullptr;
    size_t ws_own_bytes = 0;
    void* ws_user = nullptr;
    size_t ws_user_bytes = 0;
    // state of the most recent forward
    bool no_fusion = false;                    // klay_options.no_fusion
    bool have_fwd = false;
    bool last_fused = false;                   // the forward pass ran the fused plans: the values of fused AND rows do not exist
    bool bwd_followed = false;                 // klay_backward was called after the most recent forward pass
    int32_t last_B = 0;
    int last_semiring = 0;
    bool last_neg_explicit = false;            // the negated literals had weights of their own
    bool last_ws_has_bwd = false;
    // double-precision evaluation (its own library-owned workspace)
    void* ws64 = nullptr;
    size_t ws64_bytes = 0;
    bool have_fwd64 = false;
    bool bwd64_followed = false;               // the last double-precision forward pass was followed by a backward pass
    int32_t last64_B = 0;
    int last64_semiring = 0;
    bool last64_neg_explicit = false;
    const ColTail* last64_tail = nullptr;      // whose layers from last64_first on ran in the persistent kernel (null: none)
    int32_t last64_first = 0;
    // profiling
    bool profiling = false;
    std::vector<EventRec> ev_fwd, ev_bwd;
    std::vector<hipEvent_t> ev_pool;
};

namespace {

// widest layer above the padding-free part (1 if there is none): the size of the two adjoint buffers
// that the layer-by-layer part of the reverse sweep alternates between
int64_t top_layer_rows(const klay::CircuitPlan& p) {
    int64_t n = 1;
    for (int l = p.alias_top + 1; l <= p.num_layers; ++l) n = std::max(n, p.layers[(size_t)l].n);
    return n;
}

int64_t tail_stage_rows(const klay_circuit* c, int B);
int choose_top(const klay_circuit* c, int B, bool real_training = false);
int tail_columns(int B, const int64_t (&size)[2], size_t lds_bytes, bool reverse);

// Columns from which on the forward kernel reads the level below its first one from columns instead of its rows: fewer
// are not worth the launch that makes columns of them.
constexpr int kTopStageB = 17;

// top: first layer that the persistent kernels take from the TopPlan (0: none).  A pass that nothing is kept for (need_bwd =
// false) needs the same in both cases.
Workspace workspace_layout(const klay_circuit* c, int B, bool need_bwd, int top) {
    const Geometry g = geometry(B);
    const klay::CircuitPlan& p = c->plan;
    Workspace w;
    size_t off = 0;
    auto take = [&](size_t n) { const size_t at = off; off += align_floats(n); return at; };
    w.act = take((size_t)p.num_nodes * g.ld);
    w.wT = take((size_t)std::max(1, p.num_vars) * g.ld);
    const int64_t seg = std::max(p.max_fwd_seg, need_bwd ? p.max_bwd_seg : 0);
    w.seg_rows = take((size_t)std::max<int64_t>(seg, 1) * g.ld);
    if (top > 0 && need_bwd) {
        // values of the levels, column-major, and their adjoints where they go to rows afterwards
        w.top_tb = take((size_t)c->top.rows * (size_t)B);
        if (top > 1) w.top_g = take((size_t)c->top.rows * (size_t)B);
    } else {
        // values of the tail layers, one run of tail_rows floats per batch column
        w.tb = take((size_t)c->tail_rows * (size_t)B);
        // the layer below the persistent forward kernel's first one, column-major, for that kernel to read
        w.stage = take((size_t)tail_stage_rows(c, B) * (size_t)B);
    }
    if (need_bwd) {
        // adjoints: one row per node of the layers 0 .. alias_top, and two buffers of the widest layer above
        // them that the layer-by-layer part of the sweep alternates between
        w.g0 = take((size_t)p.row0[(size_t)p.alias_top + 1] * g.ld);
        w.g1 = take((size_t)top_layer_rows(p) * g.ld);
        w.g2 = take((size_t)top_layer_rows(p) * g.ld);
        // one word per layer: the real-semiring sweep's "a node value of this product layer is zero" flags
        w.flags = take((size_t)p.num_layers + 1);
    }
    w.total = off;
    if (top > 1 && B >= kTopStageB) {
        // The level below the first one has no buffer of its own.  It takes the adjoint rows, which a forward pass does not use (its
        // rows stand for as many nodes of the layers below `top`, each of which has one); without those the activation rows of the
        // layers that stay in the kernel, where they are enough.
        const size_t n = (size_t)c->top.n[(size_t)top - 1] * (size_t)B, rows = align_floats((size_t)p.row0[(size_t)top] * g.ld);
        if (need_bwd) w.top_stage = w.g0;
        else if (rows + n <= (size_t)p.num_nodes * g.ld) w.top_stage = w.act + rows;
        if (w.top_stage) w.top_stage_n = n;
    }
    return w;
}

// Waves from which on a lane of the generic kernels takes more than one column (1024, 2048 and 4096 measured: a power-law
// circuit of 62000 nodes at B = 9, training step 161 / 123 / 126 us, other workloads within 1%; always four columns: 210 us).
constexpr int64_t kFillWaves = 2048;

// Lanes per row of the generic kernels for `vec` columns a lane; a wave takes 64 / lanes rows.
int row_lanes(int B, int vec) { return std::min(64, (B + vec - 1) / vec); }
uint32_t row_inverse(int lanes) { return (uint32_t)((65536 + lanes - 1) / lanes); }

template <int OP>
void launch_op(const klay::PassArgs& a, int vec, dim3 grid, hipStream_t s, int32_t longest_seg = 0) {
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, a); };
    if constexpr (OP == klay::OP_LSE) {
        // segments alone (see pass_body; with one column a lane the launch is a small one, bound by its latency), unless a longer minimum was asked for
        // than lse_value has room for
        if (a.row_begin > 0 && a.row_begin == a.n_main && vec > 1 && longest_seg < klay::kLseFlatTerms)
            return vec == 4 ? launch(klay::pass_kernel<OP, 4, true>) : launch(klay::pass_kernel<OP, 2, true>);
    }
    vec == 4 ? launch(klay::pass_kernel<OP, 4, false>) : vec == 2 ? launch(klay::pass_kernel<OP, 2, false>) : launch(klay::pass_kernel<OP, 1, false>);
}

// workgroups of 4 waves for `rows` rows, a multiple of 8 (see xcd_block)
unsigned row_blocks(int64_t rows, int lanes) {
    const int64_t per_block = 4 * (64 / lanes);
    return (unsigned)(((rows + per_block - 1) / per_block + 7) / 8 * 8);
}

// Columns per lane of a generic launch over the rows row_begin .. n_total; sets the lanes per row.
int deal_lanes(klay::PassArgs& a) {
    const int64_t rows = (int64_t)a.n_total - a.row_begin;
    // as many columns per lane as leave 8 waves for every compute unit: a smaller launch waits for its longest rows, and
    // a row takes less time the fewer columns a lane has
    int vec = a.B >= 4 ? 4 : (a.B >= 2 ? 2 : 1);
    while (vec > 1 && rows * row_lanes(a.B, vec) < 64 * kFillWaves) vec /= 2;
    a.lanes = row_lanes(a.B, vec);
    // with one column a lane a power of two: rows whose lanes straddle the groups of 16 that a load is taken in wait
    // longer, and there are waves to spare (power-law fan-ins, us: 12000 nodes forward B = 6 300 -> 283, 2800 nodes
    // max B = 5 130 -> 123; with more columns a lane it is the other way round: 800000 nodes training B = 10 290 against 294)
    if (vec == 1)
        for (a.lanes = 1; a.lanes < std::min(64, a.B); a.lanes *= 2) {}
    a.per_wave = 64 / a.lanes;
    a.inverse = row_inverse(a.lanes);
    return vec;
}

// Launch one gather-reduce pass over `n_total` rows.  longest_seg: entries of the longest segment, where there are segments alone.
void launch_pass(int op, klay::PassArgs a, hipStream_t s, int32_t longest_seg = 0) {
    const int64_t rows = (int64_t)a.n_total - a.row_begin;
    if (rows <= 0) return;
    const int vec = deal_lanes(a);
    dim3 grid(row_blocks(rows, a.lanes), (unsigned)((a.B + a.lanes * vec - 1) / (a.lanes * vec)));
    switch (op) {
    case klay::OP_SUM: launch_op<klay::OP_SUM>(a, vec, grid, s); break;
    case klay::OP_PROD: launch_op<klay::OP_PROD>(a, vec, grid, s); break;
    case klay::OP_LSE: launch_op<klay::OP_LSE>(a, vec, grid, s, longest_seg); break;
    case klay::OP_MAX: launch_op<klay::OP_MAX>(a, vec, grid, s); break;
    case klay::OP_PROD_BWD: launch_op<klay::OP_PROD_BWD>(a, vec, grid, s); break;
    case klay::OP_SUM_H: launch_op<klay::OP_SUM_H>(a, vec, grid, s); break;
    case klay::OP_SOFTMAX_H: launch_op<klay::OP_SOFTMAX_H>(a, vec, grid, s); break;
    case klay::OP_SUM_P: launch_op<klay::OP_SUM_P>(a, vec, grid, s); break;
    case klay::OP_PROD_BWD_P: launch_op<klay::OP_PROD_BWD_P>(a, vec, grid, s); break;
    default: launch_op<klay::OP_SOFTMAX_BWD>(a, vec, grid, s); break;
    }
}

// Small batches (B <= 32): the lanes = edges kernel over the main rows and the segments of a pass.
template <int OP, int LPR>
void launch_edge_one(const DevPass& dp, const float* src, const float* src2, const float* own, float* dst,
                     float* dst_seg, int B, int ld, hipStream_t s, int* zf) {
    constexpr int EPW = 64 / LPR, CH = EPW >= 16 ? 4 : 8;
    const int64_t entries = dp.main_entries + dp.n_heavy;
    // a wave takes about two rounds of its gathers: CH steps of EPW entries each
    const double per_task = dp.n_tasks > 0 ? (double)entries / dp.n_tasks : 16.0;
    int span = (int)(2.0 * CH * EPW / std::max(1.0, per_task) + 0.5);
    span = std::max(1, span);
    const int64_t waves = ((int64_t)dp.n_tasks + span - 1) / span + ((int64_t)dp.n_seg_tasks + span - 1) / span;
    if (waves <= 0) return;
    dim3 grid((unsigned)((waves + 3) / 4));
    hipLaunchKernelGGL((klay::edge_kernel<OP, LPR>), grid, dim3(256), 0, s, reinterpret_cast<const int2*>(dp.tasks),
                       dp.n_tasks, span, dp.idx, src, src2, own, dst, B, ld, reinterpret_cast<const int2*>(dp.seg_tasks),
                       dp.n_seg_tasks, dp.seg_owner, dp.n_main, dst_seg, zf);
}

template <int OP>
void launch_edge_op(const DevPass& dp, const Geometry& g, const float* src, const float* src2, const float* own,
                    float* dst, float* dst_seg, int B, hipStream_t s, int* zf) {
    switch (g.w) {
    case 32: launch_edge_one<OP, 32>(dp, src, src2, own, dst, dst_seg, B, g.ld, s, zf); break;
    case 16: launch_edge_one<OP, 16>(dp, src, src2, own, dst, dst_seg, B, g.ld, s, zf); break;
    case 8: launch_edge_one<OP, 8>(dp, src, src2, own, dst, dst_seg, B, g.ld, s, zf); break;
    case 4: launch_edge_one<OP, 4>(dp, src, src2, own, dst, dst_seg, B, g.ld, s, zf); break;
    case 2: launch_edge_one<OP, 2>(dp, src, src2, own, dst, dst_seg, B, g.ld, s, zf); break;
    default: launch_edge_one<OP, 1>(dp, src, src2, own, dst, dst_seg, B, g.ld, s, zf); break;
    }
}

void launch_edge(int op, const DevPass& dp, const Geometry& g, const float* src, const float* src2, const float* own,
                 float* dst, float* dst_seg, int B, hipStream_t s, int* zf) {
    switch (op) {
    case klay::OP_SUM: launch_edge_op<klay::OP_SUM>(dp, g, src, src2, own, dst, dst_seg, B, s, zf); break;
    case klay::OP_PROD: launch_edge_op<klay::OP_PROD>(dp, g, src, src2, own, dst, dst_seg, B, s, zf); break;
    case klay::OP_LSE: launch_edge_op<klay::OP_LSE>(dp, g, src, src2, own, dst, dst_seg, B, s, zf); break;
    case klay::OP_MAX: launch_edge_op<klay::OP_MAX>(dp, g, src, src2, own, dst, dst_seg, B, s, zf); break;
    case klay::OP_PROD_BWD: launch_edge_op<klay::OP_PROD_BWD>(dp, g, src, src2, own, dst, dst_seg, B, s, zf); break;
    case klay::OP_SUM_H: launch_edge_op<klay::OP_SUM_H>(dp, g, src, src2, own, dst, dst_seg, B, s, zf); break;
    case klay::OP_SOFTMAX_H: launch_edge_op<klay::OP_SOFTMAX_H>(dp, g, src, src2, own, dst, dst_seg, B, s, zf); break;
    case klay::OP_SUM_P: launch_edge_op<klay::OP_SUM_P>(dp, g, src, src2, own, dst, dst_seg, B, s, zf); break;
    case klay::OP_PROD_BWD_P: launch_edge_op<klay::OP_PROD_BWD_P>(dp, g, src, src2, own, dst, dst_seg, B, s, zf); break;
    default: launch_edge_op<klay::OP_SOFTMAX_BWD>(dp, g, src, src2, own, dst, dst_seg, B, s, zf); break;
    }
}

// Streaming kernel over the main rows of a pass and the segments of its split rows (batch
// tiles of one wave, two or four columns per lane: B > 64).  dst_seg is the base of the partial rows shifted by -n_main rows: segment rows are
// numbered after the main rows.
template <int OP>
void launch_stream_op(const DevPass& dp, const Geometry& g, const float* src,
                      const float* src2, const float* own, float* dst, float* dst_seg, int B, hipStream_t s, int* zf) {
    int64_t blocks = ((int64_t)dp.n_stream_tasks + dp.n_stream_seg_tasks + 3) / 4;
    blocks = (blocks + 7) / 8 * 8;
    // outputs larger than the L2s together (8 x 4 MB) are written with streaming stores
    klay::StreamArgs a{};
    a.tasks = dp.stream_tasks;
    a.seg_tasks = dp.stream_seg_tasks;
    a.idx = dp.idx;
    a.entry_row = dp.entry_row;
    a.src = src;
    a.src2 = src2;
    a.own = own;
    a.dst = dst;
    a.dst_seg = dst_seg;
    a.seg_owner = dp.seg_owner;
    a.zero_flag = zf;
    a.n_tasks = dp.n_stream_tasks;
    a.n_seg_tasks = dp.n_stream_seg_tasks;
    a.B = B;
    a.ld = g.ld;
    a.stream_stores = (int64_t)dp.n_main * g.ld * 4 > (int64_t)64 << 20 ? 1 : 0;
    a.n_main = dp.n_main;
    dim3 grid((unsigned)blocks, (unsigned)g.tiles);
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, a); };
    if constexpr (OP == klay::OP_SUM || OP == klay::OP_PROD) {
        if (dp.entry_row) return g.vec == 4 ? launch(klay::stream_kernel<OP, 4, true>) : launch(klay::stream_kernel<OP, 2, true>);
    }
    g.vec == 4 ? launch(klay::stream_kernel<OP, 4, false>) : launch(klay::stream_kernel<OP, 2, false>);
}

void launch_stream(int op, const DevPass& dp, const Geometry& g, const float* src,
                   const float* src2, const float* own, float* dst, float* dst_seg, int B, hipStream_t s, int* zf) {
    if (dp.n_stream_tasks + dp.n_stream_seg_tasks <= 0) return;
    switch (op) {
    case klay::OP_SUM: launch_stream_op<klay::OP_SUM>(dp, g, src, src2, own, dst, dst_seg, B, s, zf); break;
    case klay::OP_PROD: launch_stream_op<klay::OP_PROD>(dp, g, src, src2, own, dst, dst_seg, B, s, zf); break;
    case klay::OP_LSE: launch_stream_op<klay::OP_LSE>(dp, g, src, src2, own, dst, dst_seg, B, s, zf); break;
    case klay::OP_MAX: launch_stream_op<klay::OP_MAX>(dp, g, src, src2, own, dst, dst_seg, B, s, zf); break;
    case klay::OP_PROD_BWD: launch_stream_op<klay::OP_PROD_BWD>(dp, g, src, src2, own, dst, dst_seg, B, s, zf); break;
    case klay::OP_SUM_H: launch_stream_op<klay::OP_SUM_H>(dp, g, src, src2, own, dst, dst_seg, B, s, zf); break;
    case klay::OP_SOFTMAX_H: launch_stream_op<klay::OP_SOFTMAX_H>(dp, g, src, src2, own, dst, dst_seg, B, s, zf); break;
    case klay::OP_SUM_P: launch_stream_op<klay::OP_SUM_P>(dp, g, src, src2, own, dst, dst_seg, B, s, zf); break;
    case klay::OP_PROD_BWD_P: launch_stream_op<klay::OP_PROD_BWD_P>(dp, g, src, src2, own, dst, dst_seg, B, s, zf); break;
    case klay::OP_LSE2: launch_stream_op<klay::OP_LSE2>(dp, g, src, src2, own, dst, dst_seg, B, s, zf); break;
    case klay::OP_MAX2: launch_stream_op<klay::OP_MAX2>(dp, g, src, src2, own, dst, dst_seg, B, s, zf); break;
    case klay::OP_SUMPROD2: launch_stream_op<klay::OP_SUMPROD2>(dp, g, src, src2, own, dst, dst_seg, B, s, zf); break;
    default: launch_stream_op<klay::OP_SOFTMAX_BWD>(dp, g, src, src2, own, dst, dst_seg, B, s, zf); break;
    }
}

struct Profiler {
    klay_circuit* c;
    std::vector<EventRec>* recs;
    hipStream_t s;
    size_t next = 0;
    bool on;
    Profiler(klay_circuit* c_, std::vector<EventRec>* r, hipStream_t s_, bool enable = true)
        : c(c_), recs(r), s(s_), on(enable && c_->profiling) {
        if (on) recs->clear();
    }
    hipEvent_t get() {
        // events of the previous forward stay referenced by ev_fwd while backward records its own
        hipEvent_t e;
        if (hipEventCreate(&e) != hipSuccess) return nullptr;
        c->ev_pool.push_back(e);
        return e;
    }
    // bytes: no-reuse model; min_bytes: compulsory bytes (every distinct row once); < 0: same as bytes
    void begin(int cls, double bytes, double min_bytes = -1.0) {
        if (!on) return;
        EventRec r{cls, get(), get(), bytes, min_bytes < 0 ? bytes : min_bytes};
        if (r.start) (void)hipEventRecord(r.start, s);
        recs->push_back(r);
    }
    void end() {
        if (!on || recs->empty()) return;
        if (recs->back().stop) (void)hipEventRecord(recs->back().stop, s);
    }
};

void release_events(klay_circuit* c) {
    for (hipEvent_t e : c->ev_pool) (void)hipEventDestroy(e);
    c->ev_pool.clear();
    c->ev_fwd.clear();
    c->ev_bwd.clear();
}

klay_status get_workspace(klay_circuit* c, size_t floats, float** base) {
    const size_t bytes = floats * sizeof(float);
    if (c->ws_user) {
        if (bytes > c->ws_user_bytes)
            return fail(KLAY_ENOMEM, "caller workspace too small: need " + std::to_string(bytes) + " bytes");
        *base = static_cast<float*>(c->ws_user);
        return KLAY_OK;
    }
    if (bytes > c->ws_own_bytes) {
        if (c->ws_own) { KLAY_HIP(hipFree(c->ws_own)); c->ws_own = nullptr; c->ws_own_bytes = 0; }
        if (hipMalloc(&c->ws_own, bytes) != hipSuccess) {
            (void)hipGetLastError();
            c->ws_own = nullptr;
            return fail(KLAY_ENOMEM, "hipMalloc of " + std::to_string(bytes) + " workspace bytes failed");
        }
        c->ws_own_bytes = bytes;
    }
    *base = static_cast<float*>(c->ws_own);
    return KLAY_OK;
}

// The memory of a forward pass: the fixed array or the handle's workspace.  `top` becomes 0 where the TopPlan would need more than
// there is and the pass without it does not; with_bwd: whether a reverse sweep can follow.
klay_status forward_workspace(klay_circuit* c, int B, bool static_ws, int& top, bool& with_bwd, float** base, Workspace* lay) {
    with_bwd = !static_ws;
    if (static_ws || c->ws_user) {
        const size_t have = (static_ws ? kStaticWorkspaceBytes : c->ws_user_bytes) / sizeof(float);
        if (with_bwd && top > 0 && workspace_layout(c, B, true, top).total > have && workspace_layout(c, B, true, 0).total <= have) top = 0;
        // the backward regions are part of the layout whenever the workspace can hold them
        if (with_bwd && workspace_layout(c, B, true, top).total > have) with_bwd = false;
        *lay = workspace_layout(c, B, with_bwd, top);
        if (top > 1 && B >= kTopStageB && !lay->top_stage_n) {
            const size_t n = (size_t)c->top.n[(size_t)top - 1] * (size_t)B;
            if (lay->total + n <= have) {
                lay->top_stage = lay->total;
                lay->top_stage_n = n;
            }
        }
        if (!static_ws) return get_workspace(c, lay->total, base);
        if (lay->total > have)
            return fail(KLAY_ENOMEM, "klay_forward_static: this circuit at B = " + std::to_string(B) + " needs " +
                                         std::to_string(lay->total * sizeof(float)) + " workspace bytes, the fixed buffer holds " +
                                         std::to_string(kStaticWorkspaceBytes));
        KLAY_HIP(static_workspace(c->device, base));
        return KLAY_OK;
    }
    // (room for either way at once: a later pass over this batch, which may be captured, allocates nothing)
    *lay = workspace_layout(c, B, true, top);
    klay_status st = get_workspace(c, c->top.first > 0 ? klay_workspace_bytes(c, B, 1) / sizeof(float) : lay->total, base);
    if (st == KLAY_ENOMEM) {
        top = 0;
        *lay = workspace_layout(c, B, true, 0);
        st = get_workspace(c, lay->total, base);
    }
    return st;
}

// Packs host arrays into one buffer with 256-byte aligned starts; returns offsets in ints.
struct Packer {
    std::vector<int32_t> buf;
    size_t add(const std::vector<int32_t>& v) { return add(v.data(), v.size()); }
    size_t add(const std::vector<uint32_t>& v) { return add(reinterpret_cast<const int32_t*>(v.data()), v.size()); }
    size_t add(const int32_t* p, size_t n) {
        size_t off = (buf.size() + kAlignInts - 1) / kAlignInts * kAlignInts;
        buf.resize(off + std::max<size_t>(n, 1), 0);
        if (n) std::memcpy(buf.data() + off, p, n * sizeof(int32_t));
        return off;
    }
};

struct PassOffsets { size_t ptr, idx, seg_owner, comb_ptr, comb_idx, comb_row, tasks, seg_tasks, stream_tasks, stream_seg_tasks; int32_t n_stream_tasks, n_stream_seg_tasks; };

// edge_tasks: the plan may go by launch_edge
PassOffsets pack_pass(Packer& pk, const klay::PassPlan& p, bool edge_tasks) {
    PassOffsets o{};
    o.ptr = pk.add(p.ptr);
    o.idx = pk.add(p.idx);
    o.seg_owner = pk.add(p.seg_owner);
    o.comb_ptr = pk.add(p.comb_ptr);
    o.comb_idx = pk.add(p.comb_idx);
    o.comb_row = pk.add(p.comb_row);
    if (edge_tasks) {
        o.tasks = pk.add(p.tasks);
        o.seg_tasks = pk.add(p.seg_tasks);
    }
    const std::vector<int32_t> main = klay::stream_tasks(p, 0, p.n_main), seg = klay::stream_tasks(p, p.n_main, (int64_t)p.n_main + p.n_seg);
    o.stream_tasks = pk.add(main);
    o.stream_seg_tasks = pk.add(seg);
    o.n_stream_tasks = (int32_t)(main.size() / klay::kTaskWords);
    o.n_stream_seg_tasks = (int32_t)(seg.size() / klay::kTaskWords);
    return o;
}

void bind_pass(DevPass& d, const klay::PassPlan& p, const PassOffsets& o, const int32_t* base, bool compact = false) {
    d.ptr = base + o.ptr;
    d.idx = reinterpret_cast<const uint32_t*>(base + o.idx);
    d.seg_owner = base + o.seg_owner;
    d.comb_ptr = base + o.comb_ptr;
    d.comb_idx = reinterpret_cast<const uint32_t*>(base + o.comb_idx);
    d.comb_row = base + o.comb_row;
    d.tasks = base + o.tasks;
    d.n_tasks = p.n_tasks;
    d.seg_tasks = base + o.seg_tasks;
    d.n_seg_tasks = p.n_seg_tasks;
    d.stream_tasks = base + o.stream_tasks;
    d.stream_seg_tasks = base + o.stream_seg_tasks;
    d.n_stream_tasks = o.n_stream_tasks;
    d.n_stream_seg_tasks = o.n_stream_seg_tasks;
    d.has_weighted = p.has_weighted;
    d.n_light = p.n_main;
    d.main_entries = p.ptr[(size_t)p.n_main];
    if (!compact) {              // (a split row is one entry)
        d.n_light -= p.n_heavy;
        d.main_entries -= p.n_heavy;
    }
    d.seg_entries = (int64_t)p.ptr[(size_t)p.n_main + (size_t)p.n_seg] - p.ptr[(size_t)p.n_main];
    d.n_main = p.n_main;
    d.n_seg = p.n_seg;
    d.n_heavy = p.n_heavy;
    d.n_comb_many = p.n_comb_many;
    for (int32_t h = 0; h < p.n_heavy; ++h) d.longest_comb = std::max(d.longest_comb, p.comb_ptr[(size_t)h + 1] - p.comb_ptr[(size_t)h]);
    for (int32_t i = p.n_main; i < p.n_main + p.n_seg; ++i) d.longest_seg = std::max(d.longest_seg, p.ptr[(size_t)i + 1] - p.ptr[(size_t)i]);
    d.edges = p.edges;
    // distinct source rows (for the compulsory-byte count of the profile)
    uint32_t max_id = 0;
    const size_t n_entries = (size_t)p.ptr[(size_t)p.n_main + (size_t)p.n_seg];
    for (size_t j = 0; j < n_entries; ++j)
        if (p.idx[j] != klay::kSkipRow) max_id = std::max(max_id, p.idx[j] & klay::kIdMask);
    std::vector<uint8_t> seen((size_t)max_id + 1, 0);
    for (size_t j = 0; j < n_entries; ++j)
        if (p.idx[j] != klay::kSkipRow && !seen[p.idx[j] & klay::kIdMask]) { seen[p.idx[j] & klay::kIdMask] = 1; ++d.n_src; }
}

// sizes of the layers that the persistent kernels may run
void describe_tails(klay_circuit* c) {
    const klay::CircuitPlan& p = c->plan;
    const size_t layers = (size_t)p.num_layers + 1;
    auto room = [&](ColTail& t) {
        for (std::vector<int64_t>* v : {&t.n, &t.kept, &t.at, &t.e, &t.words[0], &t.words[1], &t.own_at, &t.share}) v->assign(layers, 0);
        t.launches.assign(layers, 0);
    };
    if (p.tail_first > 0) {
        ColTail& t = c->tail;
        room(t);
        t.first = p.tail_first;
        t.rows = p.col_rows;
        for (size_t l = (size_t)t.first - 1; l < layers; ++l) {
            const klay::LayerPlan& lay = p.layers[l];
            t.n[l] = t.kept[l] = lay.n;
            t.at[l] = p.col_off[l];
            t.e[l] = lay.e;
            t.words[0][l] = (int64_t)lay.col_fwd.blocks.size();
            t.words[1][l] = (int64_t)lay.col_bwd.blocks.size();
            t.launches[l] = lay.fwd.n_heavy > 0 ? 2 : 1;
            t.share[l] = lay.col_fwd.share;
        }
    }
    if (p.top.first > 0) {
        ColTail& t = c->top;
        room(t);
        t.first = p.top.first;
        t.rows = p.top.rows;
        int64_t own = 0;
        for (size_t l = (size_t)t.first - 1; l < layers; ++l) {
            const klay::TopPlan::Level& lev = p.top.level((int32_t)l);
            t.n[l] = lev.n;
            t.kept[l] = lev.kept;
            t.at[l] = lev.at;
            t.e[l] = lev.e;
            t.words[0][l] = (int64_t)lev.fwd.blocks.size();
            t.words[1][l] = (int64_t)lev.bwd.blocks.size();
            t.own_at[l] = own;
            own += lev.n;
            t.launches[l] = lev.launches;
            t.share[l] = lev.fwd.share;
        }
    }
}

// The variables that the circuit has literals of, for the persistent forward kernel, where that saves its workgroups a round over the variables (a weight
// is asked for when the variable's number has arrived): their positive literals' rows of layer 0, the negated ones', their numbers.  Forward of 217
// nodes over 12 of so many variables, us, without / with: 2000 variables B = 1 9.2 / 9.0, B = 128 12.1 / 9.5; 20000 13.2 / 9.1, 37.7 / 9.5; 100000
// 31.8 / 9.2, 157 / 9.5; klay_forward_static with 100000 23.9 / 6.6, 41.8 / 6.9.
std::vector<int32_t> leaf_list(const klay::CircuitPlan& p, int32_t& n) {
    std::vector<int32_t> used, list;
    for (int32_t v = 0; v < p.num_vars; ++v)
        if (p.pos_row[(size_t)v] >= 0 || p.neg_row[(size_t)v] >= 0) used.push_back(v);
    auto rounds = [](size_t count) { return (count + klay::kColThreads - 1) / klay::kColThreads; };
    if (rounds(used.size()) >= rounds((size_t)p.num_vars)) used.clear();
    n = (int32_t)used.size();
    for (int32_t v : used) list.push_back(p.pos_row[(size_t)v]);
    for (int32_t v : used) list.push_back(p.neg_row[(size_t)v]);
    list.insert(list.end(), used.begin(), used.end());
    return list;
}

klay_status upload(klay_circuit* c) {
    const klay::CircuitPlan& p = c->plan;
    Packer pk;
    const int L = p.num_layers;
    // Streams of the persistent kernels: per wave and direction the lines and descriptors of all candidate layers
    // back to back, in the order the sweep visits them.
    struct TailOffsets { size_t layers = 0, blocks[2] = {0, 0}, units[2] = {0, 0}, tables = 0; };
    auto pack_tail = [&](ColTail& t, auto plan_of) {
        TailOffsets o;
        std::vector<klay::ColLayer> starts((size_t)(L - t.first + 1));
        std::vector<uint32_t> blocks[2], units[2], tables;
        for (int l = t.first; l <= L; ++l) {
            starts[(size_t)(l - t.first)].n = (int32_t)t.kept[(size_t)l];
            starts[(size_t)(l - t.first)].at = (int32_t)t.at[(size_t)l];
        }
        constexpr size_t kTableWords = (size_t)klay::kDescTable * klay::kDescWords;
        for (int backward = 0; backward < 2; ++backward) {
            std::vector<uint32_t>& out = blocks[backward];
            for (int w = 0; w < klay::kColWaves; ++w)
                for (int step = 0; step <= L - t.first; ++step) {
                    const int l = backward ? L - step : t.first + step;
                    const klay::ColPlan& cp = plan_of(l, backward);
                    klay::ColLayer& at = starts[(size_t)(l - t.first)];
                    (backward ? at.bwd_block : at.fwd_block)[w] = (int32_t)(out.size() / klay::kBlockWords);
                    (backward ? at.bwd_table : at.fwd_table)[w] = (int32_t)(tables.size() / kTableWords);
                    out.insert(out.end(), cp.blocks.begin() + (size_t)cp.block_at[w] * klay::kBlockWords,
                               cp.blocks.begin() + (size_t)cp.block_at[w + 1] * klay::kBlockWords);
                    tables.insert(tables.end(), cp.tables.begin() + (size_t)cp.table_at[w] * kTableWords,
                                  cp.tables.begin() + (size_t)cp.table_at[w + 1] * kTableWords);
                }
            // the narrow layers at the top, as units: dealt to the waves in turn, an empty one for a wave that has none
            const int step_waves = !backward ? klay::kColFwdWaves : &t == &c->top ? klay::kTopBwdWaves : klay::kColBwdWaves;
            int32_t& narrow = t.narrow[backward];
            for (narrow = L + 1; narrow > t.first && !plan_of(narrow - 1, backward).units.empty(); --narrow) {}
            std::vector<uint32_t>& us = units[backward];
            for (int w = 0; w < klay::kColWaves; ++w) {
                auto add = [&](uint32_t bits) {       // an empty unit
                    for (int i = 0; i < klay::kUnitWords; ++i) us.push_back(i % 4 ? 0u : bits | (uint32_t)klay::kUnitIdleSlot);
                };
                auto count = [&](int l) { return (int)(plan_of(l, backward).units.size() / klay::kUnitWords); };
                int until = L;                        // forward: a wave stops after its last rows
                if (!backward && w > 0 && p.num_roots <= kRootsOneWave)
                    while (until >= narrow && count(until) <= w) --until;
                for (int step = 0; step <= L - narrow; ++step) {
                    const int l = backward ? L - step : narrow + step;
                    klay::ColLayer& at = starts[(size_t)(l - t.first)];
                    (backward ? at.bwd_unit : at.fwd_unit)[w] = (int32_t)(us.size() / klay::kUnitWords);
                    if (l > until) continue;          // (the unit that ends it)
                    const uint32_t kind = (l & 1) == 0 ? klay::kUnitOr : 0u;
                    if (w >= step_waves || w >= count(l)) add(klay::kUnitNew | klay::kUnitIdle | kind);
                    else
                        for (int u = w; u < count(l); u += step_waves) {
                            const uint32_t* from = plan_of(l, backward).units.data() + (size_t)u * klay::kUnitWords;
                            us.insert(us.end(), from, from + klay::kUnitWords);
                            for (int i = 0; i < klay::kUnitWords; i += 4) us[us.size() - (size_t)klay::kUnitWords + (size_t)i] |= kind | (u == w ? klay::kUnitNew : 0u);
                        }
                }
                add(klay::kUnitEnd);
            }
            t.n_units[backward] = (int32_t)(us.size() / klay::kUnitWords);
            us.resize(us.size() + (size_t)klay::kUnitsAhead * klay::kUnitWords, 0u);      // read ahead
            t.n_blocks[backward] = (int32_t)(out.size() / klay::kBlockWords);
            out.resize(out.size() + klay::kBlockWords, 0u);      // the waves read one block and one table ahead
        }
        tables.resize(tables.size() + kTableWords, 0u);
        static_assert(sizeof(klay::ColLayer) % sizeof(int32_t) == 0, "must pack into ints");
        for (int i = 0; i < 2; ++i) { o.blocks[i] = pk.add(blocks[i]); o.units[i] = pk.add(units[i]); }
        o.tables = pk.add(tables);
        o.layers = pk.add(reinterpret_cast<const int32_t*>(starts.data()), starts.size() * sizeof(klay::ColLayer) / sizeof(int32_t));
        return o;
    };
    TailOffsets o_tail, o_top;
    if (c->tail.first > 0)
        o_tail = pack_tail(c->tail, [&](int l, int backward) -> const klay::ColPlan& {
            return backward ? p.layers[(size_t)l].col_bwd : p.layers[(size_t)l].col_fwd;
        });
    size_t o_own = 0, o_act_row = 0, o_top_root_pos = 0, o_top_top_ptr = 0, o_top_top_root = 0, o_top_multi = 0;
    if (c->top.first > 0) {
        const klay::TopPlan& top = p.top;
        o_top = pack_tail(c->top, [&](int l, int backward) -> const klay::ColPlan& { return backward ? top.level(l).bwd : top.level(l).fwd; });
        std::vector<int32_t> own;
        for (const klay::TopPlan::Level& lev : top.levels) own.insert(own.end(), lev.own.begin(), lev.own.end());
        o_own = pk.add(own);
        o_act_row = pk.add(top.act_row);
        o_top_root_pos = pk.add(top.root_pos);
        o_top_top_ptr = pk.add(top.top_ptr);
        o_top_top_root = pk.add(top.top_root);
        o_top_multi = pk.add(top.multi);
    }
    struct Compact { klay::PassPlan plan; size_t out_row = 0, entry_row = 0; };
    std::vector<Compact> kept((size_t)L + 1);           // the AND layers' plans without the fused rows
    std::vector<PassOffsets> fo((size_t)L + 1), bo((size_t)L + 1), fko((size_t)L + 1), f2o((size_t)L + 1);
    for (int l = 1; l <= L; ++l) {
        fo[(size_t)l] = pack_pass(pk, p.layers[(size_t)l].fwd, c->small_batch_edges);
        bo[(size_t)l] = pack_pass(pk, p.layers[(size_t)l].bwd, c->small_batch_edges);
        if (!p.layers[(size_t)l].fwd_kept.ptr.empty()) {
            Compact& k = kept[(size_t)l];
            std::vector<int32_t> out_row, entry_row;
            klay::compact_pass(p.layers[(size_t)l].fwd_kept, k.plan, out_row, entry_row);
            fko[(size_t)l] = pack_pass(pk, k.plan, false);
            k.out_row = pk.add(out_row);
            k.entry_row = pk.add(entry_row);
        }
        if (!p.layers[(size_t)l].fwd2.ptr.empty()) f2o[(size_t)l] = pack_pass(pk, p.layers[(size_t)l].fwd2, false);
    }
    std::vector<size_t> mo((size_t)L + 1, 0);
    for (int l = 2; l <= L; l += 2) mo[(size_t)l] = pk.add(p.layers[(size_t)l].multi);
    const size_t o_leaf_list = pk.add(leaf_list(p, c->n_leaf_list));
    const size_t o_pos = pk.add(p.pos_row), o_neg = pk.add(p.neg_row), o_root = pk.add(p.root_pos);
    const size_t o_tptr = pk.add(p.top_ptr), o_troot = pk.add(p.top_root);

    KLAY_HIP(hipSetDevice(c->device));
    {
        float* static_ws = nullptr;      // klay_forward_static's workspace on this device
        KLAY_HIP(static_workspace(c->device, &static_ws));
    }
    c->index_bytes = pk.buf.size() * sizeof(int32_t);
    if (hipMalloc(reinterpret_cast<void**>(&c->d_index), c->index_bytes) != hipSuccess) {
        (void)hipGetLastError();
        return fail(KLAY_ENOMEM, "hipMalloc of " + std::to_string(c->index_bytes) + " index bytes failed");
    }
    KLAY_HIP(hipMemcpy(c->d_index, pk.buf.data(), c->index_bytes, hipMemcpyHostToDevice));
    const int32_t* base = c->d_index;
    c->dl.resize((size_t)L + 1);
    int64_t row0 = 0;
    for (int l = 0; l <= L; ++l) {
        DevLayer& d = c->dl[(size_t)l];
        d.n = p.layers[(size_t)l].n;
        d.e = p.layers[(size_t)l].e;
        d.row0 = row0;
        row0 += d.n;
        if (l >= 1) {
            bind_pass(d.fwd, p.layers[(size_t)l].fwd, fo[(size_t)l], base);
            bind_pass(d.bwd, p.layers[(size_t)l].bwd, bo[(size_t)l], base);
            const klay::LayerPlan& lp = p.layers[(size_t)l];
            d.n_fused = lp.n_fused;
            if (!lp.fwd_kept.ptr.empty()) {
                bind_pass(d.fwd_kept, kept[(size_t)l].plan, fko[(size_t)l], base, true);
                d.fwd_kept.out_row = base + kept[(size_t)l].out_row;
                d.fwd_kept.entry_row = base + kept[(size_t)l].entry_row;
                d.has_fwd_kept = true;
            }
            if (!lp.fwd2.ptr.empty()) { bind_pass(d.fwd2, lp.fwd2, f2o[(size_t)l], base); d.has_fwd2 = true; }
            if ((l & 1) == 0) {
                d.multi = reinterpret_cast<const uint32_t*>(base + mo[(size_t)l]);
                for (uint32_t w : p.layers[(size_t)l].multi) d.has_multi = d.has_multi || w != 0;
            }
        }
    }
    // The one-gather form needs every layer below alias_top to either store encoded rows or read weighted
    // edges, not both: OR rows have AND parents only, so this holds for every circuit the layerizer accepts.
    c->one_gather = true;
    for (int l = 2; l < p.alias_top; l += 2)
        if (c->dl[(size_t)l].has_multi && c->dl[(size_t)l + 1].bwd.has_weighted) c->one_gather = false;
    c->d_leaf_list = base + o_leaf_list;
    c->d_pos_row = base + o_pos;
    c->d_neg_row = base + o_neg;
    c->d_root_pos = base + o_root;
    c->d_top_ptr = base + o_tptr;
    c->d_top_root = base + o_troot;
    auto bind_tail = [&](ColTail& t, const TailOffsets& o) {
        t.layers = reinterpret_cast<const klay::ColLayer*>(base + o.layers);
        for (int i = 0; i < 2; ++i) {
            t.blocks[i] = reinterpret_cast<const klay::Line*>(base + o.blocks[i]);
            t.units[i] = reinterpret_cast<const klay::Line*>(base + o.units[i]);
        }
        t.tables = reinterpret_cast<const klay::Desc*>(base + o.tables);
    };
    if (c->tail.first > 0) {
        bind_tail(c->tail, o_tail);
        c->tail.root_pos = c->d_root_pos;
        c->tail.top_ptr = c->d_top_ptr;
        c->tail.top_root = c->d_top_root;
    }
    if (c->top.first > 0) {
        bind_tail(c->top, o_top);
        c->top.own = base + o_own;
        c->top.act_row = base + o_act_row;
        c->top.root_pos = base + o_top_root_pos;
        c->top.top_ptr = base + o_top_top_ptr;
        c->top.top_root = base + o_top_top_root;
        if ((L & 1) == 0) c->top.multi = reinterpret_cast<const uint32_t*>(base + o_top_multi);
    }
    return KLAY_OK;
}

// Algorithmic bytes (no-reuse model) of a gather-reduce over `rows` output rows with `entries` index
// entries: every entry gathers one row (two in the two-gather softmax adjoint), every output row is written
// once (and, in the reverse-sweep ops other than the plain sum, reads its own value row), plus the index
// entries themselves.
double pass_bytes(int op, double entries, double rows, int B) {
    const double per_entry = op == klay::OP_SOFTMAX_BWD ? 2.0 : 1.0;
    const double per_row = (op == klay::OP_SUM || op == klay::OP_PROD || op == klay::OP_LSE || op == klay::OP_MAX ||
                            op == klay::OP_LSE2 || op == klay::OP_MAX2 || op == klay::OP_SUMPROD2) ? 1.0 : 2.0;
    return 4.0 * B * (per_entry * entries + per_row * rows) + 4.0 * (entries + rows);
}

// Compulsory bytes of the same pass: every distinct source row and every output row moves once.
double pass_min_bytes(int op, double entries, double rows, double n_src, int B) {
    const double f = op == klay::OP_SOFTMAX_BWD ? 2.0 : 1.0;
    return 4.0 * B * f * (n_src + rows) + 4.0 * (entries + rows);
}

// Combine pass of the split rows for batches wider than 32 columns (combine_kernel); `many`: rows that take a workgroup each.
template <int OP>
void launch_combine_op(const klay::PassArgs& a, const Geometry& g, int32_t many, hipStream_t s) {
    constexpr int NW = 8;
    dim3 grid((unsigned)(many + (a.n_main - many + NW - 1) / NW), (unsigned)g.tiles);
    if (g.vec == 4) hipLaunchKernelGGL((klay::combine_kernel<OP, 4, NW>), grid, dim3(NW * 64), 0, s, a, many);
    else if (g.vec == 2) hipLaunchKernelGGL((klay::combine_kernel<OP, 2, NW>), grid, dim3(NW * 64), 0, s, a, many);
    else hipLaunchKernelGGL((klay::combine_kernel<OP, 1, NW>), grid, dim3(NW * 64), 0, s, a, many);
}

// B <= 32: a workgroup of four waves per split row as well, 64 / W partial rows at a time in a wave, where a row has more than
// kShortComb partial rows; shorter lists take a lane group each (launch_pass), which needs fewer workgroups.  us with a limit of
// 0 / 4 / 8 / 16 / 32 (power-law fan-ins): 9400 nodes max B = 1 216 / 183 / 184 / 185 / 184, 12000 nodes forward B = 6
// 288 / 266 / 265 / 267 / 278, 29000 nodes training B = 18 316 / 316 / 317 / 317 / 330
constexpr int32_t kShortComb = 8;
template <int OP>
void launch_combine_small(const klay::PassArgs& a, const Geometry& g, hipStream_t s) {
    dim3 grid((unsigned)a.n_main);
    switch (g.w) {
    case 32: hipLaunchKernelGGL((klay::combine_small_kernel<OP, 32>), grid, dim3(256), 0, s, a); break;
    case 16: hipLaunchKernelGGL((klay::combine_small_kernel<OP, 16>), grid, dim3(256), 0, s, a); break;
    case 8: hipLaunchKernelGGL((klay::combine_small_kernel<OP, 8>), grid, dim3(256), 0, s, a); break;
    case 4: hipLaunchKernelGGL((klay::combine_small_kernel<OP, 4>), grid, dim3(256), 0, s, a); break;
    case 2: hipLaunchKernelGGL((klay::combine_small_kernel<OP, 2>), grid, dim3(256), 0, s, a); break;
    default: hipLaunchKernelGGL((klay::combine_small_kernel<OP, 1>), grid, dim3(256), 0, s, a); break;
    }
}

void launch_combine(int op, const klay::PassArgs& a, const Geometry& g, int32_t longest, int32_t many, hipStream_t s) {
    if (a.n_main <= 0) return;
    if (g.w != 64 && longest <= kShortComb) {
        launch_pass(op, a, s);
        return;
    }
    if (g.w != 64) {
        switch (op) {
        case klay::OP_SUM: launch_combine_small<klay::OP_SUM>(a, g, s); break;
        case klay::OP_PROD: launch_combine_small<klay::OP_PROD>(a, g, s); break;
        case klay::OP_LSE: launch_combine_small<klay::OP_LSE>(a, g, s); break;
        case klay::OP_MAX: launch_combine_small<klay::OP_MAX>(a, g, s); break;
        case klay::OP_SUM_H: launch_combine_small<klay::OP_SUM_H>(a, g, s); break;
        case klay::OP_SUM_P: launch_combine_small<klay::OP_SUM_P>(a, g, s); break;
        default: launch_pass(op, a, s); break;
        }
        return;
    }
    switch (op) {
    case klay::OP_SUM: launch_combine_op<klay::OP_SUM>(a, g, many, s); break;
    case klay::OP_PROD: launch_combine_op<klay::OP_PROD>(a, g, many, s); break;
    case klay::OP_LSE: launch_combine_op<klay::OP_LSE>(a, g, many, s); break;
    case klay::OP_MAX: launch_combine_op<klay::OP_MAX>(a, g, many, s); break;
    case klay::OP_SUM_H: launch_combine_op<klay::OP_SUM_H>(a, g, many, s); break;
    case klay::OP_SUM_P: launch_combine_op<klay::OP_SUM_P>(a, g, many, s); break;
    default: launch_pass(op, a, s); break;
    }
}

klay::PassArgs combine_args(const DevPass& dp, const float* seg_rows, const float* own, float* dst, const Geometry& g,
                            int B, int* zero_flag) {
    klay::PassArgs cmb{};
    cmb.ptr = dp.comb_ptr;
    cmb.idx = dp.comb_idx;
    cmb.src = seg_rows;
    cmb.own = own;               // OP_SUM_H, OP_SUM_P: the value rows of the nodes the combine pass writes
    cmb.zero_flag = zero_flag;
    cmb.out_row = dp.comb_row;
    cmb.dst = dst;
    cmb.dst_seg = nullptr;
    cmb.row_begin = 0;
    cmb.n_main = dp.n_heavy;
    cmb.n_total = dp.n_heavy;
    cmb.B = B;
    cmb.ld = g.ld;
    return cmb;
}

// The main rows and the combine rows of a layer in one launch (32 < B <= 64; its segments have run in a launch before it).
template <int OP, int COP>
void launch_pass_combine_op(klay::PassArgs a, const klay::PassArgs& cmb, int32_t many, hipStream_t s) {
    const int vec = deal_lanes(a);
    const int comb_blocks = (many + (cmb.n_main - many + 3) / 4 + 7) / 8 * 8;
    dim3 grid(row_blocks(a.n_total, a.lanes) + (unsigned)comb_blocks);
    if (vec == 4) hipLaunchKernelGGL((klay::pass_combine_kernel<OP, COP, 4>), grid, dim3(256), 0, s, a, comb_blocks, cmb, many);
    else if (vec == 2) hipLaunchKernelGGL((klay::pass_combine_kernel<OP, COP, 2>), grid, dim3(256), 0, s, a, comb_blocks, cmb, many);
    else hipLaunchKernelGGL((klay::pass_combine_kernel<OP, COP, 1>), grid, dim3(256), 0, s, a, comb_blocks, cmb, many);
}

bool pass_combine_pair(int op, int combine_op) {
    using namespace klay;
    return (op == combine_op && (op == OP_SUM || op == OP_PROD || op == OP_LSE || op == OP_MAX || op == OP_SUM_H || op == OP_SUM_P)) ||
           (op == OP_SOFTMAX_H && combine_op == OP_SUM) || (op == OP_PROD_BWD && combine_op == OP_SUM) ||
           (op == OP_PROD_BWD_P && combine_op == OP_SUM_P);
}

void launch_pass_combine(int op, const klay::PassArgs& a, const klay::PassArgs& cmb, int32_t many, hipStream_t s) {
    using namespace klay;
    switch (op) {
    case OP_SUM: launch_pass_combine_op<OP_SUM, OP_SUM>(a, cmb, many, s); break;
    case OP_PROD: launch_pass_combine_op<OP_PROD, OP_PROD>(a, cmb, many, s); break;
    case OP_LSE: launch_pass_combine_op<OP_LSE, OP_LSE>(a, cmb, many, s); break;
    case OP_MAX: launch_pass_combine_op<OP_MAX, OP_MAX>(a, cmb, many, s); break;
    case OP_SUM_H: launch_pass_combine_op<OP_SUM_H, OP_SUM_H>(a, cmb, many, s); break;
    case OP_SOFTMAX_H: launch_pass_combine_op<OP_SOFTMAX_H, OP_SUM>(a, cmb, many, s); break;
    case OP_SUM_P: launch_pass_combine_op<OP_SUM_P, OP_SUM_P>(a, cmb, many, s); break;
    case OP_PROD_BWD: launch_pass_combine_op<OP_PROD_BWD, OP_SUM>(a, cmb, many, s); break;
    default: launch_pass_combine_op<OP_PROD_BWD_P, OP_SUM_P>(a, cmb, many, s); break;
    }
}

// 64 < B <= 128: whether a pass takes the generic kernel, four columns per lane, instead of the streaming one, two.  Up to 84
// columns three rows fit a wave, of which the streaming kernel would use 42 lanes at most.  Above, both use as many, and the
// streaming kernel's balanced tasks win, except where most entries are segments, rows of one length.  (The plans of fused rows have no
// generic kernel.)  Training steps, us, streaming / generic throughout / this rule: 800000 nodes B = 70 623 / 558 / 558, B = 100
// 654 / 676 / 638, B = 128 705 / 720 / 691, real semiring B = 100 710 / 730 / 666; 1e6 nodes, 1e7 edges of power-law fan-ins B = 100
// 1519 / 1405 / 1449, B = 128 1561 / 1462 / 1511.  (The last two: what gains there by the generic kernel are long rows that are not split, too.)
bool generic_pair(int op, const DevPass& dp, int B) {
    if (op == klay::OP_LSE2 || op == klay::OP_MAX2 || op == klay::OP_SUMPROD2) return false;
    return B <= 84 || dp.seg_entries > dp.main_entries;
}

// One layer-level gather-reduce: main rows and segments of split rows in one launch (timed under `cls`), then the combine
// pass; in large layers at 32 < B <= 64 the segments first (KLAY_K_SPLIT), then main rows and combine rows (KLAY_K_MAIN_COMBINE).  B > 64: the streaming kernel, two or four columns per lane (see generic_pair).  Below, the generic kernel (a lane group per row, up to
// four columns per lane): a compute unit takes 16 cycles per vector memory instruction, so a wave that reads a row of at most 64 floats at a
// time stays at a quarter of the rate (1e7 edges of power-law fan-ins, us with the streaming kernel, one column per lane / now: 1e6 nodes,
// training step at B = 50 998 / 882; 290000 nodes, forward at B = 64 411 / 384).
void run_pass_set(int op, int combine_op, const DevPass& dp, const float* src, const float* src2,
                  const float* own, float* dst, float* seg_rows, const Geometry& g, int B, hipStream_t s,
                  Profiler& prof, int cls, int* zero_flag = nullptr) {
    const bool edges = prof.c->small_batch_edges;
    klay::PassArgs a{};
    a.zero_flag = zero_flag;
    a.ptr = dp.ptr;
    a.idx = dp.idx;
    a.src = src;
    a.src2 = src2;
    a.own = own;
    a.seg_owner = dp.seg_owner;
    a.out_row = dp.out_row;
    a.dst = dst;
    a.dst_seg = seg_rows;
    a.n_main = dp.n_main;
    a.n_total = dp.n_main + dp.n_seg;
    a.B = B;
    a.ld = g.ld;
    const double light_rows = (double)dp.n_light;
    if (g.w == 64 && g.vec == 1 && dp.n_heavy > 0 && dp.main_entries + dp.seg_entries > kSmallPassEntries && light_rows > 0 && pass_combine_pair(op, combine_op)) {
        prof.begin(KLAY_K_SPLIT, pass_bytes(op, (double)dp.seg_entries, (double)dp.n_seg, B),
                   pass_min_bytes(op, (double)dp.seg_entries, (double)dp.n_seg, 0.0, B));
        a.row_begin = dp.n_main;
        launch_pass(op, a, s, dp.longest_seg);
        prof.end();
        prof.begin(KLAY_K_MAIN_COMBINE,
                   pass_bytes(op, (double)dp.main_entries, light_rows, B) + pass_bytes(combine_op, (double)dp.n_seg, (double)dp.n_heavy, B),
                   pass_min_bytes(op, (double)dp.main_entries, light_rows, (double)dp.n_src, B) +
                       pass_bytes(combine_op, (double)dp.n_seg, (double)dp.n_heavy, B));
        a.row_begin = 0;
        a.n_total = dp.n_main;
        launch_pass_combine(op, a, combine_args(dp, seg_rows, own, dst, g, B, zero_flag), dp.n_comb_many, s);
        prof.end();
        return;
    }
    prof.begin(cls, pass_bytes(op, (double)(dp.main_entries + dp.seg_entries), light_rows + dp.n_seg, B),
               pass_min_bytes(op, (double)(dp.main_entries + dp.seg_entries), light_rows + dp.n_seg, (double)dp.n_src, B));
    float* seg_base = seg_rows - (ptrdiff_t)dp.n_main * g.ld;     // only indexed with rows >= n_main
    if (g.w == 64 && g.vec >= 2 && !(g.vec == 2 && generic_pair(op, dp, B))) {
        launch_stream(op, dp, g, src, src2, own, dst, seg_base, B, s, zero_flag);
    } else if (g.w != 64 && edges) {
        launch_edge(op, dp, g, src, src2, own, dst, seg_base, B, s, zero_flag);
    } else {
        a.row_begin = 0;
        launch_pass(op, a, s);
    }
    prof.end();
    if (dp.n_heavy > 0) {
        const klay::PassArgs cmb = combine_args(dp, seg_rows, own, dst, g, B, zero_flag);
        prof.begin(KLAY_K_COMBINE, pass_bytes(combine_op, (double)dp.n_seg, (double)dp.n_heavy, B));
        launch_combine(combine_op, cmb, g, dp.longest_comb, dp.n_comb_many, s);
        prof.end();
    }
}

// ---- persistent kernels for the top layers -----------------------------------------------------
struct TailChoice {
    int first = 0;       // first layer run by the persistent kernel (0: not used)
    int ct = 1;          // batch columns that share the LDS in the rule below
    int nmax = 0;        // longest of the layers
};

// The layers the persistent kernels take: as many as fit when `ct` columns share the LDS of a compute unit.  Up to 256
// columns every workgroup (a column) has a compute unit of its own; beyond, the launches of the wider layers, which
// fill the chip, are left to the ordinary kernels.  At most 4, as the kernels have (tail_columns).  us with 2 / 4 / 8 at most:
// 30000 nodes in 24 layers training B = 1800 297 / 296 / 417, 100k nodes forward B = 520 182 / 152 / 152, B = 4096
// 976 / 867 / 840, 131000 nodes in 48 layers training B = 2048 1044 / 1181 / 1293, forward B = 520 188 / 178 / 178.
int tail_ct(int B, int most) {
    int ct = 1;
    while (ct < most && (B + ct - 1) / ct > 256) ct *= 2;
    return ct;
}

// Largest suffix of the candidate layers whose two value arrays of ct columns fit the LDS of a workgroup.  The arrays
// hold the layers first .. L, and layer 0 as well
// when the kernel starts at layer 1 and evaluates the leaf layer itself.  At least two layers,
// otherwise a kernel of its own is not worth it.
TailChoice choose_tail(const klay_circuit* c, int ct) {
    TailChoice t;
    const klay::CircuitPlan& p = c->plan;
    const int lowest = p.tail_first;
    if (lowest <= 0 || c->tail_lds_bytes == 0) return t;
    t.ct = ct;
    const int L = p.num_layers;
    const int64_t words = (int64_t)(c->tail_lds_bytes / sizeof(float));
    int64_t nmax = 0;
    int first = 0;
    for (int l = L; l >= lowest; --l) {
        int64_t n2 = std::max(nmax, p.layers[(size_t)l].n);
        if (l == 1) n2 = std::max(n2, p.layers[0].n);
        if (2 * (n2 + 1) * t.ct > words) break;
        // the layer below is loaded into LDS as well
        if (2 * (std::max(n2, p.layers[(size_t)l - 1].n) + klay::kColSlots + 3) > words) break;
        nmax = n2;
        first = l;
    }
    if (first == 0 || L - first + 1 < 2) return t;
    t.first = first;
    t.nmax = (int)nmax;
    return t;
}

TailChoice choose_tail_fwd(const klay_circuit* c, int B) { return choose_tail(c, tail_ct(B, 4)); }

// The first layer that the forward kernel takes from the TopPlan at a batch of B (0: none, the layers of the plan itself go the
// other ways): the choice with the least time by a rough account.  In the persistent kernels a layer takes the time of its longest
// wave and about 2000 cycles, as it does where it goes by runs (units, which came later, take 700, so that the account is against the kernel
// where the top is narrow); a launch takes 3.5 us and what it gathers, from the caches, at 10 TB/s.  us, launches throughout / this
// choice (first layer), forward and training step:
//   290000 nodes in 30 layers, 1e7 edges, B = 1 240 / 199 (13), 408 / 356; B = 64 422 / 361 (13), 806 / 716; B = 500 1540 / 1445 (16),
//   3597 / 3468; 92000 nodes in 40 layers, 1.2e6 edges, B = 1 289 / 139 (3), 468 / 293; B = 64 322 / 151 (3), 536 / 333; B = 1000 740 / 566 (17),
//   1464 / 1323; 30000 nodes in 24 layers, 2.3e5 edges, B = 64 129 / 45 (1), 244 / 107.
// The rest of this comment was measured before there were units.
// First layers above 1 only up to B = 1024: 23200 nodes in 30 layers at B = 2000 536 / 483 (2), but 1080 / 1181 in training.  (The
// reverse kernel could leave the sweep to the launches earlier; that gains at most 8%, 92000 nodes training B = 1 284 against 259,
// and loses for B >= 64.)
// (Layers of the plan itself that the persistent kernel would take otherwise, choose_tail_fwd, count as launches here.  With what that kernel saves
// counted, no choice is another one: 37 circuits with such layers, 29 batches of 1 to 4000 columns.)
// real_training: a forward pass in the real semiring in a training loop.  Its reverse sweep goes by launches over rows that the values of all
// levels are put into first, and without the reverse kernel for the layers of the plan itself (7: a row of theirs for rows of levels).  Training
// step, us, launches / TopPlan: 27000 nodes in 42 layers (20 of the plan itself) B = 256 442 / 385, B = 400 406 / 415, B = 1000 429 / 689; 21000
// nodes in 44 layers B = 513 858 / 797, B = 1000 708 / 854; 16000 nodes in 30 layers B = 1000 465 / 361.
int choose_top(const klay_circuit* c, int B, bool real_training) {
    const ColTail& t = c->top;
    if (t.first <= 0 || c->tail_lds_bytes == 0) return 0;
    const int L = c->plan.num_layers;
    double inside = 0, outside = 0, best = 0;          // us of the layers from l on, in the kernel and outside; what the best choice saves
    int first = 0, launches = 0, first_launches = 0;   // first: of the best choice
    int64_t size[2] = {0, 0};                          // as tail_lds
    auto room = [&](int l) { size[l & 1] = std::max(size[l & 1], (t.n[(size_t)l] + klay::kColSlots + 3) / 4 * 4); };
    room(L);
    for (int l = L; l >= t.first; --l) {
        inside += (2000.0 + (double)t.share[(size_t)l]) / 2000.0;
        outside += 3.5 * t.launches[(size_t)l] + (double)t.e[(size_t)l] * B / 2.5e6;
        launches += t.launches[(size_t)l];
        room(l - 1);
        if (l > std::min(c->plan.alias_top, L - 1)) continue;
        if ((size_t)(size[0] + size[1]) * sizeof(float) > c->tail_lds_bytes) break;
        // columns in turns, several at once take longer than one
        const int ct = tail_columns(B, size, c->tail_lds_bytes, false), turns = (B + 256 * ct - 1) / (256 * ct);
        // from rows to columns and, in a reverse sweep, back
        const double transposed = l > 1 ? 5.0 + (double)(t.n[(size_t)l - 1] + t.rows - t.at[(size_t)l]) * B * 2e-6 : 0.0;
        const double saved = outside - turns * (4.0 + (ct == 4 ? 1.9 : ct == 2 ? 1.3 : 1.0) * inside) - transposed;
        if (saved > best && (l == 1 || B <= 1024)) {
            best = saved;
            first = l;
            first_launches = launches;
        }
    }
    if (first > 0 && real_training && (double)(t.rows - t.at[(size_t)first] + 7 * c->tail_rows) * B > 1.4e6 * first_launches) return 0;
    return first;
}

// Rows of the layer below the forward kernel's first one if that layer gets a place in the column-major buffer (where
// the kernel reads it as one run per column, and the reverse kernel its values): where ct arrays of its length fit the
// LDS too.  0: no place (the kernel evaluates the leaf layer itself, or reads the layer from its rows).
int64_t tail_stage_rows(const klay_circuit* c, const TailChoice& t) {
    if (t.first < 2) return 0;
    const int64_t nb = c->plan.layers[(size_t)t.first - 1].n;
    const int64_t rows = std::max<int64_t>(nb, t.nmax);
    return (size_t)2 * (size_t)(rows + 1) * t.ct * sizeof(float) <= c->tail_lds_bytes ? nb : 0;
}
// What the workspace holds for it.  (Up to 8 columns here: klay_workspace_bytes, and with it the batches that the entry point
// with a fixed buffer takes, stay what they were before the limit of 4.)
int64_t tail_stage_rows(const klay_circuit* c, int B) { return tail_stage_rows(c, choose_tail(c, tail_ct(B, 8))); }

// floats of the two LDS arrays that hold `n` values of the layers lowest .. L by turns; [0]: the one with layer `zero` in it
void tail_lds(const std::vector<int64_t>& n, int lowest, int zero, int64_t (&size)[2]) {
    size[0] = size[1] = 0;
    for (int l = lowest; l < (int)n.size(); ++l) {
        int64_t& most = size[(l - zero) & 1];
        most = std::max(most, (n[(size_t)l] + klay::kColSlots + 3) / 4 * 4);
    }
}

// LDS bytes a workgroup of the persistent kernels may use: the largest of 160, 128 and 64 KB that the
// runtime accepts for all of them (gfx950 has 160 KB per compute unit), 0 if none.
size_t enable_tail_lds() {
    static_assert(kTailLdsMax == 160 * 1024, "the first size tried is the largest");
    for (int kb : {160, 128, 64}) {
        const int bytes = kb * 1024;
        hipError_t e = hipSuccess;
        for (const void* kernel : {reinterpret_cast<const void*>(&klay::col_fwd_kernel<1, false>), reinterpret_cast<const void*>(&klay::col_fwd_kernel<2, false>),
                                   reinterpret_cast<const void*>(&klay::col_fwd_kernel<4, false>), reinterpret_cast<const void*>(&klay::col_fwd_kernel<1, true>),
                                   reinterpret_cast<const void*>(&klay::col_fwd_kernel<2, true>), reinterpret_cast<const void*>(&klay::col_fwd_kernel<4, true>),
                                   reinterpret_cast<const void*>(&klay::col_bwd_kernel<1, false, false>),
                                   reinterpret_cast<const void*>(&klay::col_bwd_kernel<2, false, false>), reinterpret_cast<const void*>(&klay::col_bwd_kernel<4, false, false>),
                                   reinterpret_cast<const void*>(&klay::col_bwd_kernel<1, true, false>), reinterpret_cast<const void*>(&klay::col_bwd_kernel<2, true, false>),
                                   reinterpret_cast<const void*>(&klay::col_bwd_kernel<4, true, false>), reinterpret_cast<const void*>(&klay::col_bwd_kernel<1, false, true>),
                                   reinterpret_cast<const void*>(&klay::col_bwd_kernel<2, false, true>), reinterpret_cast<const void*>(&klay::col_bwd_kernel<4, false, true>),
                                   reinterpret_cast<const void*>(&klay::f64::col_fwd_kernel), reinterpret_cast<const void*>(&klay::f64::col_bwd_kernel<false>),
                                   reinterpret_cast<const void*>(&klay::f64::col_bwd_kernel<true>)})
            if (e == hipSuccess) e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e == hipSuccess) return (size_t)bytes;
        (void)hipGetLastError();
    }
    return 0;
}

// Columns per workgroup: two once there are more columns than compute units, four once there are more than twice as many, as
// far as they fit the LDS (a column of its own round would wait for the same dependent steps again; two cost little more
// than one: 30000 nodes in 24 layers, real semiring forward, B = 1024 70 us with two and 46 with four, 14000 nodes training
// B = 365 181 with one and 101 with two).
int tail_columns(int B, const int64_t (&size)[2], size_t lds_bytes, bool reverse) {
    // (the reverse kernel holds kColOwn<ct> times four values per thread of a layer)
    const int64_t widest = reverse ? std::max(size[0], size[1]) : 0;
    auto fits = [&](int ct, int own) { return widest <= 4 * own * klay::kColThreads && (size_t)(size[0] + size[1]) * ct * sizeof(float) <= lds_bytes; };
    if (B > 512 && fits(4, klay::kColOwn<4>)) return 4;
    return B > 256 && fits(2, klay::kColOwn<2>) ? 2 : 1;
}

// The column-major value buffer of a persistent forward launch: `T` floats a column.  `at`: entry of the layer below
// its first one, -1 if that layer has no place there.
struct TailBuffer {
    int64_t T = 0, at = -1;
};
TailBuffer tail_buffer(const klay_circuit* c, const TailChoice& t, int B) {
    TailBuffer b;
    b.T = c->tail_rows;
    const int64_t staged = tail_stage_rows(c, t);
    const bool after = t.first == c->plan.tail_first;           // its place is after the layers that take part
    if (staged > 0 && !(after && staged > tail_stage_rows(c, B))) {
        b.at = c->plan.col_off[(size_t)t.first - 1];
        if (after) b.T += staged;
    }
    return b;
}

// The forward kernel over the layers first .. L of `t`; start: see the kernel.
void launch_col_fwd(const klay_circuit* c, const ColTail& t, int first, const float* start, int start_T, const int32_t* start_map, float* tb, int T,
                    int B, int ld, int semiring, const klay::SlabLeaf& leaf, float* out, hipStream_t s) {
    int64_t size[2];
    tail_lds(t.n, first - 1, first - 1, size);
    const int ct = tail_columns(B, size, c->tail_lds_bytes, false);
    const int n_layers = c->plan.num_layers - first + 1, wide = std::min(n_layers, std::max(0, t.narrow[0] - first));
    auto* kernel = leaf.w && c->n_leaf_list ? (ct == 4 ? klay::col_fwd_kernel<4, true> : ct == 2 ? klay::col_fwd_kernel<2, true> : klay::col_fwd_kernel<1, true>)
                                            : (ct == 4 ? klay::col_fwd_kernel<4, false> : ct == 2 ? klay::col_fwd_kernel<2, false> : klay::col_fwd_kernel<1, false>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)((B + ct - 1) / ct)), dim3(klay::kColThreads),
                       (size_t)(size[0] + size[1]) * ct * sizeof(float), s, t.layers + (first - t.first), n_layers, first & 1, t.blocks[0], t.n_blocks[0], t.tables,
                       t.units[0], t.n_units[0], wide, (int)(wide < n_layers && c->plan.num_roots <= kRootsOneWave), start,
                       (int)t.n[(size_t)first - 1], start_T, start_map, B, ld, semiring, (int)size[0], tb, T, leaf, t.root_pos, c->plan.num_roots, out);
}

// tb: the column-major buffer; its last columns' room is followed by that of the layer below (workspace_layout), so
// T may count that layer.  keep: the values are kept there for a reverse sweep (otherwise only that layer goes there).
void launch_tail_fwd(const klay_circuit* c, const TailChoice& t, const float* act, float* tb, bool keep, int B, int ld,
                     int semiring, const klay::SlabLeaf& leaf, float* out, hipStream_t s) {
    const klay::CircuitPlan& p = c->plan;
    const TailBuffer buf = tail_buffer(c, t, B);
    const int nb = (int)p.layers[(size_t)t.first - 1].n;
    const float* start = act + (size_t)c->dl[(size_t)t.first - 1].row0 * ld;
    int start_T = 0;
    if (!leaf.w && buf.at >= 0) {
        dim3 tg((unsigned)((nb + 31) / 32), (unsigned)((B + 31) / 32));
        hipLaunchKernelGGL(klay::rows_to_cols_kernel<false>, tg, dim3(256), 0, s, start, nb, B, ld, tb + buf.at, (int)buf.T, (const int32_t*)nullptr);
        start = tb + buf.at;
        start_T = (int)buf.T;
    }
    launch_col_fwd(c, c->tail, t.first, start, start_T, nullptr, keep ? tb : nullptr, (int)buf.T, B, ld, semiring, leaf, out, s);
}

// The same over the TopPlan.  stage: room for the level below the first one, or null (the kernel reads its rows); tb: as above, or
// null (the values are not kept).
void launch_top_fwd(const klay_circuit* c, int first, const float* act, float* stage, float* tb, int B, int ld, int semiring, const klay::SlabLeaf& leaf,
                    float* out, hipStream_t s) {
    const int nb = (int)c->top.n[(size_t)first - 1];
    const int32_t* own = c->top.own + c->top.own_at[(size_t)first - 1];
    const int32_t* map = own;
    const float* start = act;
    int start_T = 0;
    if (stage) {
        dim3 tg((unsigned)((nb + 31) / 32), (unsigned)((B + 31) / 32));
        hipLaunchKernelGGL(klay::rows_to_cols_kernel<true>, tg, dim3(256), 0, s, act, nb, B, ld, stage, nb, own);
        start = stage;
        start_T = nb;
        map = nullptr;
    }
    launch_col_fwd(c, c->top, first, start, start_T, map, tb, (int)c->top.rows, B, ld, semiring, leaf, out, s);
}

// Reverse sweep of the layers L .. first into layer `last` (first, or the layer below it); last_at: its entry in a
// column of the value buffer (-1: layer 0, whose values the sweep does not need).
void launch_tail_bwd(const klay_circuit* c, const ColTail& tail, int last, int last_at, const float* tb, int T, const float* dout, const uint32_t* top_multi,
                     const klay::ColBwdOut& res, const klay::ColReal* real, int B, int ld, hipStream_t s) {
    const klay::CircuitPlan& p = c->plan;
    const int L = p.num_layers;
    int64_t size[2];
    tail_lds(tail.kept, last, L, size);
    const int ct = tail_columns(B, size, c->tail_lds_bytes, true);
    // The own values of the first steps are loaded at once: as many steps as fit behind the rows of one of the two arrays,
    // into LDS that only the wider layers further down need, or behind both arrays, up to all that a compute unit has (a
    // workgroup takes one anyway).
    const int64_t all = (int64_t)(c->tail_lds_bytes / sizeof(float)) / ct;
    int cached = 0, cache_at = 0;
    int64_t rows[2] = {0, 0}, sum = 0, words = size[0] + size[1];
    for (int l = L; l > last + 1; --l) {                  // step from layer l into layer l - 1
        for (int m : {l, l - 1}) rows[(L - m) & 1] = std::max(rows[(L - m) & 1], tail.kept[(size_t)m] + klay::kColSlots);
        sum += tail.kept[(size_t)l - 1];
        const int64_t at = (size[0] + rows[1] + 3) / 4 * 4;
        if (sum <= size[0] - (rows[0] + 3) / 4 * 4) {
            cache_at = (int)((rows[0] + 3) / 4 * 4);
            words = size[0] + size[1];
        } else if (sum <= all - at) {
            cache_at = (int)at;
            words = std::max(size[0] + size[1], at + sum);
        } else {
            break;
        }
        cached = L - l + 1;
    }
    const int narrow = std::max(0, std::min({L - tail.narrow[1] + 1, cached - 1, 64}));
    auto* kernel = real ? (ct == 4 ? klay::col_bwd_kernel<4, true, false> : ct == 2 ? klay::col_bwd_kernel<2, true, false> : klay::col_bwd_kernel<1, true, false>)
                   : res.keep ? (ct == 4 ? klay::col_bwd_kernel<4, false, true> : ct == 2 ? klay::col_bwd_kernel<2, false, true> : klay::col_bwd_kernel<1, false, true>)
                              : (ct == 4 ? klay::col_bwd_kernel<4, false, false> : ct == 2 ? klay::col_bwd_kernel<2, false, false> : klay::col_bwd_kernel<1, false, false>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)((B + ct - 1) / ct)), dim3(klay::kColThreads),
                       (size_t)words * ct * sizeof(float), s, tail.layers + (L - tail.first), L - last, last_at, L & 1, tail.blocks[1], tail.n_blocks[1], tail.tables, tail.units[1], narrow, dout, tail.top_ptr,
                       tail.top_root, p.num_roots, B, ld, (int)size[0], cached, cache_at, tb, T, top_multi, res, real ? *real : klay::ColReal{});
}

// Values of layers first .. last (all run by the persistent forward kernel) from the column-major
// buffer into their rows of the activation buffer, for the ordinary launches of a reverse sweep.
void launch_tb_to_rows(const klay_circuit* c, int first, int last, const float* tb, float* act, int B, int ld, hipStream_t s) {
    const klay::CircuitPlan& p = c->plan;
    int64_t tb_first = 0, n_rows = 0;
    for (int l = p.tail_first; l < first; ++l) tb_first += p.layers[(size_t)l].n;
    for (int l = first; l <= last; ++l) n_rows += p.layers[(size_t)l].n;
    if (n_rows <= 0) return;
    dim3 grid((unsigned)((n_rows + 31) / 32), (unsigned)((ld + 31) / 32));
    hipLaunchKernelGGL(klay::tb_to_rows_kernel<false>, grid, dim3(256), 0, s, tb, (int)c->last_tail_T, (int)tb_first, (int)n_rows, B,
                       ld, act + (size_t)c->dl[(size_t)first].row0 * ld, (const int32_t*)nullptr);
}

// Values or adjoints of the levels first .. last of the TopPlan (in a column-major buffer) into the activation or adjoint rows
// that they stand for.
void launch_top_to_rows(const klay_circuit* c, int first, int last, const float* cols, float* rows, int B, int ld, hipStream_t s) {
    const ColTail& t = c->top;
    const int64_t from = t.at[(size_t)first], n = t.at[(size_t)last] + t.kept[(size_t)last] - from;
    if (n <= 0) return;
    dim3 grid((unsigned)((n + 31) / 32), (unsigned)((ld + 31) / 32));
    hipLaunchKernelGGL(klay::tb_to_rows_kernel<true>, grid, dim3(256), 0, s, cols, (int)t.rows, (int)from, (int)n, B, ld, rows, t.act_row + from);
}

double tail_alg_bytes(const ColTail& t, int first, int B, bool backward) {
    double bytes = 0;
    for (int l = first; l < (int)t.n.size(); ++l) {
        const double n = (double)t.n[(size_t)l], e = (double)t.e[(size_t)l], below = (double)t.kept[(size_t)l - 1];
        if (!backward) bytes += 4.0 * B * (e + n) + 4.0 * (e + n);
        else if (l > first) {
            const bool is_and = (l & 1) != 0;
            bytes += 4.0 * B * ((is_and ? 1.0 : 2.0) * e + (is_and ? 1.0 : 2.0) * below) + 4.0 * (e + below);
        }
    }
    return bytes;
}

// what a persistent launch has to move through memory: the values it writes (forward) or reads (reverse)
// once, its index vectors, the rows it reads from or leaves in the activation buffer
double tail_min_bytes(const ColTail& t, int first, int B, bool backward) {
    double bytes = 0;
    for (int l = first; l < (int)t.n.size(); ++l) bytes += 4.0 * B * (double)t.kept[(size_t)l] + 4.0 * (double)t.words[backward][(size_t)l];
    bytes += 4.0 * B * (double)(backward ? t.kept[(size_t)first] : t.n[(size_t)first - 1]);
    return bytes;
}


// ---- real-semiring reverse sweep -----------------------------------------------------------------
klay_status ensure_real_bwd(klay_circuit* c) {
    const klay::CircuitPlan& p = c->plan;
    const int L = p.num_layers;
    if (!c->real_layers.empty()) return KLAY_OK;
    Packer pk;
    struct Off { size_t ptr = 0, child = 0; PassOffsets pass{}; klay::PassPlan plan; };
    std::vector<Off> offs((size_t)L + 1);
    klay::Options opt;
    for (int l = 1; l <= L; l += 2) {           // AND layers: plain index vectors by parent
        offs[(size_t)l].ptr = pk.add(p.layers[(size_t)l].row_ptr);
        offs[(size_t)l].child = pk.add(p.layers[(size_t)l].child);
    }
    const int B0 = p.alias_top;
    if (B0 > 0) {
        // Every row below layer B0 gathers from its parents in any higher layer up to B0.  An AND parent's
        // row holds P (see prod_parent_kernel); a sum node's row holds plain adjoints: those entries carry
        // the weighted bit, which OP_PROD_BWD reads as "add as it is".
        const int64_t NR = p.row0[(size_t)B0];
        std::vector<int32_t> gptr((size_t)NR + 1, 0);
        for (int l = 1; l <= B0; ++l)
            for (int32_t ch : p.layers[(size_t)l].child) ++gptr[(size_t)ch + 1];
        for (int64_t i = 0; i < NR; ++i) gptr[(size_t)i + 1] += gptr[(size_t)i];
        std::vector<int32_t> gsrc((size_t)gptr[(size_t)NR]);
        std::vector<uint32_t> gflag((size_t)gptr[(size_t)NR], 0u);
        {
            std::vector<int32_t> fill(gptr.begin(), gptr.end() - 1);
            for (int l = 1; l <= B0; ++l) {
                const klay::LayerPlan& lay = p.layers[(size_t)l];
                for (int64_t r = 0; r < lay.n; ++r)
                    for (int32_t j = lay.row_ptr[(size_t)r]; j < lay.row_ptr[(size_t)r + 1]; ++j) {
                        const int32_t slot = fill[(size_t)lay.child[(size_t)j]]++;
                        gsrc[(size_t)slot] = (int32_t)(p.row0[(size_t)l] + r);
                        if ((l & 1) == 0) gflag[(size_t)slot] = klay::kWeightedEdge;
                    }
            }
        }
        for (int l = 0; l < B0; ++l) {
            const klay::LayerPlan& lay = p.layers[(size_t)l];
            Off& o = offs[(size_t)l];
            const int64_t a = p.row0[(size_t)l];
            std::vector<int32_t> lptr((size_t)lay.n + 1);
            for (int64_t i = 0; i <= lay.n; ++i) lptr[(size_t)i] = gptr[(size_t)(a + i)] - gptr[(size_t)a];
            klay::make_pass_plan(lay.n, lptr.data(), gsrc.data() + gptr[(size_t)a], opt, o.plan, gflag.data() + gptr[(size_t)a]);
            if (o.plan.n_seg > p.max_bwd_seg)
                return fail(KLAY_EINVAL, "klay_backward: split plan of the real-semiring sweep exceeds the workspace");
            o.pass = pack_pass(pk, o.plan, c->small_batch_edges);
        }
    }
    size_t o_ptr = 0, o_child = 0;
    const bool offsets = pk.buf.size() < (size_t)INT32_MAX - 4096 - 4 * (size_t)L;
    if (offsets) {
        std::vector<int32_t> ptr_at((size_t)L + 1, 0), child_at((size_t)L + 1, 0);
        for (int l = L - ((L + 1) & 1); l >= 1; l -= 2) {
            ptr_at[(size_t)(L - l)] = (int32_t)offs[(size_t)l].ptr;
            child_at[(size_t)(L - l)] = (int32_t)offs[(size_t)l].child;
        }
        o_ptr = pk.add(ptr_at);
        o_child = pk.add(child_at);
    }
    const size_t bytes = pk.buf.size() * sizeof(int32_t);
    if (hipMalloc(reinterpret_cast<void**>(&c->d_real_index), bytes) != hipSuccess) {
        (void)hipGetLastError();
        return fail(KLAY_ENOMEM, "klay_backward: hipMalloc of the real-semiring index arrays failed");
    }
    if (hipError_t e = hipMemcpy(c->d_real_index, pk.buf.data(), bytes, hipMemcpyHostToDevice); e != hipSuccess) {
        (void)hipFree(c->d_real_index);
        c->d_real_index = nullptr;
        return fail(KLAY_EHIP, std::string("klay_backward: upload of the real-semiring index arrays: ") +
                                   hipGetErrorString(e));
    }
    if (offsets) {
        c->d_real_ptr = c->d_real_index + o_ptr;
        c->d_real_child = c->d_real_index + o_child;
    }
    c->real_layers.resize((size_t)L + 1);
    for (int l = 0; l <= L; ++l) {
        klay_circuit::RealLayer& r = c->real_layers[(size_t)l];
        if (l & 1) {
            r.ptr = c->d_real_index + offs[(size_t)l].ptr;
            r.child = c->d_real_index + offs[(size_t)l].child;
        }
        if (l < B0) bind_pass(r.by_child, offs[(size_t)l].plan, offs[(size_t)l].pass, c->d_real_index);
    }
    return KLAY_OK;
}

// adjoint rows of an AND layer -> P rows, in place (see prod_parent_kernel)
void launch_prod_parent(const klay_circuit::RealLayer& r, int n, const float* below, float* gl, const float* own,
                        const int* zero_flag, const Geometry& g, int B, hipStream_t s) {
    if (n <= 0) return;                               // a layer without chain nodes can be empty
    const int rpw = 64 / g.w;
    int64_t blocks = ((int64_t)n + 4 * rpw - 1) / (4 * rpw);
    // with the values of the nodes given the kernel mostly finds nothing to do: a small grid that strides
    if (own) blocks = std::min<int64_t>(blocks, std::max<int64_t>(256, 2048 / g.tiles));
    dim3 grid((unsigned)blocks, (unsigned)g.tiles);
#define KLAY_PP(VEC, W) \
    hipLaunchKernelGGL((klay::prod_parent_kernel<VEC, W>), grid, dim3(256), 0, s, r.ptr, r.child, below, gl, n, B, g.ld, own, zero_flag)
    if (g.w == 64) {
        if (g.vec == 4) KLAY_PP(4, 64);
        else if (g.vec == 2) KLAY_PP(2, 64);
        else KLAY_PP(1, 64);
    } else {
        switch (g.w) {
        case 32: KLAY_PP(1, 32); break;
        case 16: KLAY_PP(1, 16); break;
        case 8: KLAY_PP(1, 8); break;
        case 4: KLAY_PP(1, 4); break;
        case 2: KLAY_PP(1, 2); break;
        default: KLAY_PP(1, 1); break;
        }
    }
#undef KLAY_PP
}

// ---- double-precision evaluation ---------------------------------------------------------------
struct Workspace64 {
    size_t act = 0, wT = 0, seg_rows = 0, g0 = 0, g1 = 0, g2 = 0, tb = 0, gcols = 0, total = 0;   // offsets in doubles
};

// The layers that the double-precision persistent kernels take at a batch of B: from `first` on (0: none), an odd layer, so that
// the step below it is a plain sum that needs no values; the two directions take the same layers.  The choice that saves most by a rough
// account: a workgroup takes the time of the longest wave of each layer, 256 workgroups at a time, and moves the values; a launch takes
// its time and what it gathers and writes.  (us, fitted to 11 circuits of 16 to 60 layers taken from layer 1 on, B = 1 to 2000, within 6 and 11%.)
// In a training loop (`training`) both directions count.  The real semiring's sweep goes by launches, on rows that the values are
// put into first.  us, launches / layer 1 on / this rule: 21000 nodes in 44 layers, forward B = 1000 508 / 477 / 477, B = 2000 762 / 942 / 762, training
// B = 300 596 / 516 / 516, B = 513 698 / 826 / 698, real training B = 400 792 / 849 / 792.
// From a TopPlan in part only up to 256 columns (92000 nodes with power-law fan-ins, training step at B = 512 1667 us by launches,
// 1818 from layer 13 on).
int choose64(const klay_circuit* c, const ColTail& t, int B, bool real, bool training) {
    if (t.first <= 0 || c->tail_lds_bytes == 0) return 0;
    const int L = c->plan.num_layers, turns = (B + 255) / 256;
    const bool top = &t == &c->top;
    double inside[2] = {0, 0}, work[2] = {0, 0}, launches = 0, best = 0;       // [1]: reverse sweep
    int first = 0;
    int64_t fwd[2] = {0, 0}, bwd[2] = {0, 0};
    auto room = [](int64_t (&size)[2], int l, int64_t n) { size[l & 1] = std::max(size[l & 1], (n + klay::kColSlots + 3) / 4 * 4); };
    room(fwd, L, t.n[(size_t)L]);
    for (int l = L; l >= t.first; --l) {
        room(bwd, l, t.kept[(size_t)l]);
        room(fwd, l - 1, t.n[(size_t)l - 1]);
        if (t.kept[(size_t)l] > (int64_t)klay::f64::kColOwn * klay::kColThreads) break;
        const int64_t reverse = 2 * std::max(bwd[0], l == 1 ? (t.kept[0] + klay::kColSlots + 3) / 4 * 4 : 0) + bwd[1];
        if ((size_t)std::max(fwd[0] + fwd[1], reverse) * sizeof(double) > c->tail_lds_bytes) break;
        const klay::LayerPlan& lay = c->plan.layers[(size_t)l];
        const double share = (double)t.share[(size_t)l], e = (double)lay.e * B, n = (double)lay.n * B;
        inside[0] += (l & 1 ? 0.40e-3 : 1.60e-3) * share;
        inside[1] += (l & 1 ? 0.13e-3 : 2.38e-3) * share;
        work[0] += 0.86e-6 * e + 3.66e-6 * n;
        work[1] += 1.35e-6 * e + 4.29e-6 * n;
        launches += t.launches[(size_t)l];
        if ((l & 1) == 0 || l == L || (top && (l > c->plan.alias_top || (l > 1 && B > 256)))) continue;
        const double values = (double)(t.rows - t.at[(size_t)l]) * B;
        // what a reverse sweep puts into rows: values and adjoints of all of them, or the adjoints of the first
        const double transposed = l == 1 ? 0.0 : 4.0 + (top ? 2 * values : (double)t.kept[(size_t)l] * B) * 4e-6;
        const double leaves = l == 1 ? 60e-6 * c->plan.num_vars * B : 0.0;
        double outside = 4.1 * launches + work[0] + leaves, saved = outside - 3.0 - turns * inside[0] - 1.6e-6 * values;
        if (training && real) {
            saved -= 0.7 * launches + 4.2e-6 * values;
        } else if (training) {
            const double reverse_launches = (top ? 2.7 : 4.15) * launches + work[1];
            outside += reverse_launches;
            saved += reverse_launches - turns * inside[1] - 2.1e-6 * values - transposed;
        }
        if (saved > best && saved > 0.05 * outside) {          // (not on a few percent of a rough account)
            best = saved;
            first = l;
        }
    }
    return first;
}
const ColTail& tail64(const klay_circuit* c) { return c->top.first > 0 ? c->top : c->tail; }

// first: of the layers of tail64 that the persistent kernels take (0: none)
Workspace64 workspace_layout64(const klay_circuit* c, int B, int ld, int first) {
    const klay::CircuitPlan& p = c->plan;
    Workspace64 w;
    size_t off = 0;
    auto take = [&](size_t n) { const size_t o = off; off += (n + 31) / 32 * 32; return o; };
    w.act = take((size_t)p.num_nodes * ld);
    w.wT = take((size_t)std::max(1, p.num_vars) * ld);
    w.seg_rows = take((size_t)std::max<int64_t>(std::max(p.max_fwd_seg, p.max_bwd_seg), 1) * ld);
    // adjoints: one row per node of the layers 0 .. alias_top, two sets of rows for the layers above
    w.g0 = take((size_t)p.row0[(size_t)p.alias_top + 1] * ld);
    w.g1 = take((size_t)top_layer_rows(p) * ld);
    w.g2 = take((size_t)top_layer_rows(p) * ld);
    // the persistent kernels' values, and the adjoints they leave to the launches, column-major
    if (first > 0) {
        w.tb = take((size_t)tail64(c).rows * B);
        if (first > 1) w.gcols = take((size_t)tail64(c).rows * B);
    }
    w.total = off;
    return w;
}

// Two columns per lane (16-byte loads) where that leaves enough waves (as in the fp32 kernel); one where an entry takes an
// exponential and a wave has room for the row (up to 64 columns): those passes wait for arithmetic, and twice the waves
// hide it (85000 nodes at B = 33, per launch: logsumexp 8.0 us with two and 6.8 with one, plain sums 5.1 us with one and 4.4 with
// two).
// rows, entries: of the launch (segments are rows); short rows have a kernel of their own (see f64::pass_kernel).
constexpr int64_t kShortRows64 = 6;
template <int OP>
void launch_pass64(klay::f64::PassArgs a, int64_t rows, int64_t entries, hipStream_t s) {
    if (a.n_total <= 0) return;
    const bool arithmetic = OP == klay::OP_LSE || OP == klay::OP_SOFTMAX_BWD;
    const int vec = a.B == 1 || (arithmetic && a.B <= 64) || (int64_t)a.n_total * row_lanes(a.B, 2) < 64 * kFillWaves ? 1 : 2;
    a.lanes = row_lanes(a.B, vec);
    a.per_wave = 64 / a.lanes;
    a.inverse = row_inverse(a.lanes);
    const dim3 grid(row_blocks(a.n_total, a.lanes), (unsigned)((a.B + a.lanes * vec - 1) / (a.lanes * vec)));
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, a); };
    if (a.per_wave > 1) return vec == 2 ? launch(klay::f64::pass_kernel<OP, 2, false, false>) : launch(klay::f64::pass_kernel<OP, 1, false, false>);
    if constexpr (OP == klay::OP_LSE) {
        if (entries <= kShortRows64 * rows) return vec == 2 ? launch(klay::f64::pass_kernel<OP, 2, true, true>) : launch(klay::f64::pass_kernel<OP, 1, true, true>);
    }
    vec == 2 ? launch(klay::f64::pass_kernel<OP, 2, true, false>) : launch(klay::f64::pass_kernel<OP, 1, true, false>);
}

void launch_pass64(int op, const klay::f64::PassArgs& a, int64_t rows, int64_t entries, hipStream_t s) {
    switch (op) {
    case klay::OP_SUM: launch_pass64<klay::OP_SUM>(a, rows, entries, s); break;
    case klay::OP_PROD: launch_pass64<klay::OP_PROD>(a, rows, entries, s); break;
    case klay::OP_LSE: launch_pass64<klay::OP_LSE>(a, rows, entries, s); break;
    case klay::OP_MAX: launch_pass64<klay::OP_MAX>(a, rows, entries, s); break;
    case klay::OP_PROD_BWD: launch_pass64<klay::OP_PROD_BWD>(a, rows, entries, s); break;
    default: launch_pass64<klay::OP_SOFTMAX_BWD>(a, rows, entries, s); break;
    }
}

// main rows and segments in one launch, then the combine rows of split rows
void run_pass_set64(int op, int combine_op, const DevPass& dp, const double* src, const double* src2,
                    const double* own, double* dst, double* seg_rows, int B, int ld, hipStream_t s) {
    klay::f64::PassArgs a{};
    a.ptr = dp.ptr;
    a.idx = dp.idx;
    a.src = src;
    a.src2 = src2;
    a.own = own;
    a.seg_owner = dp.seg_owner;
    a.out_row = nullptr;
    a.dst = dst;
    a.dst_seg = seg_rows;
    a.n_main = dp.n_main;
    a.n_total = dp.n_main + dp.n_seg;
    a.B = B;
    a.ld = ld;
    launch_pass64(op, a, (int64_t)dp.n_light + dp.n_seg, dp.main_entries + dp.seg_entries, s);
    if (dp.n_heavy > 0) {
        klay::f64::PassArgs cmb{};
        cmb.ptr = dp.comb_ptr;
        cmb.idx = dp.comb_idx;
        cmb.src = seg_rows;
        cmb.out_row = dp.comb_row;
        cmb.dst = dst;
        cmb.n_main = dp.n_heavy;
        cmb.n_total = dp.n_heavy;
        cmb.B = B;
        cmb.ld = ld;
        launch_pass64(combine_op, cmb, dp.n_heavy, dp.n_seg, s);
    }
}

klay_status forward64_impl(klay_circuit* c, const double* w, const double* wneg, int32_t B, double* out,
                           klay_semiring semiring, void* stream) {
    if (!c || !w || !out) return fail(KLAY_EINVAL, "klay_forward_f64: null argument");
    if (c->device < 0) return fail(KLAY_ESTATE, "klay_forward_f64: host-only handle (built with device = -1)");
    if (B < 1) return fail(KLAY_EINVAL, "klay_forward_f64: B must be >= 1");
    if (semiring != KLAY_REAL && semiring != KLAY_LOG && semiring != KLAY_MAXLOG)
        return fail(KLAY_EINVAL, "klay_forward_f64: unknown semiring");
    KLAY_HIP(hipSetDevice(c->device));
    hipStream_t s = static_cast<hipStream_t>(stream);
    const klay::CircuitPlan& p = c->plan;
    const int ld = B > 64 ? (B + 1) / 2 * 2 : B;       // even rows for two columns per lane
    c->have_fwd64 = false;
    const ColTail& tail = tail64(c);
    int first = choose64(c, tail, B, semiring == KLAY_REAL, c->bwd64_followed && semiring != KLAY_MAXLOG);
    Workspace64 lay = workspace_layout64(c, B, ld, first);
    // room for the choices of all passes over this batch at once: a later one, which may be captured, allocates nothing
    size_t room = lay.total;
    if (tail.first > 0)
        for (const auto& [real, training] : {std::pair(false, false), std::pair(false, true), std::pair(true, true)})
            room = std::max(room, workspace_layout64(c, B, ld, choose64(c, tail, B, real, training)).total);
    if (room * sizeof(double) > c->ws64_bytes) {
        if (c->ws64) { KLAY_HIP(hipFree(c->ws64)); c->ws64 = nullptr; c->ws64_bytes = 0; }
        hipError_t e = hipMalloc(&c->ws64, room * sizeof(double));
        if (e != hipSuccess && tail.first > 0) {     // the launches need less
            (void)hipGetLastError();
            first = 0;
            lay = workspace_layout64(c, B, ld, first);
            room = lay.total;
            e = hipMalloc(&c->ws64, room * sizeof(double));
        }
        if (e != hipSuccess) {
            (void)hipGetLastError();
            c->ws64 = nullptr;
            return fail(KLAY_ENOMEM, "hipMalloc of " + std::to_string(room * sizeof(double)) + " workspace bytes failed");
        }
        c->ws64_bytes = room * sizeof(double);
    }
    double* ws = static_cast<double*>(c->ws64);
    double* act = ws + lay.act;
    double* wT = ws + lay.wT;
    double* seg_rows = ws + lay.seg_rows;
    const int L = p.num_layers, V = p.num_vars;
    const bool log_domain = semiring != KLAY_REAL;
    const dim3 row_grid((unsigned)((ld + 255) / 256));
    if (V > 0)
        hipLaunchKernelGGL(klay::f64::leaf_fwd_kernel, dim3((unsigned)V, (unsigned)((ld + 255) / 256)), dim3(256), 0, s, w,
                           wneg, (int)B, V, ld, c->d_pos_row, c->d_neg_row, wT, act, log_domain ? 1 : 0);
    if (c->true_row >= 0)
        hipLaunchKernelGGL(klay::f64::fill_row_kernel, row_grid, dim3(256), 0, s, act + (size_t)c->true_row * ld, ld,
                           log_domain ? 0.0 : 1.0);
    if (c->false_row >= 0)
        hipLaunchKernelGGL(klay::f64::fill_row_kernel, row_grid, dim3(256), 0, s, act + (size_t)c->false_row * ld, ld,
                           log_domain ? (double)-INFINITY : 0.0);
    for (int l = 1; l <= (first > 0 ? first - 1 : L); ++l) {
        const DevLayer& d = c->dl[(size_t)l];
        const bool is_and = (l & 1) != 0;
        const int or_op = semiring == KLAY_MAXLOG ? klay::OP_MAX : klay::OP_LSE;
        const int op = log_domain ? (is_and ? klay::OP_SUM : or_op) : (is_and ? klay::OP_PROD : klay::OP_SUM);
        // up to alias_top child entries are rows of the whole buffer, above it of the layer below
        const double* below = l <= p.alias_top ? act : act + (size_t)c->dl[(size_t)l - 1].row0 * ld;
        run_pass_set64(op, op, d.fwd, below, nullptr, nullptr, act + (size_t)d.row0 * ld, seg_rows, B, ld, s);
    }
    if (first > 0) {
        const bool top = &tail == &c->top;
        int64_t size[2];
        tail_lds(tail.n, first - 1, first - 1, size);
        hipLaunchKernelGGL(klay::f64::col_fwd_kernel, dim3((unsigned)B), dim3(klay::kColThreads), (size_t)(size[0] + size[1]) * sizeof(double), s,
                           tail.layers + (first - tail.first), L - first + 1, first & 1, tail.blocks[0], tail.n_blocks[0], tail.tables,
                           top ? act : act + (size_t)c->dl[(size_t)first - 1].row0 * ld, (int)tail.n[(size_t)first - 1],
                           top ? tail.own + tail.own_at[(size_t)first - 1] : nullptr, ld, (int)semiring, (int)size[0], ws + lay.tb, (int)tail.rows,
                           tail.root_pos, p.num_roots, out);
    } else {
        hipLaunchKernelGGL(klay::f64::root_out_kernel, dim3((unsigned)p.num_roots), dim3(256), 0, s,
                           act + (size_t)c->dl[(size_t)L].row0 * ld, c->d_root_pos, (int)B, p.num_roots, ld, out);
    }
    KLAY_HIP(hipGetLastError());
    c->have_fwd64 = true;
    c->bwd64_followed = false;
    c->last64_B = B;
    c->last64_semiring = semiring;
    c->last64_neg_explicit = wneg != nullptr;
    c->last64_tail = first > 0 ? &tail : nullptr;
    c->last64_first = first;
    return KLAY_OK;
}

klay_status backward64_impl(klay_circuit* c, const double* dout, double* dleaf, double* dneg, void* stream) {
    if (!c || !dout || !dleaf) return fail(KLAY_EINVAL, "klay_backward_f64: null argument");
    if (c->device < 0) return fail(KLAY_ESTATE, "klay_backward_f64: host-only handle");
    if (!c->have_fwd64) return fail(KLAY_ESTATE, "klay_backward_f64: no double-precision forward pass to differentiate");
    if (c->last64_semiring == KLAY_MAXLOG)
        return fail(KLAY_EINVAL, "klay_backward_f64: the (max, +) semiring is not differentiated");
    const bool real = c->last64_semiring == KLAY_REAL;
    if (dneg && !c->last64_neg_explicit)
        return fail(KLAY_ESTATE, "klay_backward_f64: dneg given, but the forward pass had no weights for the negated literals");
    KLAY_HIP(hipSetDevice(c->device));
    c->bwd64_followed = true;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const klay::CircuitPlan& p = c->plan;
    const int B = c->last64_B, ld = B > 64 ? (B + 1) / 2 * 2 : B;
    const Workspace64 lay = workspace_layout64(c, B, ld, c->last64_tail ? c->last64_first : 0);
    double* ws = static_cast<double*>(c->ws64);
    double* act = ws + lay.act;
    double* wT = ws + lay.wT;
    double* seg_rows = ws + lay.seg_rows;
    double* G = ws + lay.g0;
    double* gcur = ws + lay.g1;
    double* gnext = ws + lay.g2;
    const int L = p.num_layers, V = p.num_vars, R = p.num_roots, B0 = p.alias_top;
    const int leaf_mode = c->last64_neg_explicit ? 2 : (real ? 0 : 1);
    const dim3 leaf_grid((unsigned)std::max(V, 1), (unsigned)((B + 255) / 256));
    auto grow = [&](int l) { return G + (size_t)c->dl[(size_t)l].row0 * ld; };   // adjoint rows of a layer <= B0
    // what the persistent kernel kept or left column-major, layers first .. last, into rows
    auto to_rows = [&](const double* cols, int first, int last, double* rows) {
        const ColTail& t = *c->last64_tail;
        const int64_t from = t.at[(size_t)first], n = t.at[(size_t)last] + t.kept[(size_t)last] - from;
        hipLaunchKernelGGL(klay::f64::cols_to_rows_kernel, dim3((unsigned)((n + 31) / 32), (unsigned)((ld + 31) / 32)), dim3(256), 0, s, cols, (int)t.rows,
                           (int)from, (int)n, B, ld, rows, &t == &c->top ? t.act_row + from : nullptr);
    };
    const int tail_first = c->last64_tail ? c->last64_first : 0;
    const bool top_plan = c->last64_tail == &c->top;
    if (tail_first > 0 && real) to_rows(ws + lay.tb, tail_first, L, top_plan ? act : act + (size_t)c->dl[(size_t)tail_first].row0 * ld);
    // Same course as the fp32 sweep (see klay_backward's implementation): the layers above B0 one by one,
    // alternating between two buffers, the last of these steps writing the rows of layer B0 into G; then
    // the rows of the layers below B0, each gathering from its parents anywhere in G.
    if (real) {
        klay_status rs = ensure_real_bwd(c);
        if (rs != KLAY_OK) return rs;
        const dim3 pp_block(256);
        auto prod_parent = [&](int l, const double* below, double* gl) {
            const DevLayer& d = c->dl[(size_t)l];
            if (d.n <= 0) return;
            const klay_circuit::RealLayer& r = c->real_layers[(size_t)l];
            hipLaunchKernelGGL(klay::f64::prod_parent_kernel, dim3((unsigned)((d.n + 3) / 4), (unsigned)((B + 63) / 64)),
                               pp_block, 0, s, r.ptr, r.child, below, gl, (int)d.n, B, ld);
        };
        hipLaunchKernelGGL(klay::f64::seed_kernel, dim3((unsigned)c->dl[(size_t)L].n), dim3(256), 0, s, dout, c->d_top_ptr,
                           c->d_top_root, B, R, ld, L == B0 ? grow(L) : gcur);
        for (int l = L; l > B0; --l) {
            const DevLayer& d = c->dl[(size_t)l];
            const DevLayer& below = c->dl[(size_t)l - 1];
            double* dst = l - 1 == B0 ? grow(B0) : gnext;
            if ((l & 1) == 0) {
                run_pass_set64(klay::OP_SUM, klay::OP_SUM, d.bwd, gcur, nullptr, nullptr, dst, seg_rows, B, ld, s);
            } else {
                prod_parent(l, act + (size_t)below.row0 * ld, gcur);
                run_pass_set64(klay::OP_PROD_BWD, klay::OP_SUM, d.bwd, gcur, nullptr, act + (size_t)below.row0 * ld, dst,
                               seg_rows, B, ld, s);
            }
            std::swap(gcur, gnext);
        }
        if (B0 > 0 && (B0 & 1)) prod_parent(B0, act, grow(B0));
        for (int l = B0 - 1; l >= 0; --l) {
            run_pass_set64(klay::OP_PROD_BWD, klay::OP_SUM, c->real_layers[(size_t)l].by_child, G, nullptr,
                           act + (size_t)c->dl[(size_t)l].row0 * ld, grow(l), seg_rows, B, ld, s);
            if (l & 1) prod_parent(l, act, grow(l));
        }
    } else {
        int from = L, low = B0 - 1;                  // the layers from .. B0 + 1 one by one, then the rows of the layers low .. 0
        if (tail_first > 0) {
            const ColTail& t = *c->last64_tail;
            const int last = tail_first == 1 ? 0 : tail_first;
            klay::f64::ColBwdOut res{};
            res.n_last = (int32_t)t.kept[(size_t)last];
            res.keep_from = L - B0;
            if (last == 0) {
                res.wT = wT;
                res.pos_row = c->d_pos_row;
                res.neg_row = c->d_neg_row;
                res.dleaf = dleaf;
                res.dneg = dneg;
                res.V = V;
                res.mode = leaf_mode;
                res.ld = ld;
            } else {
                res.g_cols = ws + lay.gcols;
            }
            int64_t size[2] = {0, 0};
            for (int l = last; l <= L; ++l) size[l & 1] = std::max(size[l & 1], (t.kept[(size_t)l] + klay::kColSlots + 3) / 4 * 4);
            hipLaunchKernelGGL((last > 0 && top_plan ? klay::f64::col_bwd_kernel<true> : klay::f64::col_bwd_kernel<false>), dim3((unsigned)B),
                               dim3(klay::kColThreads), (size_t)(2 * size[0] + size[1]) * sizeof(double), s, t.layers + (L - t.first), L - last,
                               last > 0 ? (int)t.at[(size_t)last] : -1, L & 1, t.blocks[1], t.n_blocks[1], t.tables, dout, t.top_ptr, t.top_root, R,
                               (int)(2 * size[0]), ws + lay.tb, (int)t.rows, res);
            if (last == 0) {
                KLAY_HIP(hipGetLastError());
                return KLAY_OK;
            }
            if (top_plan) {
                // the rows below gather from the adjoints and the values of their parents
                to_rows(ws + lay.tb, last, B0, act);
                to_rows(ws + lay.gcols, last, B0, G);
                from = B0;
                low = last - 1;
            } else {
                to_rows(ws + lay.gcols, last, last, gcur);
                from = last;
            }
        } else {
            hipLaunchKernelGGL(klay::f64::seed_kernel, dim3((unsigned)c->dl[(size_t)L].n), dim3(256), 0, s, dout, c->d_top_ptr,
                               c->d_top_root, B, R, ld, L == B0 ? grow(L) : gcur);
        }
        for (int l = from; l > B0; --l) {
            const DevLayer& d = c->dl[(size_t)l];
            const DevLayer& below = c->dl[(size_t)l - 1];
            double* dst = l - 1 == B0 ? grow(B0) : gnext;
            if ((l & 1) != 0 || !d.bwd.has_weighted)
                run_pass_set64(klay::OP_SUM, klay::OP_SUM, d.bwd, gcur, nullptr, nullptr, dst, seg_rows, B, ld, s);
            else
                run_pass_set64(klay::OP_SOFTMAX_BWD, klay::OP_SUM, d.bwd, gcur, act + (size_t)d.row0 * ld,
                               act + (size_t)below.row0 * ld, dst, seg_rows, B, ld, s);
            std::swap(gcur, gnext);
        }
        for (int l = low; l >= 0; --l) {
            const DevPass& dp = c->dl[(size_t)l + 1].bwd;
            run_pass_set64(dp.has_weighted ? klay::OP_SOFTMAX_BWD : klay::OP_SUM, klay::OP_SUM, dp, G, act,
                           act + (size_t)c->dl[(size_t)l].row0 * ld, grow(l), seg_rows, B, ld, s);
        }
    }
    if (V > 0)
        hipLaunchKernelGGL(klay::f64::leaf_bwd_kernel, leaf_grid, dim3(256), 0, s, G, wT, c->d_pos_row, c->d_neg_row, B, V,
                           ld, leaf_mode, dleaf, dneg);
    KLAY_HIP(hipGetLastError());
    return KLAY_OK;
}

}  // namespace

// Circuits collected for a joint layerization: node arrays concatenated, ids shifted.
struct klay_builder {
    int32_t num_vars = 0;
    std::vector<uint8_t> type;
    std::vector<int32_t> lit;
    std::vector<int64_t> ptr{0};
    std::vector<int32_t> idx;
    std::vector<int32_t> roots;
};

extern "C" {

const char* klay_last_error(void) { return g_err.c_str(); }

klay_status klay_build_ex(int32_t num_vars, int64_t num_nodes, const uint8_t* node_type,
                          const int32_t* node_lit, const int64_t* child_ptr, const int32_t* child_idx,
                          int32_t num_roots, const int32_t* roots, int32_t device,
                          const klay_options* opts, klay_circuit** out) {
    if (!out) return fail(KLAY_EINVAL, "klay_build: out is null");
    *out = nullptr;
    klay::Options o;
    o.alias_chains = true;                    // the default: padding-free below the narrow top
    if (opts) {
        o.no_reorder = opts->no_reorder != 0;
        if (opts->heavy_fan > 0) o.heavy_fan = opts->heavy_fan;
        if (opts->min_segment > 0) o.min_segment = opts->min_segment;
        o.no_tail = opts->no_tail != 0;
        o.alias_chains = opts->unary_chains == 0;
        if (opts->tail_rows_cap > 0) o.tail_rows_cap = opts->tail_rows_cap;
        o.no_merge = opts->no_merge != 0;
        o.small_batch_edges = opts->small_batch_edges != 0;
        o.no_fusion = opts->no_fusion != 0;
    }
    std::unique_ptr<klay_circuit> c;
    try {
        c.reset(new klay_circuit());
        std::string err;
        int st = klay::layerize(num_vars, num_nodes, node_type, node_lit, child_ptr, child_idx, num_roots,
                                roots, o, c->plan, err);
        if (st != 0) return fail(static_cast<klay_status>(st), err);
    } catch (const std::bad_alloc&) {
        return fail(KLAY_ENOMEM, "klay_build: out of host memory");
    }
    for (int64_t i = 0; i < c->plan.layers[0].n; ++i) {
        if (c->plan.leaf_code[(size_t)i] == INT32_MAX) c->true_row = (int32_t)i;
        if (c->plan.leaf_code[(size_t)i] == INT32_MIN) c->false_row = (int32_t)i;
    }
    c->device = device;
    c->small_batch_edges = o.small_batch_edges;
    c->no_fusion = o.no_fusion;
    if (c->plan.tail_first > 0) {
        // sizes of the persistent kernels' buffers (part of the workspace, so host-only handles know them too)
        const klay::CircuitPlan& p = c->plan;
        c->tail_rows = p.col_rows;
    }
    try {
        describe_tails(c.get());
    } catch (const std::bad_alloc&) {
        return fail(KLAY_ENOMEM, "klay_build: out of host memory");
    }
    const bool persistent = c->tail.first > 0 || c->top.first > 0;
    if (device >= 0) {
        int ndev = 0;
        if (hipGetDeviceCount(&ndev) != hipSuccess || device >= ndev) {
            (void)hipGetLastError();
            return fail(KLAY_EHIP, "klay_build: HIP device " + std::to_string(device) + " not available");
        }
        klay_status st;
        try {
            st = upload(c.get());
        } catch (const std::bad_alloc&) {
            st = fail(KLAY_ENOMEM, "klay_build: out of host memory");
        }
        if (st != KLAY_OK) {
            if (c->d_index) (void)hipFree(c->d_index);
            return st;
        }
        c->tail_lds_bytes = persistent ? enable_tail_lds() : 0;
    } else {
        // a host-only handle sizes workspaces for a device that grants the whole LDS of a compute unit
        c->tail_lds_bytes = persistent ? kTailLdsMax : 0;
    }
    *out = c.release();
    return KLAY_OK;
}

klay_status klay_build(int32_t num_vars, int64_t num_nodes, const uint8_t* node_type,
                       const int32_t* node_lit, const int64_t* child_ptr, const int32_t* child_idx,
                       int32_t num_roots, const int32_t* roots, int32_t device, klay_circuit** out) {
    return klay_build_ex(num_vars, num_nodes, node_type, node_lit, child_ptr, child_idx, num_roots, roots,
                         device, nullptr, out);
}

klay_status klay_builder_create(int32_t num_vars, klay_builder** out) {
    if (!out) return fail(KLAY_EINVAL, "klay_builder_create: out is null");
    *out = nullptr;
    if (num_vars < 0) return fail(KLAY_EINVAL, "klay_builder_create: negative num_vars");
    try {
        *out = new klay_builder();
    } catch (const std::bad_alloc&) {
        return fail(KLAY_ENOMEM, "klay_builder_create: out of host memory");
    }
    (*out)->num_vars = num_vars;
    return KLAY_OK;
}

klay_status klay_builder_add(klay_builder* b, int64_t num_nodes, const uint8_t* node_type,
                             const int32_t* node_lit, const int64_t* child_ptr, const int32_t* child_idx,
                             int32_t num_roots, const int32_t* roots, int32_t* first_root) {
    if (!b) return fail(KLAY_EINVAL, "klay_builder_add: null builder");
    if (num_nodes <= 0 || num_roots <= 0 || !node_type || !node_lit || !child_ptr || !roots)
        return fail(KLAY_EINVAL, "klay_builder_add: empty circuit or null array");
    const int64_t base = (int64_t)b->type.size();
    if (base + num_nodes > (int64_t)INT32_MAX || (int64_t)b->roots.size() + num_roots > (int64_t)INT32_MAX)
        return fail(KLAY_EINVAL, "klay_builder_add: more than 2^31-1 nodes or roots in total");
    if (child_ptr[0] != 0) return fail(KLAY_EINVAL, "klay_builder_add: child_ptr[0] must be 0");
    for (int64_t i = 0; i < num_nodes; ++i)
        if (child_ptr[i + 1] < child_ptr[i]) return fail(KLAY_EINVAL, "klay_builder_add: child_ptr not monotone");
    const int64_t ne = child_ptr[num_nodes];
    if (ne > 0 && !child_idx) return fail(KLAY_EINVAL, "klay_builder_add: child_idx is null");
    for (int64_t j = 0; j < ne; ++j)
        if (child_idx[j] < 0 || child_idx[j] >= num_nodes)
            return fail(KLAY_EINVAL, "klay_builder_add: child index out of range");
    for (int32_t r = 0; r < num_roots; ++r)
        if (roots[r] < 0 || roots[r] >= num_nodes) return fail(KLAY_EINVAL, "klay_builder_add: root out of range");
    try {
        const size_t e0 = b->idx.size();
        b->type.reserve(b->type.size() + (size_t)num_nodes);
        b->lit.reserve(b->lit.size() + (size_t)num_nodes);
        b->ptr.reserve(b->ptr.size() + (size_t)num_nodes);
        b->idx.reserve(e0 + (size_t)ne);
        b->roots.reserve(b->roots.size() + (size_t)num_roots);
        // nothing below can throw: capacity is reserved
        b->type.insert(b->type.end(), node_type, node_type + num_nodes);
        b->lit.insert(b->lit.end(), node_lit, node_lit + num_nodes);
        for (int64_t i = 0; i < num_nodes; ++i) b->ptr.push_back((int64_t)e0 + child_ptr[i + 1]);
        for (int64_t j = 0; j < ne; ++j) b->idx.push_back((int32_t)(base + child_idx[j]));
        if (first_root) *first_root = (int32_t)b->roots.size();
        for (int32_t r = 0; r < num_roots; ++r) b->roots.push_back((int32_t)(base + roots[r]));
    } catch (const std::bad_alloc&) {
        return fail(KLAY_ENOMEM, "klay_builder_add: out of host memory");
    }
    return KLAY_OK;
}

klay_status klay_builder_finish(const klay_builder* b, int32_t device, const klay_options* opts,
                                klay_circuit** out) {
    if (!b) return fail(KLAY_EINVAL, "klay_builder_finish: null builder");
    if (b->type.empty()) return fail(KLAY_ESTATE, "klay_builder_finish: no circuit was added");
    return klay_build_ex(b->num_vars, (int64_t)b->type.size(), b->type.data(), b->lit.data(), b->ptr.data(),
                         b->idx.data(), (int32_t)b->roots.size(), b->roots.data(), device, opts, out);
}

void klay_builder_destroy(klay_builder* b) { delete b; }

void klay_destroy(klay_circuit* c) {
    if (!c) return;
    if (c->device >= 0) {
        (void)hipSetDevice(c->device);
        release_events(c);
        if (c->d_index) (void)hipFree(c->d_index);
        if (c->ws_own) (void)hipFree(c->ws_own);
        if (c->d_real_index) (void)hipFree(c->d_real_index);
        if (c->ws64) (void)hipFree(c->ws64);
    }
    delete c;
}

klay_status klay_info(const klay_circuit* c, klay_info_t* info) {
    if (!c || !info) return fail(KLAY_EINVAL, "klay_info: null argument");
    const klay::CircuitPlan& p = c->plan;
    std::memset(info, 0, sizeof(*info));
    info->num_vars = p.num_vars;
    info->num_roots = p.num_roots;
    info->num_layers = p.num_layers;
    info->device = c->device;
    info->num_nodes = p.num_nodes;
    info->num_edges = p.num_edges;
    info->dag_nodes = p.dag_nodes;
    info->dag_edges = p.dag_edges;
    info->num_pad_nodes = p.num_pad_nodes;
    info->max_layer_nodes = p.max_layer_nodes;
    info->max_fan_in = p.max_fan_in;
    info->max_fan_out = p.max_fan_out;
    info->num_split_rows = p.num_split_rows;
    info->index_bytes = (int64_t)c->index_bytes;
    info->tail_first_layer = p.tail_first;
    info->num_merged_nodes = p.num_merged;
    info->alias_top_layer = p.alias_top;
    info->num_fused_rows = p.num_fused;
    return KLAY_OK;
}

klay_status klay_layer_sizes(const klay_circuit* c, int64_t* nodes, int64_t* edges) {
    if (!c || !nodes || !edges) return fail(KLAY_EINVAL, "klay_layer_sizes: null argument");
    for (int l = 0; l <= c->plan.num_layers; ++l) {
        nodes[l] = c->plan.layers[(size_t)l].n;
        edges[l] = c->plan.layers[(size_t)l].e;
    }
    return KLAY_OK;
}

klay_status klay_layer_csr(const klay_circuit* c, int32_t layer, int64_t* row_ptr, int32_t* child) {
    if (!c || !row_ptr || !child) return fail(KLAY_EINVAL, "klay_layer_csr: null argument");
    if (layer < 1 || layer > c->plan.num_layers) return fail(KLAY_EINVAL, "klay_layer_csr: layer out of range");
    const klay::LayerPlan& l = c->plan.layers[(size_t)layer];
    for (int64_t i = 0; i <= l.n; ++i) row_ptr[i] = l.row_ptr[(size_t)i];
    std::copy(l.child.begin(), l.child.end(), child);
    return KLAY_OK;
}

klay_status klay_layer_nodes(const klay_circuit* c, int32_t layer, int32_t* origin, uint8_t* is_pad) {
    if (!c || !origin || !is_pad) return fail(KLAY_EINVAL, "klay_layer_nodes: null argument");
    if (layer < 0 || layer > c->plan.num_layers) return fail(KLAY_EINVAL, "klay_layer_nodes: layer out of range");
    const klay::LayerPlan& l = c->plan.layers[(size_t)layer];
    std::copy(l.origin.begin(), l.origin.end(), origin);
    std::copy(l.is_pad.begin(), l.is_pad.end(), is_pad);
    return KLAY_OK;
}

klay_status klay_root_positions(const klay_circuit* c, int32_t* position) {
    if (!c || !position) return fail(KLAY_EINVAL, "klay_root_positions: null argument");
    std::copy(c->plan.root_pos.begin(), c->plan.root_pos.end(), position);
    return KLAY_OK;
}

size_t klay_workspace_bytes(const klay_circuit* c, int32_t B, int need_backward) {
    if (!c || B < 1) return 0;
    if (!need_backward) return workspace_layout(c, B, false, 0).total * sizeof(float);
    return std::max(workspace_layout(c, B, true, 0).total, workspace_layout(c, B, true, choose_top(c, B)).total) * sizeof(float);
}

klay_status klay_persistent_layers(const klay_circuit* c, int32_t B, klay_semiring semiring, int32_t double_precision, int32_t training,
                                   int32_t* first_layer, int32_t* plan) {
    if (!c || !first_layer || !plan) return fail(KLAY_EINVAL, "klay_persistent_layers: null argument");
    if (B < 1) return fail(KLAY_EINVAL, "klay_persistent_layers: B must be >= 1");
    if (semiring != KLAY_REAL && semiring != KLAY_LOG && semiring != KLAY_MAXLOG)
        return fail(KLAY_EINVAL, "klay_persistent_layers: unknown semiring");
    if (double_precision) {
        *first_layer = choose64(c, tail64(c), B, semiring == KLAY_REAL, training != 0 && semiring != KLAY_MAXLOG);
        *plan = *first_layer == 0 ? 0 : &tail64(c) == &c->top ? 2 : 1;
    } else if ((*first_layer = choose_top(c, B, semiring == KLAY_REAL && training != 0)) > 0) {
        *plan = 2;
    } else {
        *first_layer = choose_tail_fwd(c, B).first;
        *plan = *first_layer > 0 ? 1 : 0;
    }
    return KLAY_OK;
}

klay_status klay_set_workspace(klay_circuit* c, void* dev_ptr, size_t bytes) {
    if (!c) return fail(KLAY_EINVAL, "klay_set_workspace: null handle");
    if (dev_ptr && (reinterpret_cast<uintptr_t>(dev_ptr) & 255u))
        return fail(KLAY_EINVAL, "klay_set_workspace: pointer must be 256-byte aligned");
    c->ws_user = dev_ptr;
    c->ws_user_bytes = dev_ptr ? bytes : 0;
    c->have_fwd = false;
    return KLAY_OK;
}

klay_status klay_set_profiling(klay_circuit* c, int32_t enable) {
    if (!c) return fail(KLAY_EINVAL, "klay_set_profiling: null handle");
    if (c->device < 0) return fail(KLAY_ESTATE, "klay_set_profiling: host-only handle");
    KLAY_HIP(hipSetDevice(c->device));
    c->profiling = enable != 0;
    if (!c->profiling) release_events(c);
    return KLAY_OK;
}

klay_status klay_get_profile(klay_circuit* c, klay_profile_t* prof) {
    if (!c || !prof) return fail(KLAY_EINVAL, "klay_get_profile: null argument");
    std::memset(prof, 0, sizeof(*prof));
    for (const std::vector<EventRec>* recs : {&c->ev_fwd, &c->ev_bwd})
        for (const EventRec& r : *recs) {
            if (!r.start || !r.stop) continue;
            KLAY_HIP(hipEventSynchronize(r.stop));
            float ms = 0.f;
            KLAY_HIP(hipEventElapsedTime(&ms, r.start, r.stop));
            prof->ms[r.cls] += ms;
            prof->launches[r.cls] += 1;
            prof->alg_bytes[r.cls] += r.bytes;
            prof->min_bytes[r.cls] += r.min_bytes;
        }
    return KLAY_OK;
}

// static_ws: run in the fixed device array instead of the handle's workspace (klay_forward_static):
// no allocation, no event, nothing kept for a backward pass.
static klay_status forward_impl(klay_circuit* c, const float* leaf_weights, const float* neg_weights, int32_t B,
                                float* out, klay_semiring semiring, void* stream, bool static_ws = false) {
    if (!c || !leaf_weights || !out) return fail(KLAY_EINVAL, "klay_forward: null argument");
    if (c->device < 0) return fail(KLAY_ESTATE, "klay_forward: host-only handle (built with device = -1)");
    if (B < 1) return fail(KLAY_EINVAL, "klay_forward: B must be >= 1");
    if (semiring != KLAY_REAL && semiring != KLAY_LOG && semiring != KLAY_MAXLOG)
        return fail(KLAY_EINVAL, "klay_forward: unknown semiring");
    KLAY_HIP(hipSetDevice(c->device));
    hipStream_t s = static_cast<hipStream_t>(stream);
    const klay::CircuitPlan& p = c->plan;
    const Geometry g = geometry(B);
    const bool log_domain = semiring != KLAY_REAL;      // leaf weights are log p in both log-domain semirings
    if (!static_ws && c->profiling && !c->ev_pool.empty()) release_events(c);

    float* ws = nullptr;
    Workspace lay;
    if (!static_ws) c->have_fwd = false;     // a static call leaves the handle's own forward state alone
    // the top layers run in one persistent kernel; when that kernel starts at layer 1 it evaluates the
    // leaf layer itself (a workgroup reads its own rows of the weight arrays)
    int top_first = choose_top(c, B, semiring == KLAY_REAL && !static_ws && c->bwd_followed);
    bool with_bwd = false;
    klay_status st = forward_workspace(c, B, static_ws, top_first, with_bwd, &ws, &lay);
    if (st != KLAY_OK) return st;
    const TailChoice tail = top_first > 0 ? TailChoice() : choose_tail_fwd(c, B);
    const bool fused_leaf = tail.first == 1 || top_first == 1;

    float* act = ws + lay.act;
    float* wT = ws + lay.wT;
    float* seg_rows = ws + lay.seg_rows;
    const int L = p.num_layers;
    const int V = p.num_vars;
    Profiler prof(c, &c->ev_fwd, s, !static_ws);

    // leaf layer
    if (!fused_leaf) {
        prof.begin(KLAY_K_LEAF, 4.0 * B * V + 4.0 * B * (double)(V + p.layers[0].n));
        if (V > 0 && g.ld == B && B <= 32) {
            hipLaunchKernelGGL(klay::leaf_fwd_small_kernel, dim3((unsigned)(((int64_t)V * B + 255) / 256)), dim3(256), 0, s,
                               leaf_weights, neg_weights, (int)B, V, c->d_pos_row, c->d_neg_row, wT, act, log_domain ? 1 : 0);
        } else if (V > 0) {
            dim3 grid((unsigned)((V + 31) / 32), (unsigned)((g.ld + 63) / 64));
            hipLaunchKernelGGL(klay::leaf_fwd_kernel, grid, dim3(klay::kLeafThreads), 0, s, leaf_weights, neg_weights, (int)B, V, g.ld,
                               c->d_pos_row, c->d_neg_row, wT, act, log_domain ? 1 : 0);
        }
        if (c->true_row >= 0)
            hipLaunchKernelGGL(klay::fill_row_kernel, dim3((unsigned)((g.ld + 255) / 256)), dim3(256), 0, s,
                               act + (size_t)c->true_row * g.ld, g.ld, log_domain ? 0.0f : 1.0f);
        if (c->false_row >= 0)
            hipLaunchKernelGGL(klay::fill_row_kernel, dim3((unsigned)((g.ld + 255) / 256)), dim3(256), 0, s,
                               act + (size_t)c->false_row * g.ld, g.ld, log_domain ? -INFINITY : 0.0f);
        prof.end();
    }

    // gate layers: odd = AND, even = OR (Alg. 1 / Alg. 4)
    // The fused plans run where the streaming kernel takes main rows and segments in one launch (two or four
    // columns per lane).
    // A handle whose previous forward pass was followed by klay_backward is in a training loop: the reverse sweep
    // needs every value, so this pass writes them all (klay_backward would otherwise evaluate the fused rows first).
    const bool fused = g.w == 64 && g.vec >= 2 && p.num_fused > 0 && !c->no_fusion &&
                       (static_ws || !c->bwd_followed);
    const int last_regular = top_first > 0 ? top_first - 1 : tail.first > 0 ? tail.first - 1 : L;
    for (int l = 1; l <= last_regular; ++l) {
        const DevLayer& d = c->dl[(size_t)l];
        const bool is_and = (l & 1) != 0;
        const int or_op = semiring == KLAY_MAXLOG ? klay::OP_MAX : klay::OP_LSE;
        const int op = log_domain ? (is_and ? klay::OP_SUM : or_op) : (is_and ? klay::OP_PROD : klay::OP_SUM);
        const int cls = op == klay::OP_SUM ? KLAY_K_FWD_SUM
                        : op == klay::OP_PROD ? KLAY_K_FWD_PROD
                        : op == klay::OP_MAX ? KLAY_K_FWD_MAX : KLAY_K_FWD_LSE;
        // up to alias_top child entries are rows of the whole buffer, above it of the layer below
        const float* below = l <= p.alias_top ? act : act + (size_t)c->dl[(size_t)l - 1].row0 * g.ld;
        if (fused && is_and && d.n_fused > 0 && !(top_first > 0 && l >= top_first - 1)) {
            // the fused rows are not evaluated: the OR rows above read their children (those of the layer that the TopPlan's
            // kernel reads are)
            if (d.has_fwd_kept) run_pass_set(op, op, d.fwd_kept, below, nullptr, nullptr, act + (size_t)d.row0 * g.ld, seg_rows, g, B, s, prof, cls);
        } else if (fused && !is_and && d.has_fwd2) {
            run_pass_set(!log_domain ? klay::OP_SUMPROD2 : semiring == KLAY_MAXLOG ? klay::OP_MAX2 : klay::OP_LSE2, op, d.fwd2, below, nullptr, nullptr,
                         act + (size_t)d.row0 * g.ld, seg_rows, g, B, s, prof, KLAY_K_FWD_OR_FUSED);
        } else {
            run_pass_set(op, op, d.fwd, below, nullptr, nullptr, act + (size_t)d.row0 * g.ld, seg_rows, g, B, s, prof, cls);
        }
    }

    if (tail.first > 0 || top_first > 0) {
        // the persistent kernel also writes out[B, R]: the top layer is in its LDS
        klay::SlabLeaf leaf{};
        if (fused_leaf) {
            leaf.w = leaf_weights;
            leaf.wneg = neg_weights;
            leaf.pos_row = c->n_leaf_list ? c->d_leaf_list : c->d_pos_row;
            leaf.neg_row = c->n_leaf_list ? c->d_leaf_list + c->n_leaf_list : c->d_neg_row;
            leaf.true_row = c->true_row;
            leaf.false_row = c->false_row;
            leaf.wT = wT;
            leaf.act0 = act;
            leaf.V = V;
        }
        const ColTail& which = top_first > 0 ? c->top : c->tail;
        const int first = top_first > 0 ? top_first : tail.first;
        prof.begin(KLAY_K_TAIL_FWD, tail_alg_bytes(which, first, B, false) + 8.0 * B * p.num_roots,
                   tail_min_bytes(which, first, B, false) + 4.0 * B * p.num_roots);
        if (top_first > 0)
            launch_top_fwd(c, top_first, act, lay.top_stage_n ? ws + lay.top_stage : nullptr, with_bwd ? ws + lay.top_tb : nullptr, B, g.ld, (int)semiring, leaf, out, s);
        else
            launch_tail_fwd(c, tail, act, ws + lay.tb, !static_ws, B, g.ld, (int)semiring, leaf, out, s);
        prof.end();
    } else {
        prof.begin(KLAY_K_ROOT, 8.0 * B * p.num_roots);
        dim3 grid((unsigned)p.num_roots);
        hipLaunchKernelGGL(klay::root_out_kernel, grid, dim3(256), 0, s,
                           act + (size_t)c->dl[(size_t)L].row0 * g.ld, c->d_root_pos, (int)B, p.num_roots, g.ld, out);
        prof.end();
    }
    KLAY_HIP(hipGetLastError());
    if (static_ws) return KLAY_OK;       // the values live in the shared array: nothing to differentiate later
    c->have_fwd = true;
    c->last_fused = fused;
    c->bwd_followed = false;
    c->last_B = B;
    c->last_semiring = semiring;
    c->last_neg_explicit = neg_weights != nullptr;
    c->last_ws_has_bwd = with_bwd;
    c->last_tail_first = tail.first;
    c->last_top_first = top_first;
    const TailBuffer buf = tail.first > 0 ? tail_buffer(c, tail, B) : TailBuffer();
    c->last_tail_T = (int32_t)buf.T;
    c->last_tail_staged = buf.at >= 0;
    return KLAY_OK;
}

static klay_status backward_impl(klay_circuit* c, const float* dout, float* dleaf, float* dneg, bool lits,
                                 void* stream) {
    if (!c || !dout || !dleaf) return fail(KLAY_EINVAL, "klay_backward: null argument");
    if (c->device < 0) return fail(KLAY_ESTATE, "klay_backward: host-only handle");
    if (!c->have_fwd) return fail(KLAY_ESTATE, "klay_backward: no forward pass to differentiate");
    if (lits != c->last_neg_explicit)
        return fail(KLAY_ESTATE, lits ? "klay_backward_lits: the forward pass was not run by klay_forward_lits with neg_weights"
                                      : "klay_backward: the forward pass had weights for the negated literals; use klay_backward_lits");
    if (c->last_semiring == KLAY_MAXLOG)
        return fail(KLAY_EINVAL, "klay_backward: the (max, +) semiring is not differentiated");
    const bool real = c->last_semiring == KLAY_REAL;
    if (!c->last_ws_has_bwd) return fail(KLAY_ENOMEM, "klay_backward: caller workspace has no room for adjoints");
    KLAY_HIP(hipSetDevice(c->device));
    hipStream_t s = static_cast<hipStream_t>(stream);
    const klay::CircuitPlan& p = c->plan;
    const int B = c->last_B;
    const Geometry g = geometry(B);
    float* ws = nullptr;
    const Workspace lay = workspace_layout(c, B, true, c->last_top_first);
    klay_status st = get_workspace(c, lay.total, &ws);
    if (st != KLAY_OK) return st;
    float* act = ws + lay.act;
    float* wT = ws + lay.wT;
    float* seg_rows = ws + lay.seg_rows;
    float* G = ws + lay.g0;
    float* gcur = ws + lay.g1;
    float* gnext = ws + lay.g2;
    const int L = p.num_layers, V = p.num_vars, R = p.num_roots, B0 = p.alias_top;
    Profiler prof(c, &c->ev_bwd, s);
    // Course of the sweep.  The layers above B0 = alias_top are taken one by one, every step gathering the
    // adjoints of layer l - 1 from those of layer l, alternating between two buffers; the step into layer
    // B0 writes into G, which holds one adjoint row per node of the layers 0 .. B0, numbered like the rows
    // of the activation buffer.  Below B0 a layer's rows gather from their parents anywhere in G (all
    // final by then).  The leaf kernel reads the rows of layer 0 at the start of G.
    auto grow = [&](int l) { return G + (size_t)c->dl[(size_t)l].row0 * g.ld; };
    auto values = [&](int l) { return act + (size_t)c->dl[(size_t)l].row0 * g.ld; };

    c->bwd_followed = true;
    if (c->last_fused) {
        // The forward pass ran the fused plans: the values of the fused AND rows, which this sweep needs, were
        // never written.  Evaluate those layers now (all their rows; the others come out the same again).
        for (int l = 1; l < (c->last_top_first > 0 ? c->last_top_first - 1 : B0); l += 2) {
            const DevLayer& d = c->dl[(size_t)l];
            if (d.n_fused > 0)
                run_pass_set(real ? klay::OP_PROD : klay::OP_SUM, real ? klay::OP_PROD : klay::OP_SUM, d.fwd, act, nullptr, nullptr,
                             values(l), seg_rows, g, B, s, prof, real ? KLAY_K_FWD_PROD : KLAY_K_FWD_SUM);
        }
        c->last_fused = false;
    }

    // The layers the forward pass ran in the persistent kernel, swept by its reverse counterpart; returns the layer whose
    // adjoint rows it leaves (0: it wrote the leaf gradients).
    auto tail_sweep = [&](const uint32_t* top_multi, const klay::ColReal* real_args) {
        const int first = c->last_tail_first;
        int last = first;
        float* cols = gnext;                       // its last layer's adjoints, column-major
        if (first == 1) last = 0;
        else if (c->last_tail_staged) {
            const int64_t nb = c->dl[(size_t)first - 1].n;
            if (nb <= top_layer_rows(p)) last = first - 1;
            else if (first - 1 == B0 && nb <= c->dl[(size_t)B0].row0) { last = first - 1; cols = G; }      // rows not written yet
        }
        klay::ColBwdOut res{};
        res.n_last = (int32_t)c->dl[(size_t)last].n;
        if (last == 0) {
            res.wT = wT;
            res.pos_row = c->d_pos_row;
            res.neg_row = c->d_neg_row;
            res.dleaf = dleaf;
            res.dneg = dneg;
            res.V = V;
            res.mode = lits ? 2 : (real ? 0 : 1);
        } else {
            res.g_cols = cols;
            res.g_T = res.n_last;
        }
        prof.begin(KLAY_K_TAIL_BWD, tail_alg_bytes(c->tail, first, B, true) + 4.0 * B * R, tail_min_bytes(c->tail, first, B, true) + 4.0 * B * R);
        launch_tail_bwd(c, c->tail, last, last > 0 ? (int)p.col_off[(size_t)last] : -1, ws + lay.tb, c->last_tail_T, dout, top_multi, res,
                        real_args, B, g.ld, s);
        if (last > 0) {
            dim3 tgrid((unsigned)((res.n_last + 31) / 32), (unsigned)((g.ld + 31) / 32));
            hipLaunchKernelGGL(klay::tb_to_rows_kernel<false>, tgrid, dim3(256), 0, s, cols, res.n_last, 0, res.n_last, B, g.ld,
                               last == B0 ? grow(B0) : gcur, (const int32_t*)nullptr);
        }
        prof.end();
        return last;
    };

    const bool one = kOneGather && c->one_gather;
    if (c->last_top_first > 0 && (real || !one)) {
        // this sweep runs layer by layer on rows of the activation buffer
        launch_top_to_rows(c, c->last_top_first, L, ws + lay.top_tb, act, B, g.ld, s);
    }

    if (real) {
        // Real semiring: a sum layer passes adjoints through (plain by-child sums).  For a product layer
        // the adjoint rows of its nodes are first turned, in place, into P rows (adjoint times the product
        // of the non-zero children, prod_parent_kernel), and the by-child pass OP_PROD_BWD hands every
        // child its share, using the child's own value.  Nothing is stored per edge.
        klay_status rs = ensure_real_bwd(c);
        if (rs != KLAY_OK) return rs;
        // The layers of the persistent forward kernel go to its reverse counterpart (whose product rows arrive below as
        // finished P rows); without it the sweep runs layer by layer on rows of the activation buffer.
        const bool columns = c->last_tail_first > 0 && c->d_real_ptr;
        int top = L;
        if (columns) {
            klay::ColReal args{};
            args.index = c->d_real_index;
            args.ptr = c->d_real_ptr;
            args.child = c->d_real_child;
            args.rows = values(c->last_tail_first - 1);
            const int below = c->last_tail_first - 1;
            args.low_rows = below <= B0 ? act : values(below - 1);
            args.lowest = L - below;
            top = tail_sweep(nullptr, &args);
            if (top == 0) {
                KLAY_HIP(hipGetLastError());
                return KLAY_OK;
            }
        } else if (c->last_tail_first > 0) {
            launch_tb_to_rows(c, c->last_tail_first, L, ws + lay.tb, act, B, g.ld, s);
        }
        // `pre`: the rows arrive premultiplied by the pass that produced them (OP_SUM_P, OP_PROD_BWD_P), and the
        // kernel only repairs the columns whose node value is zero; the seed's rows are plain adjoints
        // flags[l]: raised by the pass that writes the rows of product layer l when it meets a node value of zero
        int* flags = reinterpret_cast<int*>(ws + lay.flags);
        hipLaunchKernelGGL(klay::fill_row_kernel, dim3((unsigned)((L + 256) / 256)), dim3(256), 0, s, ws + lay.flags, L + 1, 0.0f);
        auto prod_parent = [&](int l, const float* below, float* gl, bool pre) {
            const DevLayer& d = c->dl[(size_t)l];
            prof.begin(KLAY_K_PROD_EDGES, pre ? 4.0 : 4.0 * B * ((double)d.e + 2.0 * (double)d.n));
            launch_prod_parent(c->real_layers[(size_t)l], (int)d.n, below, gl, pre ? values(l) : nullptr, flags + l, g, B, s);
            prof.end();
        };
        if (!columns) {
            prof.begin(KLAY_K_SEED, 4.0 * B * R + 4.0 * B * (double)c->dl[(size_t)L].n);
            hipLaunchKernelGGL(klay::seed_kernel, dim3((unsigned)c->dl[(size_t)L].n), dim3(256), 0, s, dout, c->d_top_ptr,
                               c->d_top_root, B, R, g.ld, L == B0 ? grow(L) : gcur, (const uint32_t*)nullptr,
                               (const float*)nullptr);
            prof.end();
        }
        for (int l = top; l > B0; --l) {
            const DevLayer& d = c->dl[(size_t)l];
            float* dst = l - 1 == B0 ? grow(B0) : gnext;
            if ((l & 1) == 0) {
                // into an AND layer: plain sums, leaving premultiplied by the nodes' own values
                run_pass_set(klay::OP_SUM_P, klay::OP_SUM_P, d.bwd, gcur, nullptr, values(l - 1), dst, seg_rows, g, B, s,
                             prof, KLAY_K_BWD_SUM_MUL, flags + (l - 1));
            } else {
                if (!(columns && l == top)) prod_parent(l, values(l - 1), gcur, l != L);
                // the by-child plan of an AND layer carries no weighted bit: every entry is a P row
                run_pass_set(klay::OP_PROD_BWD, klay::OP_SUM, d.bwd, gcur, nullptr, values(l - 1), dst, seg_rows, g, B, s,
                             prof, KLAY_K_BWD_PROD);
            }
            std::swap(gcur, gnext);
        }
        // below B0 the entries of a by-child plan tell P rows (AND parents) from plain adjoint rows
        if (B0 > 0 && (B0 & 1) && !(columns && top == B0)) prod_parent(B0, act, grow(B0), B0 != L);
        for (int l = B0 - 1; l >= 0; --l) {
            const bool and_rows = (l & 1) != 0;
            run_pass_set(and_rows ? klay::OP_PROD_BWD_P : klay::OP_PROD_BWD, and_rows ? klay::OP_SUM_P : klay::OP_SUM,
                         c->real_layers[(size_t)l].by_child, G, nullptr, values(l), grow(l), seg_rows, g, B, s, prof,
                         and_rows ? KLAY_K_BWD_PROD_MUL : KLAY_K_BWD_PROD, and_rows ? flags + l : nullptr);
            if (and_rows) prod_parent(l, act, grow(l), true);
        }
    } else {
        // The adjoint rows of an OR layer with weighted edges travel in the one-gather form (encode_h): the
        // step that produces them (OP_SUM_H, the seed, or the persistent kernel's last write) folds the
        // node's own value in, and the step through the OR layer (OP_SOFTMAX_H) gathers that one row per
        // edge instead of the adjoint row and the parent's value row.
        auto encoded = [&](int l) { return one && l >= 2 && (l & 1) == 0 && c->dl[(size_t)l].has_multi; };

        // The layers the forward pass ran in the persistent kernel are swept by its reverse counterpart, which
        // seeds the adjoints itself.  Where it can it also takes the step into the layer below them: to the leaves,
        // whose gradients it then writes itself, or into a layer whose values are in the column-major buffer.
        int top = L, low = B0 - 1;        // the layers top .. B0 + 1 one by one, then the rows of the layers low .. 0
        const int first = c->last_tail_first;
        if (one && c->last_top_first > 0) {
            // the levels of a TopPlan down to its first one, whose adjoints and those above it (as far as they have rows) go
            // to their rows; the launches go on below.  From layer 1 on it takes the step to the leaves, too.
            const int top_first = c->last_top_first;
            klay::ColBwdOut res{};
            int last = top_first;
            if (top_first == 1) {
                last = 0;
                res.wT = wT;
                res.pos_row = c->d_pos_row;
                res.neg_row = c->d_neg_row;
                res.dleaf = dleaf;
                res.dneg = dneg;
                res.V = V;
                res.mode = lits ? 2 : 1;
            } else {
                res.keep = ws + lay.top_g;
                res.keep_from = L - B0;
                res.g_cols = ws + lay.top_g + c->top.at[(size_t)last];
                res.g_T = (int32_t)c->top.rows;
            }
            res.n_last = (int32_t)c->top.kept[(size_t)last];
            prof.begin(KLAY_K_TAIL_BWD, tail_alg_bytes(c->top, top_first, B, true) + 4.0 * B * R, tail_min_bytes(c->top, top_first, B, true) + 4.0 * B * R);
            launch_tail_bwd(c, c->top, last, last > 0 ? (int)c->top.at[(size_t)last] : -1, ws + lay.top_tb, (int)c->top.rows, dout, c->top.multi, res,
                            nullptr, B, g.ld, s);
            if (last > 0) launch_top_to_rows(c, last, B0, ws + lay.top_g, G, B, g.ld, s);
            prof.end();
            if (last == 0) {
                KLAY_HIP(hipGetLastError());
                return KLAY_OK;
            }
            top = B0;
            low = last - 1;
        } else
        // (its adjoints of OR nodes are in the one-gather form throughout, so it needs that form to be in use)
        if (one && first > 0) {
            top = tail_sweep(encoded(L) ? c->dl[(size_t)L].multi : nullptr, nullptr);
            if (top == 0) {
                KLAY_HIP(hipGetLastError());
                return KLAY_OK;
            }
        } else {
            // the ordinary launches below read the values the persistent forward kernel kept column-major as rows
            // of the activation buffer
            if (first > 0) launch_tb_to_rows(c, first, L, ws + lay.tb, act, B, g.ld, s);
            const bool enc = encoded(L);
            prof.begin(KLAY_K_SEED, 4.0 * B * R + 4.0 * B * (double)c->dl[(size_t)L].n * (enc ? 2.0 : 1.0));
            dim3 grid((unsigned)c->dl[(size_t)L].n);
            hipLaunchKernelGGL(klay::seed_kernel, grid, dim3(256), 0, s, dout, c->d_top_ptr, c->d_top_root, B, R, g.ld,
                               L == B0 ? grow(L) : gcur, enc ? c->dl[(size_t)L].multi : (const uint32_t*)nullptr,
                               enc ? values(L) : (const float*)nullptr);
            prof.end();
        }
        for (int l = top; l > B0; --l) {
            const DevLayer& d = c->dl[(size_t)l];
            float* dst = l - 1 == B0 ? grow(B0) : gnext;
            const bool is_and = (l & 1) != 0 || !d.bwd.has_weighted;   // no weighted edge: plain sums
            if (is_and) {
                const bool enc = encoded(l - 1);
                run_pass_set(enc ? klay::OP_SUM_H : klay::OP_SUM, enc ? klay::OP_SUM_H : klay::OP_SUM, d.bwd, gcur, nullptr,
                             enc ? values(l - 1) : nullptr, dst, seg_rows, g, B, s, prof,
                             enc ? KLAY_K_BWD_SUM_ENC : KLAY_K_BWD_SUM);
            } else if (one) {
                run_pass_set(klay::OP_SOFTMAX_H, klay::OP_SUM, d.bwd, gcur, nullptr, values(l - 1), dst, seg_rows, g, B, s,
                             prof, KLAY_K_BWD_SOFTMAX_ONE);
            } else {
                run_pass_set(klay::OP_SOFTMAX_BWD, klay::OP_SUM, d.bwd, gcur, values(l), values(l - 1), dst, seg_rows, g, B,
                             s, prof, KLAY_K_BWD_SOFTMAX);
            }
            std::swap(gcur, gnext);
        }
        for (int l = low; l >= 0; --l) {
            // rows of even layers are OR nodes, whose parents are AND nodes (plain sums; encoded on the way
            // out where the node has more than one child); rows of odd layers and leaves read weighted edges
            const DevPass& dp = c->dl[(size_t)l + 1].bwd;
            const bool enc = encoded(l);
            if (one && (enc || dp.has_weighted))
                run_pass_set(enc ? klay::OP_SUM_H : klay::OP_SOFTMAX_H, enc ? klay::OP_SUM_H : klay::OP_SUM, dp, G, nullptr,
                             values(l), grow(l), seg_rows, g, B, s, prof, enc ? KLAY_K_BWD_SUM_ENC : KLAY_K_BWD_SOFTMAX_ONE);
            else if (dp.has_weighted)
                run_pass_set(klay::OP_SOFTMAX_BWD, klay::OP_SUM, dp, G, act, values(l), grow(l), seg_rows, g, B, s, prof,
                             KLAY_K_BWD_SOFTMAX);
            else
                run_pass_set(klay::OP_SUM, klay::OP_SUM, dp, G, nullptr, nullptr, grow(l), seg_rows, g, B, s, prof,
                             KLAY_K_BWD_SUM);
        }
    }

    prof.begin(KLAY_K_BWD_LEAF, 4.0 * B * (3.0 * V));
    if (V > 0) {
        dim3 grid((unsigned)((V + 31) / 32), (unsigned)((B + 63) / 64));
        hipLaunchKernelGGL(klay::leaf_bwd_kernel, grid, dim3(klay::kLeafThreads), 0, s, G, wT, c->d_pos_row, c->d_neg_row, B, V, g.ld,
                           lits ? 2 : (real ? 0 : 1), dleaf, dneg);
    }
    prof.end();
    KLAY_HIP(hipGetLastError());
    return KLAY_OK;
}

// No C++ exception crosses the C boundary: host allocations of the launch sequences (event records,
// the index arrays of the real-semiring reverse sweep) report KLAY_ENOMEM instead.
klay_status klay_forward(klay_circuit* c, const float* leaf_weights, int32_t B, float* out,
                         klay_semiring semiring, void* stream) {
    return klay_forward_lits(c, leaf_weights, nullptr, B, out, semiring, stream);
}

klay_status klay_forward_lits(klay_circuit* c, const float* pos_weights, const float* neg_weights, int32_t B,
                              float* out, klay_semiring semiring, void* stream) {
    try {
        return forward_impl(c, pos_weights, neg_weights, B, out, semiring, stream);
    } catch (const std::bad_alloc&) {
        if (c) c->have_fwd = false;
        return fail(KLAY_ENOMEM, "klay_forward: out of host memory");
    }
}

klay_status klay_forward_static(klay_circuit* c, const float* leaf_weights, int32_t B, float* out,
                                klay_semiring semiring, void* stream) {
    try {
        return forward_impl(c, leaf_weights, nullptr, B, out, semiring, stream, true);
    } catch (const std::bad_alloc&) {
        return fail(KLAY_ENOMEM, "klay_forward_static: out of host memory");
    }
}

klay_status klay_backward(klay_circuit* c, const float* dout, float* dleaf, void* stream) {
    try {
        return backward_impl(c, dout, dleaf, nullptr, false, stream);
    } catch (const std::bad_alloc&) {
        return fail(KLAY_ENOMEM, "klay_backward: out of host memory");
    }
}

klay_status klay_backward_lits(klay_circuit* c, const float* dout, float* dpos, float* dneg, void* stream) {
    try {
        return backward_impl(c, dout, dpos, dneg, true, stream);
    } catch (const std::bad_alloc&) {
        return fail(KLAY_ENOMEM, "klay_backward_lits: out of host memory");
    }
}

klay_status klay_forward_f64(klay_circuit* c, const double* pos_weights, const double* neg_weights, int32_t B,
                             double* out, klay_semiring semiring, void* stream) {
    try {
        return forward64_impl(c, pos_weights, neg_weights, B, out, semiring, stream);
    } catch (const std::bad_alloc&) {
        if (c) c->have_fwd64 = false;
        return fail(KLAY_ENOMEM, "klay_forward_f64: out of host memory");
    }
}

klay_status klay_backward_f64(klay_circuit* c, const double* dout, double* dpos, double* dneg, void* stream) {
    try {
        return backward64_impl(c, dout, dpos, dneg, stream);
    } catch (const std::bad_alloc&) {
        return fail(KLAY_ENOMEM, "klay_backward_f64: out of host memory");
    }
}

}  // extern "C"
