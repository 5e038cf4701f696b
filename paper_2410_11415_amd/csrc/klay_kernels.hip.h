// Device kernels of the layered circuit evaluator for gfx950 (wave64).
//
// Data layout: every layer's node values live in one activation buffer, row = node,
// `ld` consecutive floats per row = the batch (batch-inner), so the gather of one edge
// (paper Section 4: E_l = N_{l-1}[S_l]) is one contiguous read of B floats.  A layer is
// evaluated by a fused gather + segment-reduce (Alg. 1 / Alg. 4 without materialising E_l,
// M or T): a lane group of W lanes owns one parent row and VEC consecutive batch columns per
// lane, loops over the row's CSR range and keeps the reduction in registers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "layerize.h"

namespace klay {

enum PassOp : int { OP_SUM = 0, OP_PROD = 1, OP_LSE = 2, OP_SOFTMAX_BWD = 3, OP_MAX = 4, OP_PROD_BWD = 5, OP_SUM_H = 6, OP_SOFTMAX_H = 7,
                    OP_SUM_P = 8, OP_PROD_BWD_P = 9,
                    // over the fused plans (see LayerPlan::fwd2): an OR row whose children are groups of entries
                    // (sum within a group, then logsumexp / max over the groups; real semiring: product within a
                    // group, then the sum of the groups)
                    OP_LSE2 = 10, OP_MAX2 = 11, OP_SUMPROD2 = 12 };
// what the ops have in common: `own` = the walk needs the value of the output row itself, `additive` = partial
// results add up
template <int OP> struct OpTraits {
    static constexpr bool own = OP == OP_SOFTMAX_BWD || OP == OP_PROD_BWD || OP == OP_SUM_H || OP == OP_SOFTMAX_H ||
                                OP == OP_SUM_P || OP == OP_PROD_BWD_P;
    static constexpr bool additive = OP == OP_SUM || own;
    static constexpr bool premul = OP == OP_SUM_P || OP == OP_PROD_BWD_P;      // the row leaves multiplied by its own value
    static constexpr bool shares = OP == OP_PROD_BWD || OP == OP_PROD_BWD_P;   // entries are P rows of AND parents
    // a segment of a split row needs the value of the row that owns it (the others only use it to finish a row)
    static constexpr bool seg_own = OP == OP_SOFTMAX_BWD || OP == OP_SOFTMAX_H || shares;
};

// Index entries: bits 0..28 = source row, bit 31 = last edge of its output row, bit 30 = weighted
// edge (reverse sweep only: the parent is an OR node with more than one child, so the adjoint
// passes through the softmax weight exp(child - parent); an unweighted edge passes it unchanged),
// bit 29 (on the last entry of a row only) = the output row is an OR node with more than one child, whose
// adjoint is stored in the one-gather form (see encode_h).
// kSkip (all ones) stands for a whole output row that this pass leaves untouched (a split row).
constexpr uint32_t kLast = kLastEdge, kWeighted = kWeightedEdge, kSkip = kSkipRow, kIdMask = kRowFlag - 1u;

struct PassArgs {
    const int32_t* ptr;        // [n_total + 1] CSR offsets into idx
    const uint32_t* idx;       // index entries (readable up to 16 entries past the end)
    const float* src;          // [*, ld] source rows (values of the layer below, adjoints, or partials)
    const float* src2;         // OP_SOFTMAX_BWD: values N_l of the parents, same row index as src
    const float* own;          // ops with OpTraits::own: values of the output rows themselves
    const int32_t* seg_owner;  // output row owning segment i (rows >= n_main), may be null
    const int32_t* out_row;    // optional output row map for rows < n_main (combine pass)
    float* dst;                // output rows for rows < n_main
    float* dst_seg;            // scratch rows for rows >= n_main
    int32_t lanes, per_wave;   // generic kernel: lanes per row, rows per wave
    uint32_t inverse;          // see lane_group
    int32_t row_begin;         // first row this launch evaluates
    int32_t n_main;
    int32_t n_total;
    int32_t B;
    int32_t ld;
    int* zero_flag;            // OP_SUM_P, OP_PROD_BWD_P: set to 1 when an output row's own value is zero in some column
};

// s_waitcnt immediate (gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8) that waits
// for vmcnt = 0 only: expcnt and lgkmcnt keep their maxima (7 and 15), so scalar loads stay in flight.
constexpr int kWaitVmcnt0 = 0x0F70;

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// exp and log on the transcendental unit (v_exp_f32 / v_log_f32 are base 2).  Arguments of
// fexp are <= 0 here, so the rounding of x*log2(e) costs at most |x| e^x 2^-24 absolute.
__device__ __forceinline__ float fexp(float x) { return __builtin_amdgcn_exp2f(x * kLog2e); }
__device__ __forceinline__ float flog(float x) { return __builtin_amdgcn_logf(x) * kLn2; }

// the largest of those that are no NaN
__device__ __forceinline__ float max3(float a, float b, float c) {
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
__device__ __forceinline__ float bigger(float a, float b) {
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
constexpr float kFltMax = 3.402823466e+38f;

// A NaN in the log domain (a weight above 0 leaves one for its negated literal) is an impossible child of an OR row, in every
// fp32 kernel: its term counts 0, the maximum passes it by, and a row of nothing else is -inf.  (An AND row with one
// is NaN.)
// exp of a term of a logsumexp, x = term - finite(maximum): at most 1; 1 for an infinite weight, 0 for a NaN.  The clamp is
// a bit of the exponential's own instruction.
__device__ __forceinline__ float term_exp(float x) { return __builtin_amdgcn_fmed3f(fexp(x), 0.0f, 1.0f); }
__device__ __forceinline__ float finite(float m) { return __builtin_amdgcn_fmed3f(m, -kFltMax, kFltMax); }

template <int VEC> struct Pack;
template <> struct Pack<1> { using T = float; };
template <> struct Pack<2> { using T = float2; };
template <> struct Pack<4> { using T = float4; };

template <int VEC>
__device__ __forceinline__ void load_vec(float (&x)[VEC], const float* p) {
    using T = typename Pack<VEC>::T;
    T t = *reinterpret_cast<const T*>(p);
    const float* f = reinterpret_cast<const float*>(&t);
#pragma unroll
    for (int v = 0; v < VEC; ++v) x[v] = f[v];
}

// Streaming store: the rows of a wide layer are written once and next read by another kernel,
// long after they have left the 4 MB L2, so they are marked non-temporal to leave the L2 to the
// gathers.  Narrow layers keep ordinary stores: their rows are still in L2 when the next layer reads.
template <int VEC>
__device__ __forceinline__ void store_vec_stream(float* p, const float (&x)[VEC]) {
    typedef float vf __attribute__((ext_vector_type(VEC)));
    vf t;
#pragma unroll
    for (int v = 0; v < VEC; ++v) t[v] = x[v];
    __builtin_nontemporal_store(t, reinterpret_cast<vf*>(p));
}
template <>
__device__ __forceinline__ void store_vec_stream<1>(float* p, const float (&x)[1]) {
    __builtin_nontemporal_store(x[0], p);
}

template <int VEC>
__device__ __forceinline__ void store_vec(float* p, const float (&x)[VEC]) {
    using T = typename Pack<VEC>::T;
    T t;
    float* f = reinterpret_cast<float*>(&t);
#pragma unroll
    for (int v = 0; v < VEC; ++v) f[v] = x[v];
    *reinterpret_cast<T*>(p) = t;
}

// Workgroups are handed to the 8 XCDs round-robin; give each XCD a contiguous eighth of the
// rows so that neighbouring rows (which read neighbouring children) share one L2.  The grid's
// x extent is a multiple of 8.  (Measured on the headline workload: 4% of the step, and 28% of
// the time of the split-row segments, which are ordered by the rows they read.)
__device__ __forceinline__ int xcd_block(int bid, int nblocks) { return (bid & 7) * (nblocks >> 3) + (bid >> 3); }

// One step of the streaming reductions.  acc/mx carry the state of the current output row:
//   OP_SUM / OP_PROD  acc = running sum / product
//   OP_MAX            acc = running maximum (OR layers of the (max, +) semiring)
//   OP_LSE            (mx, acc) = (running max, sum of exp(x - mx)); one exp per element:
//                     a new maximum rescales the sum by exp(mx - x), otherwise exp(x - mx) is added
//   OP_SOFTMAX_BWD    acc += g * exp(own - parent value) on weighted edges (a parent at -inf
//                     passes nothing down), acc += g on unweighted ones
//   OP_PROD_BWD       real-semiring reverse sweep: x is the row that prod_parent_kernel left for an AND
//                     parent r, P_r = G_r * (product of r's non-zero children), with the lowest mantissa
//                     bit telling whether r has exactly one zero child (rows with more are all zero).
//                     The child with value `own` gets P_r / own when r has no zero child, P_r when the
//                     child is r's one zero, nothing otherwise.  A weighted entry is a plain adjoint row
//                     (a sum node above, or a root's dout row) and is added as it is.  acc = sum of the plain entries, mx = sum of
//                     the P_r that concern the child (-0 as long as there is none), divided by `own` once, in finish():
//                     a division takes ten instructions, and one per entry and column bound the wide layers (800000
//                     nodes at B = 256, training step 1251 -> 1185 us).  Where that sum may leave the range, the P_r are
//                     added times a power of two that is about 1 / own (share_scale): it stays in range wherever the quotients do.
//   OP_SUM_P, OP_PROD_BWD_P   OP_SUM / OP_PROD_BWD whose output rows are AND nodes: the finished adjoint G
//                     leaves as G * (the node's own value), lowest mantissa bit clear, which is the row P
//                     above whenever the node has no zero child; where the own value is zero G is left
//                     as it is for prod_parent_kernel to deal with (see there).
// One-gather form of the softmax adjoint (log semiring, reverse sweep through an OR layer).  The adjoint
// G_r of an OR node r with more than one child only ever reaches its children as G_r exp(N_c - N_r), so
// the pass that produces G_r (OP_SUM_H: a plain sum, finished with the node's own value N_r) stores
//   H_r = log|G_r| - N_r, with the sign of G_r in the lowest mantissa bit (-inf when G_r = 0 or N_r = -inf),
// and the pass through the OR layer (OP_SOFTMAX_H) gathers that one row per edge and adds
// +-exp(H_r + N_c): N_c <= N_r, so nothing overflows.  Rows of single-child OR nodes (and chain nodes)
// keep the plain adjoint; their edges are the unweighted ones and pass it unchanged.
__device__ __forceinline__ float encode_h(float g, float n) {
    const bool none = g == 0.0f || n == -INFINITY;
    const float h = none ? -INFINITY : flog(fabsf(g)) - n;
    return __uint_as_float((__float_as_uint(h) & ~1u) | ((g < 0.0f && !none) ? 1u : 0u));
}
__device__ __forceinline__ float decode_h(float hbits, float nc) {
    const uint32_t b = __float_as_uint(hbits);
    const float v = fexp(__uint_as_float(b & ~1u) + nc);
    return __uint_as_float(__float_as_uint(v) | (b << 31));      // v >= 0: the stored sign bit goes on with one shift-or
}

__device__ __forceinline__ float premultiply(float g, float n) {
    return n != 0.0f ? __uint_as_float(__float_as_uint(g * n) & ~1u) : g;
}

// The power of two by which the P_r of a child of value n are scaled before they are added: n times it is in [1/2, 1) (less
// below 2^-126; from 2^126 on up to 4, where P_r / n is below 4), so a scaled P_r is in range wherever the quotient
// P_r / n is, and scaling rounds nothing that the quotient would not.  1 for n = 0.
__device__ __forceinline__ float share_scale(float n) {
    const int bits = 0x7E800000 - (int)(__float_as_uint(n) & 0x7F800000u);
    return n == 0.0f ? 1.0f : __uint_as_float((uint32_t)(bits > 0x00800000 ? bits : 0x00800000));
}

// one element of a running logsumexp: (mx, acc) = (maximum so far, sum of exp(x - mx)), one exp per element
__device__ __forceinline__ void lse_step(float& acc, float& mx, float x) {
    // d is +inf on the first finite element (e = 0, acc = 1), -inf for an impossible child under a finite
    // maximum (e = 0), and NaN only for -inf - -inf and for a NaN, where the clamp of the exponential makes it 0 and the comparison fails
    const float d = x - mx;
    const float e = term_exp(-fabsf(d));
    const bool up = d > 0.0f;                                 // the same as x > mx
    acc = up ? fmaf(acc, e, 1.0f) : acc + e;
    mx = bigger(x, mx);
}

// the same for the first element of a row (acc = 0, mx = -inf before)
template <int VEC>
__device__ __forceinline__ void lse_first(float (&acc)[VEC], float (&mx)[VEC], const float (&x)[VEC]) {
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
        mx[v] = bigger(x[v], -INFINITY);      // (NaN: an impossible child)
        acc[v] = 1.0f;
    }
}

// nc: the value of the output row itself where the operation needs it; OP_LSE2 / OP_MAX2 keep the sum of the
// group in hand there (weighted = the entry closes its group).  y: OP_SOFTMAX_BWD the parent's value, the P row ops share_scale(nc), or 1
// (a single entry, or a sum that is then looked at).
template <int OP>
__device__ __forceinline__ void accumulate(float& acc, float& mx, float x, float y, float& nc, bool weighted = true) {
    if (OP == OP_SUM_H || OP == OP_SUM_P) { acc += x; return; }
    if (OP == OP_SOFTMAX_H) { acc += weighted ? decode_h(x, nc) : x; return; }
    if (OP == OP_SUMPROD2) {
        nc *= x;
        if (weighted) { acc += nc; nc = 1.0f; }
        return;
    }
    if (OP == OP_LSE2 || OP == OP_MAX2) {
        nc += x;
        if (weighted) {
            if (OP == OP_LSE2) lse_step(acc, mx, nc);
            else acc = nc > acc ? nc : acc;
            nc = 0.0f;
        }
        return;
    }
    if (OpTraits<OP>::shares) {
        const uint32_t bits = __float_as_uint(x);
        const bool mine = !weighted && ((bits & 1u) != 0) == (nc == 0.0f);
        mx = fmaf(mine ? __uint_as_float(bits & ~1u) : -0.0f, y, mx);
        acc += weighted ? x : 0.0f;
        return;
    }
    if (OP == OP_SUM) acc += x;
    else if (OP == OP_PROD) acc *= x;
    else if (OP == OP_MAX) acc = x > acc ? x : acc;               // (acc is no NaN: two instructions, fmaxf takes three)
    else if (OP == OP_LSE) lse_step(acc, mx, x);
    else {
        const float wgt = !weighted ? 1.0f : ((y == -INFINITY) ? 0.0f : fexp(nc - y));
        acc = fmaf(x, wgt, acc);
    }
}

template <int OP>
__device__ __forceinline__ float finish(float acc, float mx, float nc = 0.0f, float scale = 1.0f) {
    // (no entry that concerns the row: no quotient, which a NaN value would make one)
    if (OpTraits<OP>::shares) return acc + (nc != 0.0f && __float_as_uint(mx) != 0x80000000u ? mx / (nc * scale) : mx);
    if (OP == OP_LSE || OP == OP_LSE2) return (mx == -INFINITY) ? -INFINITY : mx + flog(acc);
    return acc;
}

// the second part of a row's state before its first entry
template <int OP>
__device__ __forceinline__ float identity2() { return OpTraits<OP>::shares ? -0.0f : -INFINITY; }

template <int OP>
__device__ __forceinline__ float identity() { return OP == OP_PROD ? 1.0f : ((OP == OP_MAX || OP == OP_MAX2) ? -INFINITY : 0.0f); }

// what an index entry that is not part of the row contributes: nothing
template <int OP>
__device__ __forceinline__ float dead_value() {
    return (OP == OP_PROD || OP == OP_SUMPROD2) ? 1.0f : ((OP == OP_LSE || OP == OP_MAX) ? -INFINITY : 0.0f);
}

// ---------------------------------------------------------------------------------------------
// Streaming segmented gather-reduce for B > 64 (one wave spans the batch tile, VEC = 2 or 4 columns per
// lane).  A task is a run of consecutive output rows with a bounded number of edges, fixed at
// build time (stream_tasks); the wave walks the task's edges in chunks of CH, closes an output row whenever
// an entry carries the end-of-row bit, and has the gathers of the next chunk on their way while it works on one, the entries of
// the one after that, too; the first ones come with the task.  Everything that steers control flow is wave-uniform and branches; entries past the task's end
// are valid entries of later rows (or zero padding) that nothing is done with.
//   What bounds it: where the children fit the caches, the scalar unit (one instruction a cycle for the whole compute unit; 26 of them an
// entry with addresses summed per lane, skip entries and every entry tested against the task's end, now 11) and the vector instructions
// of a logsumexp (a row's first element takes two instead of ten a column); where they do not, what misses the L2.  With one
// chunk in flight, all of it waited for / as it is, us a pass: 811k nodes forward B = 256 368 / 334, (max, +) B = 100 246 / 188, real
// training step B = 256 1185 / 1149; 3e6 nodes, training step B = 256 3656 / 3500.  (The P row ops wait for each chunk: with two of them in
// flight, a value of the output row beside every entry, they take 145 registers a lane at four columns, three waves a SIMD, with one 68, seven: 298 -> 313
// us of that real step.)
// MAPPED: the main rows are not numbered through; entry_row says which one an entry belongs to (compact_pass).  For the AND layers without their
// fused rows; left in as a skip entry a row, these were most of what the walk read (seven layers of 811k nodes, three of four AND rows
// fused, us: four columns a lane, B = 256 87 -> 77, which is the rate of what is left; two, B = 100 64 -> 55).
// ---------------------------------------------------------------------------------------------
// index vectors that a wave reads as a whole, with scalar loads (nothing writes them while a kernel runs)
template <class T> using Scalars = const __attribute__((address_space(4))) T*;
template <class T>
__device__ __forceinline__ Scalars<T> scalars(const T* p) { return (Scalars<T>)p; }

struct StreamArgs {
    const int32_t *tasks, *seg_tasks;   // main rows; segments of split rows (see stream_tasks)
    const uint32_t* idx;
    const int32_t* entry_row;           // MAPPED
    const float *src, *src2, *own;      // as PassArgs
    float *dst, *dst_seg;               // dst_seg: the scratch rows shifted by -n_main rows
    const int32_t* seg_owner;
    int* zero_flag;
    int32_t n_tasks, n_seg_tasks, B, ld, stream_stores, n_main;
};

template <int OP, int VEC, bool MAPPED>
__global__ __launch_bounds__(256) void stream_kernel(StreamArgs a) {
    constexpr bool OWN = OpTraits<OP>::own, TWO = OP == OP_SOFTMAX_BWD;
    constexpr int CH = TWO ? 2 : kStreamChunk;         // entries per chunk
    static_assert(CH <= kStreamChunk && kStreamChunk - 1 + 2 * kStreamChunk <= kIdxPad, "what is read past a task's end (stream_reads)");
    constexpr bool PIPE = !OpTraits<OP>::shares;
    static_assert(kGroupEnd == kWeighted, "the fused plans reuse this bit");
    static_assert(!(MAPPED && OWN), "the value of a row is looked up by its number");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = ((int)blockIdx.y * 64 + lane) * VEC;
    if (col >= a.B) return;
    int t = xcd_block((int)blockIdx.x, (int)gridDim.x) * 4 + wave;
    if (t >= a.n_tasks + a.n_seg_tasks) return;
    // tasks past the main list are segments of split rows: same walk, output rows go to scratch
    const bool seg = t >= a.n_tasks;
    if (seg) t -= a.n_tasks;
    const Scalars<int32_t> task = scalars((seg ? a.seg_tasks : a.tasks) + kTaskWords * (size_t)t);
    const int2 t0 = make_int2(task[0], task[1]), t1 = make_int2(task[2], task[3]);
    const Scalars<uint32_t> idx = scalars(a.idx + t0.y);
    const Scalars<int32_t> row_of = scalars(MAPPED ? static_cast<const int32_t*>(task_entry_rows(a.idx, a.entry_row, t0.y, seg)) : nullptr);
    const Scalars<int32_t> owner = scalars(a.seg_owner);
    int left = t1.y - t0.y;                 // entries
    const uint32_t row_bytes = (uint32_t)a.ld * 4u;
    uint32_t lane_bytes = (uint32_t)col * 4u;
    float* const dst = seg ? a.dst_seg : a.dst;
    const bool nt = !seg && a.stream_stores != 0;
    // One address for the wave and an offset of the lane's own: scalar work in place of 64-bit sums in vector registers.  (The first
    // statement keeps the compiler from adding base and lane first, the second from widening the offset once, after which it no longer sees
    // that 32 bits are enough.)
    auto at = [&](const float* rows, uint32_t row) {
        uint64_t p = reinterpret_cast<uint64_t>(rows) + (uint64_t)row * row_bytes;
        asm("" : "+s"(p));
        asm volatile("" : "+v"(lane_bytes));
        return (float*)(reinterpret_cast<__attribute__((address_space(1))) char*>(p) + lane_bytes);
    };

    struct Ids {
        uint32_t id[CH];
        int to[MAPPED ? CH : 1];
    };
    struct Chunk {
        float x[CH][VEC], y[TWO ? CH : 1][VEC], z[OWN ? CH : 1][VEC];
    };
    int row = t0.x, row_ahead = t0.x;       // the next row to finish; the row of the next entry to gather
    auto load_ids = [&](int j) {            // (readable past the end)
        Ids r;
#pragma unroll
        for (int i = 0; i < CH; ++i) r.id[i] = idx[j + i];
        if constexpr (MAPPED)
#pragma unroll
            for (int i = 0; i < CH; ++i) r.to[i] = row_of[j + i];
        return r;
    };
    auto gather_one = [&](Chunk& c, int i, uint32_t id, uint32_t own_id) {
        load_vec<VEC>(c.x[i], at(a.src, id & kIdMask));
        // an unweighted edge needs no parent value: re-read the row just requested (an L1 hit)
        if constexpr (TWO) load_vec<VEC>(c.y[i], at((id & kWeighted) ? a.src2 : a.src, id & kIdMask));
        if constexpr (OWN) {
            // (a segment of a split row works with the value of the row that owns it, if with any)
            int own_row = row_ahead < t1.x ? row_ahead : t1.x - 1;
            if (seg) own_row = OpTraits<OP>::seg_own ? owner[own_row - a.n_main] : 0;
            load_vec<VEC>(c.z[i], at(a.own, (uint32_t)own_row));
            row_ahead += (int)(own_id >> 31);
        }
    };
    // n entries are the task's; in place of those past it the chunk's first row again
    auto gather = [&](Chunk& c, const Ids& ids, int n) {
#pragma unroll
        for (int i = 0; i < CH; ++i) gather_one(c, i, i == 0 || i < n ? ids.id[i] : ids.id[0], ids.id[i]);
    };

    float acc[VEC], mx[VEC], nc[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) { acc[v] = identity<OP>(); mx[v] = identity2<OP>(); nc[v] = OP == OP_SUMPROD2 ? 1.0f : 0.0f; }
    bool beyond = false;                     // P row ops: a sum of P rows is not finite
    bool fresh = true;                       // the row in hand has nothing yet
    auto consume = [&](const Chunk& c, const Ids& ids, int n, auto whole) {
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            if (!decltype(whole)::value && i >= n) break;
            const uint32_t id = ids.id[i];
            const bool weighted = (id & kWeighted) != 0;
            if constexpr (OP == OP_LSE) {
                if (fresh) lse_first<VEC>(acc, mx, c.x[i]);
                else
#pragma unroll
                    for (int v = 0; v < VEC; ++v) lse_step(acc[v], mx[v], c.x[i][v]);
                fresh = false;
            } else if constexpr (OP == OP_LSE2 || OP == OP_MAX2 || OP == OP_SUMPROD2) {
#pragma unroll
                for (int v = 0; v < VEC; ++v) nc[v] = OP == OP_SUMPROD2 ? nc[v] * c.x[i][v] : nc[v] + c.x[i][v];
                if (weighted) {
                    if constexpr (OP == OP_LSE2) {
                        if (fresh) lse_first<VEC>(acc, mx, nc);
                        else
#pragma unroll
                            for (int v = 0; v < VEC; ++v) lse_step(acc[v], mx[v], nc[v]);
                        fresh = false;
                    }
#pragma unroll
                    for (int v = 0; v < VEC; ++v) {
                        if (OP == OP_MAX2) acc[v] = bigger(nc[v], acc[v]);
                        if (OP == OP_SUMPROD2) acc[v] += nc[v];
                        nc[v] = OP == OP_SUMPROD2 ? 1.0f : 0.0f;
                    }
                }
            } else {
                if constexpr (OWN) {
                    if (fresh)
#pragma unroll
                        for (int v = 0; v < VEC; ++v) nc[v] = c.z[i][v];
                    fresh = false;
                }
#pragma unroll
                for (int v = 0; v < VEC; ++v) accumulate<OP>(acc[v], mx[v], c.x[i][v], TWO ? c.y[i][v] : 1.0f, nc[v], weighted);
            }
            if (id & kLast) {
                float o[VEC];
#pragma unroll
                for (int v = 0; v < VEC; ++v) {
                    if (OpTraits<OP>::shares) beyond |= !(fabsf(mx[v]) < INFINITY);
                    // (logsumexp: the sum is at least 1 here, see lse_first, so that a row of impossible children needs no test)
                    o[v] = OP == OP_LSE || OP == OP_LSE2 ? mx[v] + flog(acc[v]) : finish<OP>(acc[v], mx[v], nc[v]);
                    // the adjoint of an OR node with more than one child leaves in the one-gather form
                    if (OP == OP_SUM_H && !seg && (id & kRowFlag)) o[v] = encode_h(o[v], nc[v]);
                    if (OpTraits<OP>::premul && !seg) {
                        if (nc[v] == 0.0f && a.zero_flag) *a.zero_flag = 1;          // this layer needs prod_parent_kernel's repair
                        o[v] = premultiply(o[v], nc[v]);
                    }
                    if (OP != OP_LSE && OP != OP_LSE2) { acc[v] = identity<OP>(); mx[v] = identity2<OP>(); }
                }
                const int out = MAPPED && !seg ? ids.to[i] : row;
                float* to = at(dst, (uint32_t)out);
                if (nt) store_vec_stream<VEC>(to, o);
                else store_vec<VEC>(to, o);
                ++row;
                fresh = true;
            }
        }
    };
    int j = 0;
    Ids i0, i1;                             // (with the task itself: one read less before the first gather)
    static_assert(kTaskHead + 2 * CH <= kTaskWords, "two chunks");
#pragma unroll
    for (int i = 0; i < CH; ++i) { i0.id[i] = (uint32_t)task[kTaskHead + i]; i1.id[i] = (uint32_t)task[kTaskHead + CH + i]; }
    if constexpr (MAPPED)
#pragma unroll
        for (int i = 0; i < CH; ++i) { i0.to[i] = row_of[i]; i1.to[i] = row_of[CH + i]; }
    if constexpr (PIPE) {
        Chunk c0, c1;
        gather(c0, i0, left);
        for (;;) {
            const Ids i2 = load_ids(j + 2 * CH);
            if (left <= CH) { consume(c0, i0, left, std::false_type()); break; }
            gather(c1, i1, left - CH);
            consume(c0, i0, CH, std::true_type());
            left -= CH;
            const Ids i3 = load_ids(j + 3 * CH);
            if (left <= CH) { consume(c1, i1, left, std::false_type()); break; }
            gather(c0, i2, left - CH);
            consume(c1, i1, CH, std::true_type());
            left -= CH;
            j += 2 * CH;
            i0 = i2;
            i1 = i3;
        }
    } else {
        Chunk c;
        for (;;) {
            gather(c, i0, left);
            const Ids i2 = load_ids(j + 2 * CH);
            // s_waitcnt vmcnt(0) (scalar prefetch left in flight): the gathers are complete on every
            // path from here on, so no later register reuse has to wait on them again.
            __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
            if (left <= CH) { consume(c, i0, left, std::false_type()); break; }
            consume(c, i0, CH, std::true_type());
            i0 = i1;
            i1 = i2;
            left -= CH;
            j += CH;
        }
    }
    if (!OpTraits<OP>::shares || !__any(beyond)) return;
    // A sum of P rows left the range (or is NaN, as one that did and met an infinite row): the task's rows once more, every P row scaled before it is added.  (Rare; scaling always costs 7 to
    // 10% where layers are narrow: 16000 nodes in 40 layers at B = 256, training step 373 us / 401.)
    row = t0.x;
    fresh = true;
    for (int k = 0; k < t1.y - t0.y; ++k) {
        const uint32_t id = idx[k];
        const bool last = (id & kLast) != 0;
        {
            if (fresh) {
                load_vec<VEC>(nc, at(a.own, (uint32_t)(seg ? owner[row - a.n_main] : row)));
#pragma unroll
                for (int v = 0; v < VEC; ++v) { acc[v] = identity<OP>(); mx[v] = identity2<OP>(); }
            }
            float x[VEC];
            load_vec<VEC>(x, at(a.src, id & kIdMask));
#pragma unroll
            for (int v = 0; v < VEC; ++v) accumulate<OP>(acc[v], mx[v], x[v], share_scale(nc[v]), nc[v], (id & kWeighted) != 0);
            if (last) {
                float o[VEC];
#pragma unroll
                for (int v = 0; v < VEC; ++v) {
                    o[v] = finish<OP>(acc[v], mx[v], nc[v], share_scale(nc[v]));
                    if (OpTraits<OP>::premul && !seg) o[v] = premultiply(o[v], nc[v]);
                }
                store_vec<VEC>(at(dst, (uint32_t)row), o);
            }
        }
        fresh = last;
        row += last ? 1 : 0;
    }
}

// ---------------------------------------------------------------------------------------------
// Small batches (B <= 32): lanes = edges.  A lane group of LPR lanes (B rounded up to a power of two)
// holds one index entry, its lanes the batch columns, so a wave takes EPW = 64 / LPR consecutive entries
// per step (all 64 at B = 1): one coalesced read of the entries, one gather of their rows, and the
// entries of an output row, which sit in neighbouring lane groups, are reduced across the wave:
//   - a step in which no row ends only accumulates, every lane group into a partial of its own;
//   - a step in which rows end folds those partials into one (butterfly over the lane groups), adds
//     it to the first lane group, and runs a segmented inclusive scan over the lane groups (wave
//     shuffles; a lane knows its segment's start from the ballot of the end-of-row bits, so only values
//     travel); the lane groups that hold a row's last entry store the row, the part of a row that is
//     still open stays behind as the last lane group's partial.
// Same index entries as the streaming kernel, task lists of its own (PassPlan::tasks; a wave takes `span` consecutive ones);
// tasks past the main list are the segments of split rows.  The log-domain OR reduction travels as
// (maximum, sum of exp(x - maximum)) pairs.
// ---------------------------------------------------------------------------------------------
template <int OP>
__device__ __forceinline__ void edge_combine(float& am, float& as, float bm, float bs) {
    if (OpTraits<OP>::additive) am += bm;
    else if (OP == OP_PROD) am *= bm;
    else if (OP == OP_MAX) am = fmaxf(am, bm);
    else {
        const float M = fmaxf(am, bm), m = finite(M);
        as = as * term_exp(am - m) + bs * term_exp(bm - m);
        am = M;
    }
}

template <int OP, int LPR>
__global__ __launch_bounds__(256) void edge_kernel(const int2* __restrict__ tasks, int n_tasks, int span,
                                                   const uint32_t* __restrict__ idx, const float* __restrict__ src,
                                                   const float* __restrict__ src2, const float* __restrict__ own,
                                                   float* __restrict__ dst, int B, int ld,
                                                   const int2* __restrict__ seg_tasks, int n_seg_tasks,
                                                   const int32_t* __restrict__ seg_owner, int n_main,
                                                   float* __restrict__ dst_seg, int* __restrict__ zero_flag) {
    constexpr int EPW = 64 / LPR;                 // entries per step
    constexpr int CH = EPW >= 16 ? 4 : 8;         // steps whose gathers are in flight together
    constexpr bool LSE = OP == OP_LSE;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int sub = lane / LPR, c = lane % LPR;
    const bool active = c < B;
    const int cc = active ? c : B - 1;            // lanes past the batch re-read its last column and store nothing
    const int n_main_waves = (n_tasks + span - 1) / span;
    int wt = (int)blockIdx.x * 4 + wave;
    bool seg = false;
    if (wt >= n_main_waves) {
        wt -= n_main_waves;
        seg = true;
        tasks = seg_tasks;
        n_tasks = n_seg_tasks;
        dst = dst_seg;
    }
    const int t0 = wt * span;
    if (t0 >= n_tasks) return;
    const int t1 = t0 + span < n_tasks ? t0 + span : n_tasks;
    const int2 ta = tasks[t0], tb = tasks[t1];
    int row = ta.x;
    const int e1 = tb.y;
    float accm = identity<OP>(), accs = 0.0f;     // this lane group's partial of the open row
    if (LSE) accm = -INFINITY;
    int state = 0;     // partials: 0 none holds anything, 1 only the last lane group's does, 2 any may
    for (int j = ta.y; j < e1; j += CH * EPW) {
        uint32_t id[CH];
        bool in[CH];
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int pos = j + i * EPW + sub;
            in[i] = pos < e1;
            id[i] = idx[in[i] ? pos : e1 - 1];
        }
        // rows of the entries: the open row plus the rows that end before them
        unsigned long long lm[CH], below[CH];
        int rowidx[CH];
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const bool last = in[i] && (id[i] & kLast) != 0;
            lm[i] = __builtin_amdgcn_ballot_w64(last && c == 0);
            below[i] = lm[i] & ((1ull << (sub * LPR)) - 1ull);
            rowidx[i] = row + __builtin_popcountll(below[i]);
            row += __builtin_popcountll(lm[i]);
        }
        float x[CH], y[CH], z[CH];
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const bool live = in[i] && id[i] != kSkip;
            const size_t off = (size_t)(live ? (id[i] & kIdMask) : 0u) * (size_t)ld + cc;
            x[i] = src[off];
            y[i] = 0.0f;
            z[i] = 0.0f;
            if (OpTraits<OP>::own) {
                const bool weighted = live && (id[i] & kWeighted) != 0;
                // value of the parent, and of the row the entry belongs to (a segment: of its owner)
                if (OP == OP_SOFTMAX_BWD) y[i] = (weighted ? src2 : src)[off];
                int orow = live ? rowidx[i] : (seg ? n_main : 0);      // an entry past the task's end has no row
                if (seg) orow = seg_owner[orow - n_main];
                z[i] = own[(size_t)orow * (size_t)ld + cc];
            }
        }
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const bool live = in[i] && id[i] != kSkip;
            const bool last = in[i] && (id[i] & kLast) != 0;
            float vm, vs = 0.0f;
            if (OP == OP_SOFTMAX_BWD) {
                const bool weighted = live && (id[i] & kWeighted) != 0;
                const float wgt = !weighted ? 1.0f : ((y[i] == -INFINITY) ? 0.0f : fexp(z[i] - y[i]));
                vm = live ? x[i] * wgt : 0.0f;
            } else if (OP == OP_SOFTMAX_H) {
                vm = live ? ((id[i] & kWeighted) ? decode_h(x[i], z[i]) : x[i]) : 0.0f;
            } else if (OpTraits<OP>::shares) {
                float plain = 0.0f, shared = identity2<OP>();
                accumulate<OP>(plain, shared, x[i], 1.0f, z[i], (id[i] & kWeighted) != 0);
                vm = live ? finish<OP>(plain, shared, z[i]) : 0.0f;
            } else if (LSE) {
                vm = live ? fmaxf(x[i], -INFINITY) : -INFINITY;
                vs = live ? 1.0f : 0.0f;
            } else {
                vm = live ? (OP == OP_MAX ? fmaxf(x[i], -INFINITY) : x[i]) : dead_value<OP>();
            }
            if (lm[i] == 0ull) {                      // no row ends in this step
                edge_combine<OP>(accm, accs, vm, vs);
                state = 2;
                continue;
            }
            if (state == 2) {                         // fold the partials of all lane groups
#pragma unroll
                for (int d = LPR; d < 64; d <<= 1) {
                    const float om = __shfl_xor(accm, d), os = LSE ? __shfl_xor(accs, d) : 0.0f;
                    edge_combine<OP>(accm, accs, om, os);
                }
            } else if (state == 1) {                  // only the last lane group holds one
                accm = __shfl(accm, (EPW - 1) * LPR + c);
                if (LSE) accs = __shfl(accs, (EPW - 1) * LPR + c);
            }
            if (sub == 0) edge_combine<OP>(vm, vs, accm, accs);
            // segmented inclusive scan over the lane groups: a segment starts after every end of row
            const int start = below[i] ? (63 - __builtin_clzll(below[i])) / LPR + 1 : 0;
            const int dist = sub - start;
#pragma unroll
            for (int d = 1; d < EPW; d <<= 1) {
                const float om = __shfl_up(vm, d * LPR), os = LSE ? __shfl_up(vs, d * LPR) : 0.0f;
                if (dist >= d) edge_combine<OP>(vm, vs, om, os);
            }
            if (last && live && active) {
                float o = vm;
                if (LSE) o = (vm == -INFINITY) ? -INFINITY : vm + flog(vs);
                if (OP == OP_SUM_H && !seg && (id[i] & kRowFlag)) o = encode_h(o, z[i]);
                if (OpTraits<OP>::premul && !seg) {
                    if (z[i] == 0.0f && zero_flag) *zero_flag = 1;
                    o = premultiply(o, z[i]);
                }
                dst[(size_t)rowidx[i] * (size_t)ld + c] = o;
            }
            // the open row's part stays with the last lane group
            const bool tail_last = ((lm[i] >> ((EPW - 1) * LPR)) & 1ull) != 0ull;
            const bool keep = sub == EPW - 1 && !tail_last;
            accm = keep ? vm : (LSE ? -INFINITY : identity<OP>());
            accs = keep ? vs : 0.0f;
            state = tail_last ? 0 : 1;
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Generic gather-reduce: a group of a.lanes lanes owns one output row, VEC batch columns per lane,
// so a wave takes 64 / lanes rows (any number of lanes: 21 rows at B = 10 with four columns a lane, 4 at B = 64).  Also evaluates the segments of split rows (rows >= n_main, written
// to scratch rows) and the combine pass (out_row map).
//   What bounds it is the number of vector memory instructions: a compute unit takes 16 cycles for each, whatever it
// fetches, and the rows of a small batch are short.  Hence four columns per lane also where that leaves rows unaligned
// (the loads need four bytes) or the batch is no multiple of four (the last lane steps back and shares columns with its
// neighbour, computing the same values), the offsets of a row in one load, its entries four at a time, and
// the second four gathers only where a row of the wave has more than four entries.  (800000 nodes at B = 10, free
// literals, training step: 381 -> 280 us; power-law fan-ins, 1e7 edges at B = 64: 515 -> 457 us.  One column per lane and
// eight gathers for every row before.)  A launch of few rows takes fewer columns per lane (launch_pass).
// ---------------------------------------------------------------------------------------------
template <int VEC>
__device__ __forceinline__ void load_cols(float (&x)[VEC], const float* p) {
    typedef float vf __attribute__((ext_vector_type(VEC), aligned(4)));
    const vf t = *reinterpret_cast<const vf*>(p);
#pragma unroll
    for (int v = 0; v < VEC; ++v) x[v] = t[v];
}
template <>
__device__ __forceinline__ void load_cols<1>(float (&x)[1], const float* p) { x[0] = *p; }
template <int VEC>
__device__ __forceinline__ void store_cols(float* p, const float (&x)[VEC]) {
    typedef float vf __attribute__((ext_vector_type(VEC), aligned(4)));
    vf t;
#pragma unroll
    for (int v = 0; v < VEC; ++v) t[v] = x[v];
    *reinterpret_cast<vf*>(p) = t;
}
template <>
__device__ __forceinline__ void store_cols<1>(float* p, const float (&x)[1]) { *p = x[0]; }

// Which row of the wave a lane works for and its first column; false: none.  inverse = ceil(65536 / lanes), so that the
// product below is lane / lanes for every lane of a wave.
template <class Args>
__device__ __forceinline__ bool lane_group(const Args& a, int vec, int& sub, int& col) {
    const uint32_t lane = threadIdx.x & 63;
    sub = (int)(lane * a.inverse >> 16);
    col = ((int)blockIdx.y * a.lanes + (int)lane - sub * a.lanes) * vec;
    return sub < a.per_wave && col < a.B;
}

typedef uint32_t Entries4 __attribute__((ext_vector_type(4), aligned(4)));
typedef int32_t Offsets2 __attribute__((ext_vector_type(2), aligned(4)));

// four entries of a row joined to its state; `live` of them are part of the row
template <int OP, int VEC>
__device__ __forceinline__ void accumulate4(float (&acc)[VEC], float (&mx)[VEC], const float (&x)[4][VEC], const float (&y)[4][VEC],
                                            float (&nc)[VEC], Entries4 e, int live) {
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
        if (OP == OP_LSE) {
            // (one maximum for the four, no test for -inf: see the persistent kernels)
            const float x0 = live > 0 ? x[0][v] : -INFINITY, x1 = live > 1 ? x[1][v] : -INFINITY;
            const float x2 = live > 2 ? x[2][v] : -INFINITY, x3 = live > 3 ? x[3][v] : -INFINITY;
            const float hi = max3(max3(x0, x1, x2), x3, mx[v]), m = finite(hi);
            acc[v] = fmaf(acc[v], term_exp(mx[v] - m), (term_exp(x0 - m) + term_exp(x1 - m)) + (term_exp(x2 - m) + term_exp(x3 - m)));
            mx[v] = hi;
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float xv = i < live ? x[i][v] : dead_value<OP>();
                const float yv = OP == OP_SOFTMAX_BWD ? (i < live ? y[i][v] : -INFINITY) : 1.0f;
                accumulate<OP>(acc[v], mx[v], xv, yv, nc[v], OpTraits<OP>::shares ? i >= live || (e[i] & kWeighted) != 0 : i < live && (e[i] & kWeighted) != 0);
            }
        }
    }
}

// Logsumexp of many terms: the state of a row is (mx, acc) = (maximum so far, sum of 2^(x log2(e) - lse_scale(mx))), one fused
// multiply-add and one exponential per term.  lse_scale is a float at or just above mx log2(e), so that no term leaves [0, 1];
// by how much, lse_value takes off again.  Beyond kLseFlat, where an ulp of mx is 16, a row is its maximum (the logarithm of fewer
// than kLseFlatTerms = e^8 terms rounds away; a segment has 24 unless a longer minimum is asked for); that leaves out infinite maxima as well, whose scale is no number.
constexpr float kLseFlat = 134217728.0f, kLseUp = 2.384185791015625e-7f;
constexpr int32_t kLseFlatTerms = 2980;
__device__ __forceinline__ float lse_scale(float m) {
    float p = m * kLog2e;
    asm("" : "+v"(p));                                 // (a product of its own: one that is fused into a later sum is another number)
    return fmaf(fabsf(m), kLseUp, p);
}
__device__ __forceinline__ float unit_exp2(float x) { return __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(x), 0.0f, 1.0f); }
__device__ __forceinline__ float lse_term(float x, float scale) { return unit_exp2(fmaf(x, kLog2e, -scale)); }
__device__ __forceinline__ float lse_value(float acc, float mx) {
    const float over = fmaf(mx, kLog2e, -lse_scale(mx));
    return fabsf(mx) > kLseFlat ? mx : fmaf(__builtin_amdgcn_logf(acc) - over, kLn2, mx);
}

// N terms of every column joined to the state of its row: all of them (FULL), or the first `live`.  first: nothing came before.
template <int VEC, int N, bool FULL>
__device__ __forceinline__ void lse_join(float (&acc)[VEC], float (&mx)[VEC], const float (&x)[N][VEC], int live, bool first) {
    float sum[VEC], scale[VEC], hi[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
        float t[N];
#pragma unroll
        for (int i = 0; i < N; ++i) t[i] = FULL || i < live ? x[i][v] : -INFINITY;
        hi[v] = mx[v];
#pragma unroll
        for (int i = 0; i < N; i += 2) hi[v] = max3(t[i], t[i + 1], hi[v]);
        scale[v] = lse_scale(hi[v]);
#pragma unroll
        for (int i = 0; i < N; ++i) t[i] = lse_term(t[i], scale[v]);
#pragma unroll
        for (int d = 1; d < N; d *= 2)
#pragma unroll
            for (int i = 0; i < N; i += 2 * d) t[i] += t[i + d];
        sum[v] = t[0];
    }
    if (!first)
#pragma unroll
        for (int v = 0; v < VEC; ++v) sum[v] = fmaf(acc[v], unit_exp2(lse_scale(mx[v]) - scale[v]), sum[v]);
#pragma unroll
    for (int v = 0; v < VEC; ++v) { acc[v] = sum[v]; mx[v] = hi[v]; }
}

// All arguments in one go: left to the compiler their reads sit behind the branches before their first use, one line after
// another, and a launch of few rows is a chain of such reads (with the entries, see below, us: 2800 nodes max B = 5, 39
// launches, 121 -> 116; 800000 nodes B = 1 108 -> 105, training B = 10 289 -> 281).
__device__ __forceinline__ void arguments_now(const PassArgs& a) {
    asm volatile("" ::"s"(a.ptr), "s"(a.idx), "s"(a.src), "s"(a.own), "s"(a.seg_owner), "s"(a.out_row), "s"(a.dst), "s"(a.dst_seg),
                 "s"(a.per_wave), "s"(a.row_begin), "s"(a.n_main), "s"(a.n_total), "s"(a.B), "s"(a.ld), "s"(gridDim.x));
}

// bx of nbx: the workgroup's place among those that take rows (nbx a multiple of 8, bx mod 8 the XCD the workgroup runs on)
// LONG: the segments of split logsumexp rows, 24 entries for the most part, in a launch of their own.  They run from the caches, and what
// bounds them is the vector unit: per entry and column a select, a share of two maxima per four, a subtraction, a product, an exponential
// (four instructions' time), a sum, and per four entries a rescaling of what came before.  Eight entries a step, without the selects,
// without a rescaling before the first step, one fused multiply-add in front of the exponential: 24 entries take about 177 instructions a
// column instead of 250.  Power-law fan-ins, 1e7 edges, B = 64, the six launches, us: 45.1 30.2 22.0 16.0 10.7 9.1 -> 37.2 26.1 19.4 13.7 9.7
// 8.1; whole pass 376 -> 361.  (Not for the main rows beside combine rows, most of which are shorter: 58.4 -> 58.2, 14.2 -> 13.6, 17.0 -> 17.7 in
// two circuits; nor, without its logsumexp, for the other ops: 62 -> 62 for the longest launch of sums.)
template <int OP, int VEC, bool LONG>
__device__ __forceinline__ void pass_body(int bx, int nbx, const PassArgs& a) {
    constexpr bool OWN = OpTraits<OP>::own;
    int sub, colu;
    if (!lane_group(a, VEC, sub, colu)) return;
    const int col = colu <= a.B - VEC ? colu : a.B - VEC;
    const int64_t row64 = ((int64_t)xcd_block(bx, nbx) * 4 + (threadIdx.x >> 6)) * a.per_wave + sub + a.row_begin;
    if (row64 >= a.n_total) return;
    const int row = (int)row64;
    const Offsets2 range = *reinterpret_cast<const Offsets2*>(a.ptr + row);
    const int end = range.y;
    int j = range.x;
    // (entries past the row's end are entries of later rows or zero padding: they can be followed, their data is ignored)
    Entries4 e0 = *reinterpret_cast<const Entries4*>(a.idx + j), e1 = *reinterpret_cast<const Entries4*>(a.idx + j + 4);
    asm volatile("" ::"v"(e0.x), "v"(e1.x));           // (both now: the second load would move behind the return)
    if (e0.x == kSkip) return;                        // split row: evaluated by segments + combine
    float nc[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) nc[v] = 0.0f;
    if (OWN) {
        // the row whose value this output belongs to: itself, the row a combine pass writes, or a segment's owner
        const int owner = row < a.n_main ? (a.out_row ? a.out_row[row] : row) : a.seg_owner[row - a.n_main];
        load_cols<VEC>(nc, a.own + (size_t)owner * a.ld + col);
    }
    float acc[VEC], mx[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) { acc[v] = identity<OP>(); mx[v] = identity2<OP>(); }
    uint32_t last = 0;
    if constexpr (LONG) {
        static_assert(OP == OP_LSE, "the other ops gain nothing");
        bool first = true;
        auto gather = [&](uint32_t e, float (&to)[VEC]) { load_cols<VEC>(to, a.src + (size_t)(e & kIdMask) * a.ld + col); };
        // as long as every row of the wave has eight entries left: nothing to test per entry
        while (__all(j + 8 <= end)) {
            float x[8][VEC];
#pragma unroll
            for (int i = 0; i < 8; ++i) gather(i < 4 ? e0[i] : e1[i - 4], x[i]);
            j += 8;
            e0 = *reinterpret_cast<const Entries4*>(a.idx + j);
            e1 = *reinterpret_cast<const Entries4*>(a.idx + j + 4);
            lse_join<VEC, 8, true>(acc, mx, x, 8, first);
            first = false;
        }
        while (__any(j < end)) {
            float x0[4][VEC], x1[4][VEC];
            const bool second = __any(j + 4 < end), more = __any(j + 8 < end);
#pragma unroll
            for (int i = 0; i < 4; ++i) gather(j + i < end ? e0[i] : 0u, x0[i]);
            if (second)
#pragma unroll
                for (int i = 0; i < 4; ++i) gather(j + 4 + i < end ? e1[i] : 0u, x1[i]);
            if (more) {
                const int at = j + 8 < end ? j + 8 : range.x;    // (a row that has ended reads its first entries again)
                e0 = *reinterpret_cast<const Entries4*>(a.idx + at);
                e1 = *reinterpret_cast<const Entries4*>(a.idx + at + 4);
            }
            if (j < end) lse_join<VEC, 4, false>(acc, mx, x0, end - j, first);
            if (second && j + 4 < end) lse_join<VEC, 4, false>(acc, mx, x1, end - j - 4, false);
            j += 8;
            first = false;
        }
    } else
    for (;;) {
        float x0[4][VEC], x1[4][VEC], y0[4][VEC], y1[4][VEC];
        auto gather = [&](Entries4 e, float (&x)[4][VEC], float (&y)[4][VEC]) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const size_t off = (size_t)(e[i] == kSkip ? 0u : e[i] & kIdMask) * a.ld + col;
                load_cols<VEC>(x[i], a.src + off);
                if (OP == OP_SOFTMAX_BWD) load_cols<VEC>(y[i], ((e[i] & kWeighted) ? a.src2 : a.src) + off);
            }
        };
        const bool second = __any(j + 4 < end), more = __any(j + 8 < end);
        Entries4 n0 = e0, n1 = e1;
        gather(e0, x0, y0);
        if (second) gather(e1, x1, y1);
        if (more) {
            const int at = j + 8 < end ? j + 8 : range.x;        // (a row that has ended reads its first entries again)
            n0 = *reinterpret_cast<const Entries4*>(a.idx + at);
            n1 = *reinterpret_cast<const Entries4*>(a.idx + at + 4);
        }
        if (j < end) accumulate4<OP, VEC>(acc, mx, x0, y0, nc, e0, end - j);
        if (second && j + 4 < end) accumulate4<OP, VEC>(acc, mx, x1, y1, nc, e1, end - j - 4);
        if (j < end && OP == OP_SUM_H) {
            const int at = end - j - 1;               // the row's last entry carries its flag
            if (at < 8) {
                const Entries4 e = at < 4 ? e0 : e1;
                last = (at & 3) == 0 ? e.x : (at & 3) == 1 ? e.y : (at & 3) == 2 ? e.z : e.w;
            }
        }
        j += 8;
        if (!more) break;
        e0 = n0;
        e1 = n1;
    }
    float o[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) o[v] = OP == OP_LSE ? (LONG ? lse_value(acc[v], mx[v]) : mx[v] + flog(acc[v])) : finish<OP>(acc[v], mx[v], nc[v]);
    if (OpTraits<OP>::shares) {
        // a sum of P rows out of range: the row once more, as in the streaming kernel
        bool beyond = false;
#pragma unroll
        for (int v = 0; v < VEC; ++v) beyond |= !(fabsf(mx[v]) < INFINITY);
        if (beyond) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) { acc[v] = identity<OP>(); mx[v] = identity2<OP>(); }
            for (int k = range.x; k < end; ++k) {
                const uint32_t id = a.idx[k];
                float x[VEC];
                load_cols<VEC>(x, a.src + (size_t)(id & kIdMask) * a.ld + col);
#pragma unroll
                for (int v = 0; v < VEC; ++v) accumulate<OP>(acc[v], mx[v], x[v], share_scale(nc[v]), nc[v], (id & kWeighted) != 0);
            }
#pragma unroll
            for (int v = 0; v < VEC; ++v) o[v] = finish<OP>(acc[v], mx[v], nc[v], share_scale(nc[v]));
        }
    }
    if (OP == OP_SUM_H && row < a.n_main && (last & kRowFlag)) {
#pragma unroll
        for (int v = 0; v < VEC; ++v) o[v] = encode_h(o[v], nc[v]);
    }
    if (OpTraits<OP>::premul && row < a.n_main) {
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            if (nc[v] == 0.0f && a.zero_flag) *a.zero_flag = 1;
            o[v] = premultiply(o[v], nc[v]);
        }
    }
    float* out;
    if (row < a.n_main) out = a.dst + (size_t)(a.out_row ? a.out_row[row] : row) * a.ld + col;
    else out = a.dst_seg + (size_t)(row - a.n_main) * a.ld + col;
    store_cols<VEC>(out, o);
}

template <int OP, int VEC, bool LONG>
__global__ __launch_bounds__(256) void pass_kernel(PassArgs a) {
    arguments_now(a);
    pass_body<OP, VEC, LONG>((int)blockIdx.x, (int)gridDim.x, a);
}

// ---------------------------------------------------------------------------------------------
// Combine pass of split rows for B > 32, NW waves in a workgroup.  A row of many partial rows (up to a few hundred; the first `many`
// rows of the lists) takes a workgroup: its partial rows are dealt to the waves in chunks of 8, every wave
// reduces its share with all its gathers of a chunk in flight, and wave 0 folds the NW states in wave
// order (so the result does not depend on timing) and finishes the row like pass_kernel does.  A single
// wave would walk the widest row 8 partial rows at a time, and the launch lasts as long as that walk.  The
// others, which are nearly all, take a wave: a workgroup for each of them is mostly waves that have no chunk, and a
// barrier (9454 rows at B = 50 16.3 us, 7616 at B = 256 34.8).
// Arguments as for pass_kernel's combine use: ptr / idx = combine lists, src = partial rows, out_row = the
// rows to write, n_main = number of split rows.
// ---------------------------------------------------------------------------------------------
template <int OP, int VEC, int NW>
__device__ __forceinline__ void combine_body(int bx, const PassArgs& a, int many) {
    constexpr int CH = 8;
    constexpr bool LSE = OP == OP_LSE;
    __shared__ float part_v[NW][64 * VEC];
    __shared__ float part_m[LSE ? NW : 1][LSE ? 64 * VEC : 1];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int colu = ((int)blockIdx.y * 64 + lane) * VEC;
    const int col = colu < a.B ? colu : 0;                 // lanes past the batch work on column 0 and store nothing
    const bool shared = bx < many;
    const int row = shared ? bx : many + (bx - many) * NW + wave;
    if (row >= a.n_main) return;                           // (all waves of a shared row are there)
    const int beg = a.ptr[row], end = a.ptr[row + 1];
    const int step = shared ? NW * CH : CH;
    float acc[VEC], mx[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) { acc[v] = identity<OP>(); mx[v] = -INFINITY; }
    for (int j = beg + (shared ? wave * CH : 0); j < end; j += step) {
        float x[CH][VEC];
#pragma unroll
        for (int i = 0; i < CH; ++i)                         // padded list: always in bounds
            load_vec<VEC>(x[i], a.src + (size_t)(a.idx[j + i] & kIdMask) * a.ld + col);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const bool live = j + i < end;
#pragma unroll
            for (int v = 0; v < VEC; ++v) { float none = 0.0f; accumulate<OP>(acc[v], mx[v], live ? x[i][v] : dead_value<OP>(), 0.0f, none, false); }
        }
    }
    if (shared) {
        if (wave > 0) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                part_v[wave][lane * VEC + v] = acc[v];
                if (LSE) part_m[wave][lane * VEC + v] = mx[v];
            }
        }
        __syncthreads();
        if (wave > 0) return;
        for (int w = 1; w < NW; ++w) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                const float ov = part_v[w][lane * VEC + v];
                if (LSE) {
                    const float om = part_m[w][lane * VEC + v];
                    edge_combine<OP>(mx[v], acc[v], om, ov);
                } else {
                    float unused = 0.0f;
                    edge_combine<OP>(acc[v], unused, ov, 0.0f);
                }
            }
        }
    }
    if (colu >= a.B) return;
    const int out_row = a.out_row[row];
    float o[VEC], nc[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) { o[v] = finish<OP>(acc[v], mx[v]); nc[v] = 0.0f; }
    if (OP == OP_SUM_H || OP == OP_SUM_P) load_vec<VEC>(nc, a.own + (size_t)out_row * a.ld + col);
    if (OP == OP_SUM_H && (a.idx[end - 1] & kRowFlag)) {
#pragma unroll
        for (int v = 0; v < VEC; ++v) o[v] = encode_h(o[v], nc[v]);
    }
    if (OP == OP_SUM_P) {
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            if (nc[v] == 0.0f && a.zero_flag) *a.zero_flag = 1;
            o[v] = premultiply(o[v], nc[v]);
        }
    }
    store_vec<VEC>(a.dst + (size_t)out_row * a.ld + col, o);
}

template <int OP, int VEC, int NW>
__global__ __launch_bounds__(NW * 64) void combine_kernel(PassArgs a, int many) {
    combine_body<OP, VEC, NW>((int)blockIdx.x, a, many);
}

// 32 < B <= 64: the combine rows and the main rows of a large layer, after the launch of its segments.  The first n_comb_blocks
// workgroups (a multiple of 8, so that the others keep their XCDs) take combine rows, the rest the main rows: neither waits for the other.
template <int OP, int COP, int VEC>
__global__ __launch_bounds__(256) void pass_combine_kernel(PassArgs a, int n_comb_blocks, PassArgs cmb, int many) {
    if ((int)blockIdx.x < n_comb_blocks) combine_body<COP, 1, 4>((int)blockIdx.x, cmb, many);
    else pass_body<OP, VEC, false>((int)blockIdx.x - n_comb_blocks, (int)gridDim.x - n_comb_blocks, a);
}

// The same for B <= 32 and split rows of many partial rows (kShortComb): W lanes (a power of two) hold the columns of a partial row, so a wave takes 64 / W partial rows at
// a time, four of them in flight; the lane groups meet in a butterfly, the four waves in LDS, in a fixed order.  (A lane
// group per split row walked the partial rows of the widest row, up to a few hundred, alone.)
template <int OP, int W>
__global__ __launch_bounds__(256) void combine_small_kernel(PassArgs a) {
    constexpr int G = 64 / W, CH = 4;
    constexpr bool LSE = OP == OP_LSE;
    arguments_now(a);
    __shared__ float part_v[4][W], part_m[LSE ? 4 : 1][LSE ? W : 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int sub = lane / W, c = lane % W;
    const int col = c < a.B ? c : a.B - 1;
    const int row = (int)blockIdx.x;
    const int beg = a.ptr[row], end = a.ptr[row + 1];
    // (accm, accs): the reduction, or (maximum, sum of exp(x - maximum))
    float accm = LSE ? -INFINITY : identity<OP>(), accs = 0.0f;
    for (int j = beg + wave * G + sub; __any(j < end); j += 4 * G * CH) {
        float x[CH];
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int at = j + i * 4 * G < end ? j + i * 4 * G : beg;
            x[i] = a.src[(size_t)(a.idx[at] & kIdMask) * a.ld + col];
        }
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const bool live = j + i * 4 * G < end;
            edge_combine<OP>(accm, accs, live ? x[i] : (LSE ? -INFINITY : identity<OP>()), live ? 1.0f : 0.0f);
        }
    }
#pragma unroll
    for (int d = W; d < 64; d <<= 1) {
        const float om = __shfl_xor(accm, d), os = LSE ? __shfl_xor(accs, d) : 0.0f;
        edge_combine<OP>(accm, accs, om, os);
    }
    if (sub == 0) {
        part_v[wave][c] = LSE ? accs : accm;
        if (LSE) part_m[wave][c] = accm;
    }
    __syncthreads();
    if (threadIdx.x >= W || (int)threadIdx.x >= a.B) return;
    for (int w = 1; w < 4; ++w) edge_combine<OP>(accm, accs, LSE ? part_m[w][c] : part_v[w][c], LSE ? part_v[w][c] : 0.0f);
    const int out_row = a.out_row[row];
    float o = LSE ? (accm == -INFINITY ? -INFINITY : accm + flog(accs)) : accm;
    if (OP == OP_SUM_H || OP == OP_SUM_P) {
        const float own = a.own[(size_t)out_row * a.ld + c];
        if (OP == OP_SUM_H && (a.idx[end - 1] & kRowFlag)) o = encode_h(o, own);
        if (OP == OP_SUM_P) {
            if (own == 0.0f && a.zero_flag) *a.zero_flag = 1;
            o = premultiply(o, own);
        }
    }
    a.dst[(size_t)out_row * a.ld + c] = o;
}

// ---------------------------------------------------------------------------------------------
// Persistent kernels for the top of the circuit (the layers that taper to the roots; for a small
// circuit every layer): instead of one launch per layer, a workgroup of 16 waves owns CT batch columns (1, 2 or 4, see
// tail_columns), keeps
// the values (forward) or the adjoints (reverse) of the layer in hand and of the one below or above in LDS and
// walks the layers with a barrier in between.  Batch columns are independent, so no grid-wide
// barrier is needed.  More than 256 workgroups take turns on the compute units (one needs the registers of a whole one).
//   Index vectors stay in global memory, as blocks and tables of runs (ColPlan, layerize.h): one stream of each per
// wave, contiguous over all layers, so a wave fetches the next block and the next table ahead of the ones it works
// on, also across the layer barriers.  A table is read one descriptor per lane and broadcast to scalars
// (readlane); scalar loads would share their wait counter with the LDS gathers.
//   What bounds these kernels: one compute unit evaluates whole columns, so first the longest wave of each layer
// (hence several lanes per long row, and shares of equal cost), then the latency of the dependent steps of a row and
// the control flow around it (hence runs of one kind, 16 gathers of a lane in flight together) and then the
// instructions per entry, of which a
// logsumexp entry has most (hence whole rows: one maximum, one exponential per entry, no running rescale).
//   Measured against one lane per row, chunks dealt in turn and a running logsumexp (forward / forward + backward, log
// semiring): 85000 nodes, 263000 edges, 20 layers at B = 128: 52 -> 42 us / 211 -> 100 us (there the reverse kernel
// could not take layers with nodes of more than 64 parents); 467 nodes, 22 layers at B = 4: 19.5 -> 16.6 us.  A
// wide layer costs about 5 ns per 64 entries, a narrow one cost 2000 cycles of dependent steps and costs 700 as units (ColUnits).
//   A lane owns rows of few batch columns, so writing values into the row-major activation buffer
// would cost one cache line per lane.  The values go to a column-major buffer tb[column][T] instead
// (T = rows of all candidate layers), where consecutive lanes write consecutive floats; the reverse
// kernel reads it the same way, and rows that an ordinary launch needs are transposed back on demand
// (tb_to_rows_kernel).
// ---------------------------------------------------------------------------------------------
constexpr int kColThreads = 64 * kColWaves;
// a layer: its nodes, its first entry in a column of the value buffer, and where the streams of the 16 waves start
// (blocks, tables; bwd: of the step into the layer below)
struct ColLayer {
    int32_t n, at;
    int32_t fwd_block[kColWaves], fwd_table[kColWaves];
    int32_t bwd_block[kColWaves], bwd_table[kColWaves];
    int32_t fwd_unit[kColWaves], bwd_unit[kColWaves];        // narrow layers: the waves' first units
};

typedef uint32_t Line __attribute__((ext_vector_type(4)));       // a lane's 16 bytes of a line
typedef uint32_t Desc __attribute__((ext_vector_type(2)));

// A copy of what a load brought, so that the next load can go to the same registers.  Without it the compiler loads the next block
// into others, moves it over where the ways through a run or a layer meet, and waits for it there: in front of the
// barrier.  (Forward, us: 85000 nodes in 20 layers, B = 128 41.4 -> 39.7; 467 nodes in 22 layers, B = 4 16.2 -> 15.9; 800000 nodes, B = 1 103.9
// -> 101.4.  With one loop over blocks of any kind it never waits there, but the branches for every block cost more: 42.8, 17.9, 104.4.)
__device__ __forceinline__ Desc taken(Desc x) {
    Desc r;
    asm volatile("v_mov_b64 %0, %1" : "=v"(r) : "v"(x));
    return r;
}
__device__ __forceinline__ Line taken(Line x) {
    const Desc a = taken(Desc{x.x, x.y}), b = taken(Desc{x.z, x.w});
    return Line{a.x, a.y, b.x, b.y};
}

// a wave's place in its two streams: the block and the table in flight
struct ColWalk {
    const Line* q;
    const Desc* d;
    Line r0, r1;
    Desc ahead;

    __device__ __forceinline__ void start(const Line* blocks, const Desc* tables) {
        q = blocks;
        d = tables;
        r0 = q[0];
        r1 = q[64];
        ahead = *d;
    }
    __device__ __forceinline__ void block(Line& w0, Line& w1) {
        w0 = taken(r0);
        w1 = taken(r1);
        q += 128;
        r0 = q[0];
        r1 = q[64];
    }
    __device__ __forceinline__ Desc table() {
        const Desc t = taken(ahead);
        d += kDescTable;
        ahead = *d;
        return t;
    }
};

// a run, from its descriptor in the table
struct ColRun {
    int slot, rows, k, kind, blocks;
    __device__ __forceinline__ bool read(ColWalk& walk, Desc& table, int& i) {
        i = __builtin_amdgcn_readfirstlane(i);
        uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)table.x, i), b = (uint32_t)__builtin_amdgcn_readlane((int)table.y, i);
        if ((b & 0xFFFFu) == 0) {
            if (a == 0) return false;
            table = walk.table();
            i = 0;
            a = (uint32_t)__builtin_amdgcn_readlane((int)table.x, 0);
            b = (uint32_t)__builtin_amdgcn_readlane((int)table.y, 0);
        }
        ++i;
        slot = (int)(a & 0x7FFFu);
        rows = (int)(b & 0xFFFFu);
        k = (int)((b >> 16) & 15u);
        kind = (int)((b >> 20) & 15u);
        blocks = (int)(a >> 15);
        return true;
    }
};

// The values of a node in the CT columns of a workgroup.
template <int CT> struct ColValue { typedef float T __attribute__((ext_vector_type(CT))); };
template <> struct ColValue<1> { using T = float; };

// f of each column
template <class F>
__device__ __forceinline__ float each(F f, float a) { return f(a); }
template <class F>
__device__ __forceinline__ float each(F f, float a, float b) { return f(a, b); }
template <class F>
__device__ __forceinline__ float each(F f, float a, float b, float c) { return f(a, b, c); }
template <class F, class V, int N = (int)(sizeof(V) / sizeof(float)), class = decltype(V().x)>
__device__ __forceinline__ V each(F f, V a) {
    V r;
#pragma unroll
    for (int i = 0; i < N; ++i) r[i] = f(a[i]);
    return r;
}
template <class F, class V, int N = (int)(sizeof(V) / sizeof(float)), class = decltype(V().x)>
__device__ __forceinline__ V each(F f, V a, V b) {
    V r;
#pragma unroll
    for (int i = 0; i < N; ++i) r[i] = f(a[i], b[i]);
    return r;
}
template <class F, class V, int N = (int)(sizeof(V) / sizeof(float)), class = decltype(V().x)>
__device__ __forceinline__ V each(F f, V a, V b, V c) {
    V r;
#pragma unroll
    for (int i = 0; i < N; ++i) r[i] = f(a[i], b[i], c[i]);
    return r;
}
template <class V, class = decltype(V().x)>
__device__ __forceinline__ V term_exp(V x) { return each([](float a) { return term_exp(a); }, x); }
template <class V, class = decltype(V().x)>
__device__ __forceinline__ V flog(V x) { return each([](float a) { return flog(a); }, x); }
template <class V, class = decltype(V().x)>
__device__ __forceinline__ V finite(V x) { return each([](float a) { return finite(a); }, x); }
template <class V, class = decltype(V().x)>
__device__ __forceinline__ V max3(V a, V b, V c) { return each([](float x, float y, float z) { return max3(x, y, z); }, a, b, c); }
template <class V, class = decltype(V().x)>
__device__ __forceinline__ V bigger(V a, V b) { return each([](float x, float y) { return bigger(x, y); }, a, b); }
template <class V>
__device__ __forceinline__ V apart(V a, V b) { return each([](float x, float y) { return fabsf(x - y); }, a, b); }
template <class V>
__device__ __forceinline__ V muladd(V a, V b, V c) { return each([](float x, float y, float z) { return fmaf(x, y, z); }, a, b, c); }

template <class V>
__device__ __forceinline__ V col_at(const V* values, uint32_t slot) { return values[slot]; }

// lane i's value from lane i ^ (1 << step), for reductions in which the lanes below that distance already agree
template <int STEP>
__device__ __forceinline__ float fly(float x) {
    constexpr int kCtrl = STEP == 0 ? 0xB1 : STEP == 1 ? 0x4E : STEP == 2 ? 0x141 : 0x140;      // quad_perm, half mirror, mirror
    if (STEP < 4) return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), kCtrl, 0xF, 0xF, true));
    return __shfl_xor(x, 1 << STEP);
}
template <int STEP, class V, class = decltype(V().x)>
__device__ __forceinline__ V fly(V x) { return each([](float a) { return fly<STEP>(a); }, x); }

template <int OP, class V>
__device__ __forceinline__ V col_join(V a, V b) {
    if constexpr (OP == OP_PROD) return a * b;
    else if constexpr (OP == OP_MAX || OP == OP_LSE) return bigger(a, b);      // (OP_LSE: the maxima)
    else return a + b;
}

// reduce over the 2^k lanes of a row; every lane of the row ends with the result
template <int OP, class V>
__device__ __forceinline__ V col_fly(V x, int k) {
    if (k >= 1) x = col_join<OP>(x, fly<0>(x));
    if (k >= 2) x = col_join<OP>(x, fly<1>(x));
    if (k >= 3) x = col_join<OP>(x, fly<2>(x));
    if (k >= 4) x = col_join<OP>(x, fly<3>(x));
    if (k >= 5) x = col_join<OP>(x, fly<4>(x));
    if (k >= 6) x = col_join<OP>(x, fly<5>(x));
    return x;
}

// Logsumexp in the persistent kernel: m = maximum so far, s = sum of exp(x - finite(m)), where finite() keeps the
// subtrahend between -FLT_MAX and FLT_MAX, so that no difference is inf - inf: a row of impossible children ends as
// -inf + log(0) = -inf, one with an infinite weight as inf.
// the value of a row of one entry, of two, of four
template <int OP, class V>
__device__ __forceinline__ V col_one(V x) {
    if (OP != OP_LSE && OP != OP_MAX) return x;
    return bigger(x, V(-INFINITY));
}
template <int OP, class V>
__device__ __forceinline__ V col_two(V x, V y) {
    if (OP != OP_LSE && OP != OP_MAX) return col_join<OP>(x, y);
    const V hi = max3(x, y, V(-INFINITY));
    return OP == OP_MAX ? hi : hi + flog(1.0f + term_exp(-apart(x, y)));      // (apart: NaN for two equal infinities too, a term of 0)
}
template <int OP, class V>
__device__ __forceinline__ V col_four(V x0, V x1, V x2, V x3) {
    if (OP != OP_LSE && OP != OP_MAX) return col_join<OP>(col_join<OP>(x0, x1), col_join<OP>(x2, x3));
    const V hi = max3(max3(x0, x1, x2), x3, V(-INFINITY));
    if (OP == OP_MAX) return hi;
    const V m = finite(hi);
    return hi + flog((term_exp(x0 - m) + term_exp(x1 - m)) + (term_exp(x2 - m) + term_exp(x3 - m)));
}

// Reads one word of every 128 bytes of the blocks and units, shared out among the workgroups of an XCD (every eighth one), so that
// they are in its L2 when the waves get to them: the workgroups walk the layers in step, and without this the first
// one to reach a block would wait for the memory behind the L2, a few thousand cycles, at every layer (1m nodes at B = 256:
// 413 -> 390 us; a few workgroups alone read more than they save, so only from 64 on).  In the forward kernel by the wave that has nothing else to
// do in the first layer; the others wait for it only where they wait anyway (kernel alone, with 16-byte loads of the layer below the first one, us:
// 85000 nodes B = 128 37.8 -> 36.8, 800000 nodes B = 1 37.2 -> 33.5).
template <int N> struct ColTouch {
    const uint32_t* words;
    int n, at, step;
    uint32_t x[N];
    // `thread` of the `threads` of this workgroup that take part
    __device__ __forceinline__ void ask(const Line* lines, int n_kb, int thread, int threads) {
        words = reinterpret_cast<const uint32_t*>(lines);
        n = n_kb * 8;
        step = ((int)gridDim.x + 7) / 8 * threads;
        at = (int)blockIdx.x / 8 * threads + thread;
        more();
    }
    __device__ __forceinline__ void more() {
#pragma unroll
        for (int j = 0; j < N; ++j) x[j] = words[(size_t)(at + j * step < n ? at + j * step : 0) * 32];
        at += N * step;
    }
    __device__ __forceinline__ void finish() {
        for (;;) {
#pragma unroll
            for (int j = 0; j < N; ++j) asm volatile("" ::"v"(x[j]));
            if (!__any(at < n)) return;
            more();
        }
    }
};

// The values of the rows that two words (four entries) of a lane stand for: four rows of one entry, two of two, one of four.
template <int OP, int KIND, class V>
__device__ __forceinline__ void col_rows(const V* below, uint32_t a, uint32_t b, V* v) {
    const V x0 = col_at(below, a & 0xFFFFu), x1 = col_at(below, a >> 16), x2 = col_at(below, b & 0xFFFFu), x3 = col_at(below, b >> 16);
    if (KIND == 0) { v[0] = col_one<OP>(x0); v[1] = col_one<OP>(x1); v[2] = col_one<OP>(x2); v[3] = col_one<OP>(x3); }
    if (KIND == 1) { v[0] = col_two<OP>(x0, x1); v[1] = col_two<OP>(x2, x3); }
    if (KIND == 2) v[0] = col_four<OP>(x0, x1, x2, x3);
}

// the last rows of a run, in one quarter of a block
template <int OP, int KIND, class V>
__device__ __forceinline__ void col_fwd_rest(const V* below, uint32_t a, uint32_t b, V* out, int rows) {
    constexpr int N = 4 >> KIND;
    const int lane = threadIdx.x & 63;
    V v[N];
    col_rows<OP, KIND>(below, a, b, v);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if (rows >= 64 * (i + 1)) out[64 * i] = v[i];
        else if (lane + 64 * i < rows) out[64 * i] = v[i];
    }
}

// a run of kind 0, 1 or 2
template <int OP, int KIND, class V>
__device__ __forceinline__ void col_fwd_short(ColWalk& walk, const V* below, V* out, int rows) {
    constexpr int N = 4 >> KIND;                     // rows of a lane in a quarter of a block
    out += threadIdx.x & 63;
    Line w0, w1;
    for (; rows >= 256 * N; rows -= 256 * N, out += 256 * N) {
        walk.block(w0, w1);
        if constexpr (sizeof(V) <= 8) {
            V v[4 * N];
            col_rows<OP, KIND>(below, w0.x, w0.y, v);
            col_rows<OP, KIND>(below, w0.z, w0.w, v + N);
            col_rows<OP, KIND>(below, w1.x, w1.y, v + 2 * N);
            col_rows<OP, KIND>(below, w1.z, w1.w, v + 3 * N);
#pragma unroll
            for (int i = 0; i < 4 * N; ++i) out[64 * i] = v[i];
        } else {
            // (four columns: half a block, so that the values fit the registers)
            V v[2 * N];
            col_rows<OP, KIND>(below, w0.x, w0.y, v);
            col_rows<OP, KIND>(below, w0.z, w0.w, v + N);
#pragma unroll
            for (int i = 0; i < 2 * N; ++i) out[64 * i] = v[i];
            col_rows<OP, KIND>(below, w1.x, w1.y, v);
            col_rows<OP, KIND>(below, w1.z, w1.w, v + N);
#pragma unroll
            for (int i = 0; i < 2 * N; ++i) out[64 * (2 * N + i)] = v[i];
        }
    }
    if (rows > 0) {
        walk.block(w0, w1);
        col_fwd_rest<OP, KIND>(below, w0.x, w0.y, out, rows);
        if (rows > 64 * N) col_fwd_rest<OP, KIND>(below, w0.z, w0.w, out + 64 * N, rows - 64 * N);
        if (rows > 128 * N) {
            col_fwd_rest<OP, KIND>(below, w1.x, w1.y, out + 128 * N, rows - 128 * N);
            if (rows > 192 * N) col_fwd_rest<OP, KIND>(below, w1.z, w1.w, out + 192 * N, rows - 192 * N);
        }
    }
}

// the lanes of a row have (m, s): its value
template <class V>
__device__ __forceinline__ V col_lse_fly(V m, V s, int k) {
    if (k > 0) {
        const V m2 = col_fly<OP_LSE>(m, k);
        s = col_fly<OP_SUM>(s * term_exp(m - finite(m2)), k);
        m = m2;
    }
    return m + flog(s);
}

// one line of a row that takes several lanes or lines, joined to what the lines before gave
template <int OP, class V>
__device__ __forceinline__ void col_long(const V* below, Line w, bool fresh, V& m, V& s) {
    const V x0 = col_at(below, w.x & 0xFFFFu), x1 = col_at(below, w.x >> 16), x2 = col_at(below, w.y & 0xFFFFu), x3 = col_at(below, w.y >> 16);
    const V x4 = col_at(below, w.z & 0xFFFFu), x5 = col_at(below, w.z >> 16), x6 = col_at(below, w.w & 0xFFFFu), x7 = col_at(below, w.w >> 16);
    if (OP == OP_LSE) {
        const V hi = max3(max3(max3(x0, x1, x2), x3, x4), max3(x5, x6, x7), m), m2 = finite(hi);
        const V s2 = ((term_exp(x0 - m2) + term_exp(x1 - m2)) + (term_exp(x2 - m2) + term_exp(x3 - m2))) +
                         ((term_exp(x4 - m2) + term_exp(x5 - m2)) + (term_exp(x6 - m2) + term_exp(x7 - m2)));
        s = fresh ? s2 : muladd(s, term_exp(m - m2), s2);
        m = hi;
    } else {
        const V x = col_join<OP>(col_four<OP>(x0, x1, x2, x3), col_four<OP>(x4, x5, x6, x7));
        s = fresh ? x : col_join<OP>(s, x);
    }
}

// one layer, forward
template <int OP, class V>
__device__ __forceinline__ void col_fwd_layer(ColWalk& walk, const V* below, V* here) {
    const int lane = threadIdx.x & 63;
    Desc table = walk.table();
    ColRun run;
    for (int i = 0; run.read(walk, table, i);) {
        V* out = here + run.slot;
        if (run.kind == 0) col_fwd_short<OP, 0>(walk, below, out, run.rows);
        else if (run.kind == 1) col_fwd_short<OP, 1>(walk, below, out, run.rows);
        else if (run.kind == 2) col_fwd_short<OP, 2>(walk, below, out, run.rows);
        else {
            const int r = lane >> run.k, per = 64 >> run.k;
            const bool writes = (lane & ((1 << run.k) - 1)) == 0;
            for (int rows = run.rows; rows > 0; rows -= per, out += per) {
                V m = V(-INFINITY), s = V(0.0f);
                Line w0, w1;
                walk.block(w0, w1);
                col_long<OP>(below, w0, true, m, s);
                if (run.kind == 3) {
                    col_long<OP>(below, w1, false, m, s);
                    for (int b = 1; b < run.blocks; ++b) {
                        walk.block(w0, w1);
                        col_long<OP>(below, w0, false, m, s);
                        col_long<OP>(below, w1, false, m, s);
                    }
                }
                s = OP == OP_LSE ? col_lse_fly(m, s, run.k) : col_fly<OP>(s, run.k);
                if (writes && r < rows) out[r] = s;
            }
        }
    }
}

// The narrow layers (ColPlan::units).  A run of the walk above costs a wave 600 cycles before its first row (descriptor, branches,
// a block that was asked for one block ago), more than all the work of a layer of a few hundred rows.  A unit says everything itself and was
// asked for four units ago, so what is left is the barrier, the gathers and the sum.  Kernel alone, us, runs throughout / units up to
// 30 / 60 / 90 of them in a layer: 467 nodes in 22 layers at B = 4 16.3 / 9.7 / 9.7 / 9.7; 85000 nodes in 20 layers at B = 128 41.1 / 36.8 / 35.2 /
// 35.1; 800000 nodes, 26 of 40 layers in the kernel, B = 1 42.8 / 33.5 / 31.3 / 32.4, B = 256 53.8 / 45.9 / 44.7 / 44.3; the reverse kernel there at
// B = 10 65.9 / - / 59.2.
struct ColUnits {
    const Line* q;
    Line r[kUnitsAhead];
    __device__ __forceinline__ void start(const Line* units) {
        q = units;
#pragma unroll
        for (int i = 0; i < kUnitsAhead; ++i) r[i] = q[64 * i];
        q += 64 * kUnitsAhead;
    }
    // r[i] has been worked off
    __device__ __forceinline__ void next(int i) {
        r[i] = *q;
        q += 64;
    }
};

// reduce over the 2^lanes lanes of a row, k the most of the unit
template <int OP, class V>
__device__ __forceinline__ V unit_fly(V x, int lanes, int k) {
    x = lanes >= 1 ? col_join<OP>(x, fly<0>(x)) : x;
    x = lanes >= 2 ? col_join<OP>(x, fly<1>(x)) : x;
    if (k > 2) {
        x = lanes >= 3 ? col_join<OP>(x, fly<2>(x)) : x;
        x = lanes >= 4 ? col_join<OP>(x, fly<3>(x)) : x;
    }
    if (k > 4) {
        x = lanes >= 5 ? col_join<OP>(x, fly<4>(x)) : x;
        x = lanes >= 6 ? col_join<OP>(x, fly<5>(x)) : x;
    }
    return x;
}

// the value of a lane's row
template <int OP, class V>
__device__ __forceinline__ V col_fwd_row(const V* below, Line w, uint32_t head) {
    const int lanes = (int)(w.x >> kUnitLanesAt) & 7, k = (int)(head >> kUnitLanesAt) & 7;
    const V x0 = col_at(below, w.y & 0xFFFFu), x1 = col_at(below, w.y >> 16), x2 = col_at(below, w.z & 0xFFFFu);
    V m = V(-INFINITY), s;
    if (head & kUnitShort) {
        if constexpr (OP == OP_LSE || OP == OP_MAX) {
            m = bigger(max3(x0, x1, x2), m);
            if (OP == OP_MAX) return m;
            const V f = finite(m);
            s = (term_exp(x0 - f) + term_exp(x1 - f)) + term_exp(x2 - f);
            return m + flog(s);
        }
        return col_join<OP>(col_join<OP>(x0, x1), x2);
    }
    const V x3 = col_at(below, w.z >> 16), x4 = col_at(below, w.w & 0xFFFFu), x5 = col_at(below, w.w >> 16);
    if constexpr (OP == OP_LSE || OP == OP_MAX) {
        m = bigger(max3(max3(x0, x1, x2), x3, max3(x4, x5, m)), m);
        if (k > 0) m = unit_fly<OP>(m, lanes, k);
        if (OP == OP_MAX) return m;
        const V f = finite(m);
        s = ((term_exp(x0 - f) + term_exp(x1 - f)) + (term_exp(x2 - f) + term_exp(x3 - f))) + (term_exp(x4 - f) + term_exp(x5 - f));
        if (k > 0) s = unit_fly<OP_SUM>(s, lanes, k);
        return m + flog(s);
    }
    s = col_join<OP>(col_join<OP>(col_join<OP>(x0, x1), col_join<OP>(x2, x3)), col_join<OP>(x4, x5));
    return k > 0 ? unit_fly<OP>(s, lanes, k) : s;
}

// one unit; true: the wave has no further rows
template <int AND, int OR, class V>
__device__ __forceinline__ bool col_fwd_unit(Line w, V*& below, V*& here) {
    const uint32_t head = (uint32_t)__builtin_amdgcn_readfirstlane((int)w.x);
    if (head & kUnitEnd) return true;
    if (head & kUnitNew) {
        __syncthreads();
        V* tmp = below; below = here; here = tmp;
    }
    if (head & kUnitIdle) return false;
    V* out = here + (w.x & kUnitSlot);
    if (head & kUnitOr) *out = col_fwd_row<OR>(below, w, head);
    else *out = col_fwd_row<AND>(below, w, head);
    return false;
}

// the wave's units of the narrow layers; `below` ends as the last one's values
template <int AND, int OR, class V>
__device__ __forceinline__ void col_fwd_units(const Line* units, V*& below, V*& here) {
    ColUnits walk;
    walk.start(units);
    V* tmp = below; below = here; here = tmp;            // (as after a layer)
    for (bool done = false; !done;) {
#pragma unroll
        for (int i = 0; i < kUnitsAhead; ++i) {
            if ((done = col_fwd_unit<AND, OR>(walk.r[i], below, here))) break;
            walk.next(i);
        }
    }
    below = here;
}

// a finished layer's values from LDS to the column-major buffer, by one wave, 16 bytes a lane
__device__ __forceinline__ void col_move(const float* values, int n, float* __restrict__ to) {
    typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
    const int lane = threadIdx.x & 63;
    const int whole = n / 4 * 4;
#pragma unroll 4
    for (int i = lane * 4; i < whole; i += 256) {
        const float4 v = *reinterpret_cast<const float4*>(values + i);
        *reinterpret_cast<f4u*>(to + i) = f4u{v.x, v.y, v.z, v.w};
    }
    if (whole + lane < n) to[whole + lane] = values[whole + lane];
}
// (CT columns, T floats apart, `columns` of them there; also 16 bytes a lane and column: with a float a lane the wave took
// longer than the others took for layers of short rows, 131000 nodes in 48 layers forward at B = 400: 141 us, so 106)
template <int CT>
__device__ __forceinline__ void col_move(const float* values, int n, float* __restrict__ to, int T, int columns) {
    if constexpr (CT == 1) {
        col_move(values, n, to);
    } else {
        typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
        const int lane = threadIdx.x & 63;
        const int whole = n / 4 * 4;
        float* column[CT];                                // (one that is not there: the last one again)
#pragma unroll
        for (int c = 0; c < CT; ++c) column[c] = to + (size_t)(c < columns ? c : columns - 1) * T;
#pragma unroll (8 / CT)
        for (int i = lane * 4; i < whole; i += 256) {
            float4 v[CT];
#pragma unroll
            for (int j = 0; j < CT; ++j) v[j] = *reinterpret_cast<const float4*>(values + CT * i + 4 * j);
            const float* x = reinterpret_cast<const float*>(v);
#pragma unroll
            for (int c = 0; c < CT; ++c) *reinterpret_cast<f4u*>(column[c] + i) = f4u{x[c], x[CT + c], x[2 * CT + c], x[3 * CT + c]};
        }
        if (whole + lane < n)
            for (int c = 0; c < CT; ++c) column[c][whole + lane] = values[CT * (whole + lane) + c];
    }
}

__device__ __forceinline__ float log1mexp_f(float x) {
    return x > -0.69314718f ? logf(-expm1f(x)) : log1pf(-expf(x));
}

// Where the values of the CT columns of a workgroup are in the column-major buffer: T floats apart, `columns` of them there (one
// that is not: the last one again).
struct ColColumns {
    int T, columns;
    __device__ __forceinline__ int operator()(int c) const { return (c < columns ? c : columns - 1) * T; }
};

// four rows of the columns to their slots
typedef float Float4u __attribute__((ext_vector_type(4), aligned(4)));
template <int CT, class V>
__device__ __forceinline__ void col_put4(V* to, const Float4u (&v)[CT]) {
    float x[4 * CT];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int c = 0; c < CT; ++c) x[j * CT + c] = v[c][j];
#pragma unroll
    for (int i = 0; i < CT; ++i) reinterpret_cast<float4*>(to)[i] = make_float4(x[4 * i], x[4 * i + 1], x[4 * i + 2], x[4 * i + 3]);
}

// n node values of the columns into LDS, 16-byte aligned, up to twenty values of a column per thread in flight (at one column a layer of
// kTailRowsCap rows)
template <int CT, class V>
__device__ __forceinline__ void col_load(V* to, const float* from, ColColumns column, int n) {
    constexpr int kFlight = CT == 4 ? 2 : CT == 2 ? 4 : 5;
    const int whole = n / 4 * 4;
    for (int i0 = 4 * (int)threadIdx.x; i0 < whole; i0 += 4 * kFlight * kColThreads) {
        Float4u v[kFlight][CT];
#pragma unroll
        for (int j = 0; j < kFlight; ++j) {
            const int i = i0 + 4 * j * kColThreads < whole ? i0 + 4 * j * kColThreads : i0;
#pragma unroll
            for (int c = 0; c < CT; ++c) v[j][c] = *reinterpret_cast<const Float4u*>(from + column(c) + i);
        }
#pragma unroll
        for (int j = 0; j < kFlight; ++j) col_put4<CT>(to + (i0 + 4 * j * kColThreads < whole ? i0 + 4 * j * kColThreads : i0), v[j]);
    }
    const int rest = whole + (int)threadIdx.x;
    if (rest < n)
        for (int c = 0; c < CT; ++c) reinterpret_cast<float*>(to + rest)[c] = from[column(c) + rest];
}

// Arguments of the leaf layer when the persistent kernel evaluates it itself (its first layer is
// layer 1): a workgroup reads its own rows of the leaf-weight arrays, which are contiguous.
struct SlabLeaf {
    const float* w;             // [B, V] leaf weights (null: the leaf layer was evaluated by leaf_fwd_kernel)
    const float* wneg;          // [B, V] weights of the negated literals, or null
    const int32_t *pos_row, *neg_row;    // [V] layer-0 row of each literal or -1; LISTED: of some variables alone, the two arrays and these variables' numbers one after another
    float* wT;                  // [V, ld] transposed leaf weights kept for the reverse sweep (which reads those of variables with a negated literal)
    float* act0;                // [n_0, ld] rows of layer 0 in the activation buffer
    int32_t V, true_row, false_row;      // rows of the constants or -1
};

// LDS: two value arrays, slots kColSlots + position; size0 floats for the layer below the first one and every second
// layer from there, the rest for the others.  start_rows / start_at: the layer below the first one (start_rows of them),
// column-major, start_T floats a column, if start_T > 0 (and start_map is null), otherwise rows of the activation buffer (start_map[i], or null: one after another).
// tb (or null): every layer's values are kept there.  CT: columns of a workgroup.
// wide: so many layers before the narrow ones (n_layers: there are none), whose units end a wave early (leaves != 0) where the first wave alone reads the
// roots.
// LISTED: the leaf layer goes through a list of variables (leaf_list).  (A kernel of its own: the test for a list costs the others 0.4 us of 34, 85000
// nodes at B = 128.)
template <int CT, bool LISTED>
__global__ __launch_bounds__(kColThreads) void col_fwd_kernel(const ColLayer* __restrict__ first, int n_layers, int first_is_and,
                                                              const Line* __restrict__ blocks, int n_blocks, const Desc* __restrict__ tables,
                                                              const Line* __restrict__ units, int n_units, int wide, int leaves,
                                                              const float* __restrict__ start, int start_rows, int start_T, const int32_t* __restrict__ start_map,
                                                              int B, int ld, int semiring, int size0, float* __restrict__ tb, int T,
                                                              SlabLeaf leaf, const int32_t* __restrict__ root_pos, int R,
                                                              float* __restrict__ out) {
    using V = typename ColValue<CT>::T;
    extern __shared__ float smem[];
    V* below = reinterpret_cast<V*>(smem);
    V* here = below + size0;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int col0 = (int)blockIdx.x * CT, columns = B - col0 < CT ? B - col0 : CT;      // (a column that is not there repeats the last one)
    const bool log_domain = semiring != 0;
    ColWalk walk;
    if (wide > 0) walk.start(blocks + (size_t)first->fwd_block[wave] * 128 + lane, tables + (size_t)first->fwd_table[wave] * kDescTable + lane);
    const int root = leaves ? lane : (int)threadIdx.x, root_step = leaves ? 64 : kColThreads;
    const int root_at = root < R ? root_pos[root] : 0;               // (asked for early: far away at the end)
    if (threadIdx.x < 2) {
        // identities of the two kinds of layers, in the slots that padding names
        V* a = threadIdx.x == 0 ? below : here;
        a[kColPadAnd] = V(log_domain ? 0.0f : 1.0f);
        a[kColPadOr] = V(log_domain ? -INFINITY : 0.0f);
    }
    if (leaf.w) {
        // Leaf layer into LDS, by variable (by row the weight would be asked for only when the row's literal has arrived); the transposed weights and the rows of layer 0 also go to global memory
        // for the reverse sweep (every column of [0, ld): the last workgroup zeroes the padding columns)
        auto put = [&](int row, int c, float x) {
            reinterpret_cast<float*>(below + kColSlots + row)[c] = x;
            if (!tb || c >= columns) return;
            leaf.act0[(size_t)row * ld + col0 + c] = x;
            if (col0 + c == B - 1)
                for (int b = B; b < ld; ++b) leaf.act0[(size_t)row * ld + b] = 0.0f;
        };
        const int n_vars = LISTED ? (int)(leaf.neg_row - leaf.pos_row) : leaf.V;
        for (int i = threadIdx.x; i < n_vars; i += kColThreads) {
            const int pr = leaf.pos_row[i], nr = leaf.neg_row[i], v = LISTED ? leaf.neg_row[n_vars + i] : i;
            float x[CT], y[CT];
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const size_t at = (size_t)(col0 + (c < columns ? c : columns - 1)) * leaf.V + v;
                x[c] = leaf.w[at];
                y[c] = leaf.wneg ? leaf.wneg[at] : 0.0f;
            }
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                if (pr >= 0) put(pr, c, x[c]);
                if (nr >= 0) put(nr, c, leaf.wneg ? y[c] : log_domain ? log1mexp_f(x[c]) : 1.0f - x[c]);
                if (!tb || c >= columns) continue;
                leaf.wT[(size_t)v * ld + col0 + c] = x[c];
                if (col0 + c == B - 1)
                    for (int b = B; b < ld; ++b) leaf.wT[(size_t)v * ld + b] = 0.0f;
            }
        }
        if (threadIdx.x < CT) {
            if (leaf.true_row >= 0) put(leaf.true_row, (int)threadIdx.x, log_domain ? 0.0f : 1.0f);
            if (leaf.false_row >= 0) put(leaf.false_row, (int)threadIdx.x, log_domain ? -INFINITY : 0.0f);
        }
    } else if (start_map || start_T == 0) {
#pragma unroll 4
        for (int i = threadIdx.x; i < start_rows; i += kColThreads) {
            float* slot = reinterpret_cast<float*>(below + kColSlots + i);
            const size_t row = (size_t)(start_map ? start_map[i] : i) * ld + col0;
#pragma unroll
            for (int c = 0; c < CT; ++c) slot[c] = start[row + (c < columns ? c : columns - 1)];
        }
    } else {
        col_load<CT>(below + kColSlots, start + (size_t)col0 * start_T, ColColumns{start_T, columns}, start_rows);
    }
    float* tbc = tb ? tb + (size_t)col0 * T : nullptr;
    if (wave == kColFwdWaves) {
        // the wave that keeps the values, a layer behind the others (in a wave that computes, the wait for the next
        // lines would wait for the stores as well)
        const bool touch = gridDim.x >= 64 && wide > 0;
        ColTouch<8> blocks_ahead;
        ColTouch<2> units_ahead;
        if (touch) {
            blocks_ahead.ask(blocks, 2 * n_blocks, lane, 64);
            units_ahead.ask(units, n_units, lane, 64);
        }
        for (int t = 0; t < n_layers; ++t) {
            __syncthreads();
            if (touch && t == 0) {
                blocks_ahead.finish();
                units_ahead.finish();
            }
            if (tbc && t > 0) col_move<CT>(reinterpret_cast<const float*>(below + kColSlots), first[t - 1].n, tbc + first[t - 1].at, T, columns);
            V* tmp = below; below = here; here = tmp;
        }
    } else {
        for (int t = 0; t < wide; ++t) {
            const bool is_and = ((t & 1) == 0) == (first_is_and != 0);
            __syncthreads();
            if (is_and) {
                if (log_domain) col_fwd_layer<OP_SUM>(walk, below, here);
                else col_fwd_layer<OP_PROD>(walk, below, here);
            } else if (semiring == 1) col_fwd_layer<OP_LSE>(walk, below, here);
            else if (semiring == 2) col_fwd_layer<OP_MAX>(walk, below, here);
            else col_fwd_layer<OP_SUM>(walk, below, here);
            V* tmp = below; below = here; here = tmp;
        }
        if (wide < n_layers) {
            const Line* own = units + (size_t)first[wide].fwd_unit[wave] * 64 + lane;
            if (semiring == 1) col_fwd_units<OP_SUM, OP_LSE>(own, below, here);
            else if (semiring == 2) col_fwd_units<OP_SUM, OP_MAX>(own, below, here);
            else col_fwd_units<OP_PROD, OP_SUM>(own, below, here);
            if (leaves && wave > 0) {
                // (the barriers count the waves that are there; what this one wrote has to be in the LDS before)
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                return;
            }
        }
    }
    __syncthreads();
    if (wave == kColFwdWaves && tbc) col_move<CT>(reinterpret_cast<const float*>(below + kColSlots), first[n_layers - 1].n, tbc + first[n_layers - 1].at, T, columns);
    // roots: the top layer is in LDS
    if (leaves && wave > 0) return;
    for (int r = root; r < R; r += root_step) {
        const float* slot = reinterpret_cast<const float*>(below + kColSlots + (r == root ? root_at : root_pos[r]));
        for (int c = 0; c < columns; ++c) out[(size_t)(col0 + c) * R + r] = slot[c];
    }
}

// One step of the reverse sweep.  Log semiring, through an OR layer (LogOr): the weighted edges (bit 15 of an entry) read the
// parent's adjoint in the one-gather form (see encode_h) and need the value of the row they belong to.
// Through an AND layer (LogAnd) every edge passes the adjoint on, and a row that is an OR node with more than one child (bit 15
// of its entries) is stored in that form, again with the row's own value.
// Real semiring, through a sum layer (RealOr): plain sums, and the finished adjoint G of a product node leaves as the row P of
// prod_parent_kernel (G times the product of the other children, whichever they are; ColRepair does the rows that
// hold a zero).  Through a product layer (RealAnd): a child gets the sum of its parents' P over its own value, or, if it
// is zero, the sum of the P of those parents whose one zero it is (see OP_PROD_BWD; one quotient per row here).
// own: the values of the rows by slot; it may be the array the adjoints go to (a slot is read by the lanes of its row only).
enum ColMode { kLogAnd, kLogOr, kRealOr, kRealAnd };

// what a row's parents pass down: the sum (RealAnd: of the parents without a zero child, and of those with exactly one).
// Sums are balanced over the entries of a line and the two lines of a block: shorter chains and fewer roundings than one
// entry after another.
template <int MODE, class V> struct ColSum {
    V a = V(0.0f), b = V(0.0f);
};
template <int MODE, class V>
__device__ __forceinline__ ColSum<MODE, V> operator+(const ColSum<MODE, V>& x, const ColSum<MODE, V>& y) {
    if constexpr (MODE == kRealAnd) return {x.a + y.a, x.b + y.b};
    else return {x.a + y.a, x.b};
}
template <int MODE, class V>
__device__ __forceinline__ ColSum<MODE, V> col_entry(const V* above, uint32_t e, V own) {
    const V g = col_at(above, e & 0x7FFFu);
    if constexpr (MODE == kRealAnd)
        return {each([](float x) { return __float_as_uint(x) & 1u ? 0.0f : x; }, g),
                each([](float x) { return __float_as_uint(x) & 1u ? __uint_as_float(__float_as_uint(x) & ~1u) : 0.0f; }, g)};
    else return {MODE == kLogOr && (e & 0x8000u) ? each([](float x, float y) { return decode_h(x, y); }, g, own) : g, V(0.0f)};
}
template <int MODE, class V>
__device__ __forceinline__ ColSum<MODE, V> col_pair(const V* above, uint32_t w, V own) {
    return col_entry<MODE>(above, w & 0xFFFFu, own) + col_entry<MODE>(above, w >> 16, own);
}
template <int MODE, class V>
__device__ __forceinline__ ColSum<MODE, V> col_line(const V* above, Line w, V own) {
    return (col_pair<MODE>(above, w.x, own) + col_pair<MODE>(above, w.y, own)) + (col_pair<MODE>(above, w.z, own) + col_pair<MODE>(above, w.w, own));
}

// Product rows that hold a zero: the product of a row's non-zero children and how many are zero, per column, from the
// node values (rare, so straight from global memory).
struct ColRepair {
    const int32_t *ptr, *child;       // index vectors of the layer, by parent
    const float* values;              // values of the layer below, first column; child c of column i at values[c * by_child + i * by_column]
    size_t by_child, by_column;
    int last;                         // column (one past it: that one again)
    __device__ __forceinline__ float row(float g, float own, int r, int column) const {
        if (own != 0.0f) return premultiply(g, own);
        if (column > last) column = last;
        float q = 1.0f;
        int zeros = 0;
        for (int j = ptr[r]; j < ptr[r + 1]; ++j) {
            const float x = values[(size_t)child[j] * by_child + column * by_column];
            if (x == 0.0f) ++zeros;
            else q *= x;
        }
        const float p = zeros >= 2 ? 0.0f : g * q;
        return __uint_as_float((__float_as_uint(p) & ~1u) | (zeros == 1 ? 1u : 0u));
    }
};

// what a row leaves; r: its position in the layer
template <int MODE, class V>
__device__ __forceinline__ V col_finish(const ColSum<MODE, V>& s, V own, bool flagged, const ColRepair& repair, int r) {
    if constexpr (MODE == kLogAnd) return flagged ? each([](float a, float b) { return encode_h(a, b); }, s.a, own) : s.a;
    else if constexpr (MODE == kRealAnd) return each([](float a, float b, float n) { return n != 0.0f ? a / n : b; }, s.a, s.b, own);
    else if constexpr (MODE == kRealOr) {
        if constexpr (sizeof(V) == sizeof(float)) {
            return repair.row(s.a, own, r, 0);
        } else {
            V p;
#pragma unroll
            for (int c = 0; c < (int)(sizeof(V) / sizeof(float)); ++c) p[c] = repair.row(s.a[c], own[c], r, c);
            return p;
        }
    } else return s.a;
}

// a quarter of a block (FULL: all its rows are there); r: position of the lane's first row
template <int MODE, int KIND, bool FULL, class V>
__device__ __forceinline__ void col_bwd_quarter(const V* above, uint32_t a, uint32_t b, const V* own_at, V* out, int rows,
                                                const ColRepair& repair, int r) {
    constexpr int N = 4 >> KIND;
    const int lane = threadIdx.x & 63;
    V own[N];
    ColSum<MODE, V> v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) own[i] = own_at[FULL || lane + 64 * i < rows ? 64 * i : -lane];
    const uint32_t e[4] = {a & 0xFFFFu, a >> 16, b & 0xFFFFu, b >> 16};
    if constexpr (KIND == 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = col_entry<MODE>(above, e[i], own[i]);
    } else if constexpr (KIND == 1) {
        v[0] = col_pair<MODE>(above, a, own[0]);
        v[1] = col_pair<MODE>(above, b, own[1]);
    } else {
        v[0] = col_pair<MODE>(above, a, own[0]) + col_pair<MODE>(above, b, own[0]);
    }
#pragma unroll
    for (int i = 0; i < N; ++i)
        if (FULL || lane + 64 * i < rows) out[64 * i] = col_finish<MODE>(v[i], own[i], (e[i << KIND] & 0x8000u) != 0, repair, r + 64 * i);
}

// a run of kind 0, 1 or 2, from position r of the layer on
template <int MODE, int KIND, class V>
__device__ __forceinline__ void col_bwd_short(ColWalk& walk, const V* above, const V* own_at, V* out, int rows, const ColRepair& repair, int r) {
    constexpr int N = 4 >> KIND;
    const int lane = threadIdx.x & 63;
    out += lane;
    own_at += lane;
    r += lane;
    Line w0, w1;
    for (; rows >= 256 * N; rows -= 256 * N, out += 256 * N, own_at += 256 * N, r += 256 * N) {
        walk.block(w0, w1);
        col_bwd_quarter<MODE, KIND, true>(above, w0.x, w0.y, own_at, out, 0, repair, r);
        col_bwd_quarter<MODE, KIND, true>(above, w0.z, w0.w, own_at + 64 * N, out + 64 * N, 0, repair, r + 64 * N);
        col_bwd_quarter<MODE, KIND, true>(above, w1.x, w1.y, own_at + 128 * N, out + 128 * N, 0, repair, r + 128 * N);
        col_bwd_quarter<MODE, KIND, true>(above, w1.z, w1.w, own_at + 192 * N, out + 192 * N, 0, repair, r + 192 * N);
    }
    if (rows > 0) {
        walk.block(w0, w1);
        col_bwd_quarter<MODE, KIND, false>(above, w0.x, w0.y, own_at, out, rows, repair, r);
        if (rows > 64 * N) col_bwd_quarter<MODE, KIND, false>(above, w0.z, w0.w, own_at + 64 * N, out + 64 * N, rows - 64 * N, repair, r + 64 * N);
        if (rows > 128 * N) {
            col_bwd_quarter<MODE, KIND, false>(above, w1.x, w1.y, own_at + 128 * N, out + 128 * N, rows - 128 * N, repair, r + 128 * N);
            if (rows > 192 * N) col_bwd_quarter<MODE, KIND, false>(above, w1.z, w1.w, own_at + 192 * N, out + 192 * N, rows - 192 * N, repair, r + 192 * N);
        }
    }
}

template <int MODE, class V>
__device__ __forceinline__ void col_bwd_layer(ColWalk& walk, const V* above, V* here, const V* owns, const ColRepair& repair) {
    const int lane = threadIdx.x & 63;
    Desc table = walk.table();
    ColRun run;
    for (int i = 0; run.read(walk, table, i);) {
        V* out = here + run.slot;
        const V* own_at = owns + run.slot;
        int first = run.slot - kColSlots;
        if (run.kind == 0) col_bwd_short<MODE, 0>(walk, above, own_at, out, run.rows, repair, first);
        else if (run.kind == 1) col_bwd_short<MODE, 1>(walk, above, own_at, out, run.rows, repair, first);
        else if (run.kind == 2) col_bwd_short<MODE, 2>(walk, above, own_at, out, run.rows, repair, first);
        else {
            const int r = lane >> run.k, per = 64 >> run.k;
            const bool writes = (lane & ((1 << run.k) - 1)) == 0;
            for (int rows = run.rows; rows > 0; rows -= per, out += per, own_at += per, first += per) {
                const V own = own_at[r < rows ? r : 0];
                Line w0, w1;
                walk.block(w0, w1);
                const bool flagged = (w0.x & 0x8000u) != 0;
                ColSum<MODE, V> acc = col_line<MODE>(above, w0, own);
                if (run.kind == 3) {
                    acc = acc + col_line<MODE>(above, w1, own);
                    for (int b = 1; b < run.blocks; ++b) {
                        walk.block(w0, w1);
                        acc = acc + (col_line<MODE>(above, w0, own) + col_line<MODE>(above, w1, own));
                    }
                }
                acc.a = col_fly<OP_SUM>(acc.a, run.k);
                if (MODE == kRealAnd) acc.b = col_fly<OP_SUM>(acc.b, run.k);
                if (writes && r < rows) out[r] = col_finish<MODE>(acc, own, flagged, repair, first + r);
            }
        }
    }
}

// The same for a unit of a narrow layer; own: the values of the rows by slot
template <int MODE, class V>
__device__ __forceinline__ void col_bwd_row(const V* above, V* here, const V* owns, Line w, uint32_t head, const ColRepair& repair) {
    const uint32_t slot = w.x & kUnitSlot;
    const int lanes = (int)(w.x >> kUnitLanesAt) & 7, k = (int)(head >> kUnitLanesAt) & 7;
    const V own = owns[slot];
    ColSum<MODE, V> acc = col_pair<MODE>(above, w.y, own);
    if (head & kUnitShort) {
        acc = acc + col_entry<MODE>(above, w.z & 0xFFFFu, own);
    } else {
        acc = (acc + col_pair<MODE>(above, w.z, own)) + col_pair<MODE>(above, w.w, own);
        if (k > 0) {
            acc.a = unit_fly<OP_SUM>(acc.a, lanes, k);
            if (MODE == kRealAnd) acc.b = unit_fly<OP_SUM>(acc.b, lanes, k);
        }
    }
    if (slot != kUnitIdleSlot) here[slot] = col_finish<MODE>(acc, own, (w.x & kUnitRow) != 0, repair, (int)slot - kColSlots);
}

// Where the reverse kernel leaves its last layer's adjoints: the leaf gradients themselves (w_T != null, the last
// layer is layer 0), or g_cols[B][g_T], column-major (a lane owns rows of one column, so row-major stores would be
// 4 bytes per cache line; tb_to_rows_kernel transposes afterwards).
struct ColBwdOut {
    float* g_cols;
    int32_t g_T, n_last;        // g_T: floats in a column of g_cols
    float* keep;                // TopPlan: column-major buffer, as tb, that takes the adjoints of every layer from the keep_from-th below the top one on
    int32_t keep_from;
    const float* wT;            // [V, ld] transposed leaf weights
    const int32_t *pos_row, *neg_row;
    float *dleaf, *dneg;
    int32_t V, mode;            // mode: as for leaf_bwd_kernel
};

// Real semiring only: index vectors by parent of the product layers (offsets into `index` by depth under the top layer; see
// ColRepair), and where the values below the column-major buffer are.
struct ColReal {
    const int32_t* index;
    const int32_t *ptr, *child;
    const float* rows;          // activation rows of the layer below the first one the forward kernel ran
    const float* low_rows;      // activation rows that the index vectors of that layer name
    int32_t lowest;             // its depth
};

// Reverse sweep over the same layers: seeds the top layer's adjoints from dout and walks n_steps layers
// down.  LDS: the adjoints of the layer in hand and of the one below, size0 floats for the top layer and every second
// one from there.  Node values come from the column-major buffer tb, once per row, and are far away (a read of them
// takes about 2000 cycles, three times as long as a layer of units): those of the first `cached` steps are loaded at once to
// cache_at, into LDS that only later steps use or that lies behind both arrays (launch_tail_bwd; 67000 nodes in 48 layers of
// about 1400, log training step at B = 4: 143 -> 116 us by what lies behind, 29000 nodes in 30 layers 91 -> 68); from there
// on those of the next step's rows are fetched into registers during a step (up to kColOwn times four per thread: any
// layer that fits; as many as the layer has, 116 -> 109 us there) and put into the slots of the array that the step
// frees.  (Four at a time: a load instruction of one float a lane takes the memory pipe as long.)  last_at: entry of the last layer in tb (-1: its values are not needed).  The adjoints
// of OR nodes with more than one child are kept in the one-gather form throughout, also on the way out; top_multi
// (or null) flags such nodes of the top layer for the seed.
// (tb is not __restrict__: a load known to be invariant would be moved down past the barrier to its use.)
// (two and four columns: where no layer is longer)
template <int CT> constexpr int kColOwn = CT == 1 ? (int)((kTailRowsCap + 4 * kColThreads - 1) / (4 * kColThreads)) : CT == 2 ? 3 : 1;

// narrow: so many steps from the top layer down go by units (at most 64, all of them with cached own values).
// KEEP: ColBwdOut::keep takes the adjoints of every layer, by a wave that does nothing else (see col_fwd_kernel).
template <int CT, bool REAL, bool KEEP>
__global__ __launch_bounds__(kColThreads) void col_bwd_kernel(const ColLayer* __restrict__ top, int n_steps, int last_at,
                                                              int top_is_and, const Line* __restrict__ blocks, int n_blocks,
                                                              const Desc* __restrict__ tables, const Line* __restrict__ units, int narrow,
                                                              const float* __restrict__ dout,
                                                              const int32_t* __restrict__ top_ptr, const int32_t* __restrict__ top_root,
                                                              int R, int B, int ld, int size0, int cached, int cache_at,
                                                              const float* tb, int T,
                                                              const uint32_t* __restrict__ top_multi, ColBwdOut res, ColReal real) {
    using V = typename ColValue<CT>::T;
    extern __shared__ float smem[];
    V* above = reinterpret_cast<V*>(smem);
    V* here = above + size0;
    V* const cache = above + cache_at;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int col0 = (int)blockIdx.x * CT, columns = B - col0 < CT ? B - col0 : CT;      // (a column that is not there repeats the last one)
    const float* tbc = tb + (size_t)col0 * T;
    const ColColumns column{T, columns};
    ColWalk walk;
    walk.start(blocks + (size_t)top[-narrow].bwd_block[wave] * 128 + lane, tables + (size_t)top[-narrow].bwd_table[wave] * kDescTable + lane);
    ColUnits walk_units;
    if (narrow > 0) walk_units.start(units + (size_t)top->bwd_unit[wave] * 64 + lane);
    ColTouch<2> blocks_ahead;
    if (gridDim.x >= 64) blocks_ahead.ask(blocks, 2 * n_blocks, (int)threadIdx.x, kColThreads);
    auto value_at = [&](int at) {
        if constexpr (CT == 1) {
            return tbc[at];
        } else {
            V v;
#pragma unroll
            for (int c = 0; c < CT; ++c) v[c] = tbc[column(c) + at];
            return v;
        }
    };
    // own values of the rows of step t (the t-th layer below the top one): how many and where
    auto own_of = [&](int t, int& n, int& at) {
        n = at = 0;
        if (t + 1 < n_steps) { n = top[-1 - t].n; at = top[-1 - t].at; }
        else if (t < n_steps && last_at >= 0) { n = res.n_last; at = last_at; }
    };
    if (threadIdx.x < 2) (threadIdx.x == 0 ? above : here)[kColPadAnd] = V(0.0f);       // what padding names: adjoint 0
    const int n_top = top->n, top_at = top->at;
    // how to repair the rows of the layer `depth` below the top one (a product layer)
    auto repair_of = [&](int depth) {
        ColRepair r{};
        if (REAL) {
            r.ptr = real.index + real.ptr[depth];
            r.child = real.index + real.child[depth];
            const bool stored = depth + 1 < real.lowest;       // the layer below that one is in tb, otherwise in rows
            r.values = stored ? tbc + top[-1 - depth].at : (depth < real.lowest ? real.rows : real.low_rows) + col0;
            r.by_child = stored ? 1 : (size_t)ld;
            r.by_column = stored ? (size_t)T : 1;
            r.last = columns - 1;
        }
        return r;
    };
    // the leaves' own values (real semiring; they are not in tb)
    auto leaf_values = [&](V* to) {
        for (int i = threadIdx.x; i < res.n_last; i += kColThreads) {
            const float* from = real.rows + (size_t)i * ld + col0;
#pragma unroll
            for (int c = 0; c < CT; ++c) reinterpret_cast<float*>(to + kColSlots + i)[c] = from[c < columns ? c : columns - 1];
        }
    };
    // t: depth of the one in hand under the top layer
    const bool keeper = KEEP && wave == kTopBwdWaves;
    auto keep_layer = [&](int t) {
        if (t >= res.keep_from)
            col_move<CT>(reinterpret_cast<const float*>(above + kColSlots), top[-t].n, res.keep + (size_t)col0 * T + top[-t].at, T, columns);
    };
    int cache_low = 0;
    if (cached > 0) {
        // the cached layers follow one another in tb
        cache_low = top[-cached].at;
        col_load<CT>(cache, tbc + cache_low, column, top_at - cache_low);
    } else {
        int n, at;
        own_of(0, n, at);
        for (int i = threadIdx.x; i < n; i += kColThreads) here[kColSlots + i] = value_at(at + i);
        if (REAL && n_steps == 1 && last_at < 0) leaf_values(here);
    }
    for (int i = threadIdx.x; i < n_top; i += kColThreads) {      // adjoint seed of the top layer
        V acc = V(0.0f);
        for (int t = top_ptr[i]; t < top_ptr[i + 1]; ++t) {
            const float* from = dout + (size_t)col0 * R + top_root[t];
            if constexpr (CT == 1) {
                acc += from[0];
            } else {
                V g;
#pragma unroll
                for (int c = 0; c < CT; ++c) g[c] = from[(size_t)(c < columns ? c : columns - 1) * R];
                acc += g;
            }
        }
        if (REAL && top_is_and) {
            ColSum<kRealOr, V> g;
            g.a = acc;
            acc = col_finish<kRealOr>(g, value_at(top_at + i), false, repair_of(0), i);
        }
        if (!REAL && top_multi && ((top_multi[i >> 5] >> (i & 31)) & 1u)) acc = each([](float a, float b) { return encode_h(a, b); }, acc, value_at(top_at + i));
        above[kColSlots + i] = acc;
    }
    if (gridDim.x >= 64) blocks_ahead.finish();
    int t = 0;
    if (narrow > 0) {
        if (keeper) {
            for (; t < narrow; ++t) {
                __syncthreads();
                keep_layer(t);
                V* tmp = above; above = here; here = tmp;
            }
        } else {
            // (where the own values of a step are, a lane each: scalar loads would share their wait counter with the gathers)
            const int ats = top[-1 - (lane < narrow ? lane : 0)].at;
            const V* owns = cache;
            t = -1;
            V* tmp = above; above = here; here = tmp;        // (as after a step)
            for (bool done = false; !done;) {
#pragma unroll
                for (int i = 0; i < kUnitsAhead; ++i) {
                    const Line w = walk_units.r[i];
                    const uint32_t head = (uint32_t)__builtin_amdgcn_readfirstlane((int)w.x);
                    if (head & (kUnitNew | kUnitEnd)) {
                        if (t + 1 == narrow) { done = true; break; }
                        ++t;
                        owns = cache + (__builtin_amdgcn_readlane(ats, t) - cache_low) - kColSlots;
                        __syncthreads();
                        tmp = above; above = here; here = tmp;
                    }
                    if (!(head & kUnitIdle)) {
                        if (head & kUnitOr) col_bwd_row<REAL ? kRealOr : kLogOr>(above, here, owns, w, head, REAL ? repair_of(t + 1) : ColRepair{});
                        else col_bwd_row<REAL ? kRealAnd : kLogAnd>(above, here, owns, w, head, ColRepair{});
                    }
                    walk_units.next(i);
                }
            }
            ++t;
            tmp = above; above = here; here = tmp;
        }
    }
    for (; t + 1 < cached; ++t) {
        const V* owns = cache + (top[-1 - t].at - cache_low) - kColSlots;
        __syncthreads();
        if (keeper) keep_layer(t);
        else if (((t & 1) == 0) == (top_is_and != 0)) col_bwd_layer<REAL ? kRealAnd : kLogAnd>(walk, above, here, owns, ColRepair{});
        else col_bwd_layer<REAL ? kRealOr : kLogOr>(walk, above, here, owns, repair_of(t + 1));
        V* tmp = above; above = here; here = tmp;
    }
    for (; t < n_steps; ++t) {
        int own_n, own_at;
        own_of(t + 1, own_n, own_at);
        // (the last rows are read, and written, by a lane that steps back to them; a layer of less than four rows reads
        // up to three floats past its own, still inside the workspace)
        Float4u own[kColOwn<CT>][CT];
#pragma unroll
        for (int i = 0; i < kColOwn<CT>; ++i) {
            if (4 * (wave * 64 + i * kColThreads) >= own_n) continue;      // (the same for all lanes of a wave)
            const int at = 4 * ((int)threadIdx.x + i * kColThreads), back = own_n - 4 < 0 ? 0 : own_n - 4;
            const float* from = tbc + own_at + (at < back ? at : at < own_n ? back : 0);
#pragma unroll
            for (int c = 0; c < CT; ++c) own[i][c] = *reinterpret_cast<const Float4u*>(from + column(c));
        }
        const V* owns = t < cached ? cache + (top[-1 - t].at - cache_low) - kColSlots : here;
        __syncthreads();
        if (keeper) keep_layer(t);
        else if (((t & 1) == 0) == (top_is_and != 0)) col_bwd_layer<REAL ? kRealAnd : kLogAnd>(walk, above, here, owns, ColRepair{});
        else col_bwd_layer<REAL ? kRealOr : kLogOr>(walk, above, here, owns, repair_of(t + 1));
        __syncthreads();
        // the adjoints above are done with: their array takes the next step's own values
#pragma unroll
        for (int i = 0; i < kColOwn<CT>; ++i) {
            if (4 * (wave * 64 + i * kColThreads) >= own_n) continue;
            const int at = 4 * ((int)threadIdx.x + i * kColThreads), back = own_n - 4 < 0 ? 0 : own_n - 4;
            if (at + 4 <= own_n) {
                col_put4<CT>(above + kColSlots + at, own[i]);
            } else if (at < own_n) {
                float* slot = reinterpret_cast<float*>(above + kColSlots + back);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (back + j < own_n)
#pragma unroll
                        for (int c = 0; c < CT; ++c) slot[j * CT + c] = own[i][c][j];
            }
        }
        if (REAL && t + 2 == n_steps && last_at < 0) leaf_values(above);
        V* tmp = above; above = here; here = tmp;
    }
    __syncthreads();
    const float* slots = reinterpret_cast<const float*>(above + kColSlots);
    for (int c = 0; c < columns; ++c) {
        const int col = col0 + c;
        if (!res.wT) {
            for (int r = threadIdx.x; r < res.n_last; r += kColThreads) res.g_cols[(size_t)col * res.g_T + r] = slots[r * CT + c];
            continue;
        }
        for (int v = threadIdx.x; v < res.V; v += kColThreads) {
            const int pr = res.pos_row[v], nr = res.neg_row[v];
            float d = pr >= 0 ? slots[pr * CT + c] : 0.0f, dn = 0.0f;
            if (nr >= 0) {
                const float gn = slots[nr * CT + c];
                if (res.mode == 2) dn = gn;
                else if (gn != 0.0f) d += res.mode == 1 ? -gn / expm1f(-res.wT[(size_t)v * ld + col]) : -gn;
            }
            res.dleaf[(size_t)col * res.V + v] = d;
            if (res.mode == 2 && res.dneg) res.dneg[(size_t)col * res.V + v] = dn;
        }
    }
}

// cols[b * T + r] = rows[r, b] (MAP: rows[map[r], b]) for r < n_rows, b < B: the rows of a layer of the activation buffer into the column-major
// form in which a workgroup of the persistent forward kernel reads its column (32 x 32 tiles through LDS).
template <bool MAP>
__global__ __launch_bounds__(256) void rows_to_cols_kernel(const float* __restrict__ rows, int n_rows, int B, int ld,
                                                           float* __restrict__ cols, int T, const int32_t* __restrict__ map) {
    __shared__ float tile[32][33];
    const int r0 = blockIdx.x * 32, b0 = blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;       // 32 x 8
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int r = r0 + ty + 8 * j, b = b0 + tx;
        tile[ty + 8 * j][tx] = (r < n_rows && b < B) ? rows[(size_t)(MAP ? map[r] : r) * ld + b] : 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int b = b0 + ty + 8 * j, r = r0 + tx;
        if (b < B && r < n_rows) cols[(size_t)b * T + r] = tile[tx][ty + 8 * j];
    }
}

// rows[r, b] (MAP: rows[map[r], b], where that is not negative) = tb[b, first + r] for r < n_rows: values that the persistent forward kernel left in the
// column-major buffer, transposed into rows of the activation buffer through a 32 x 33 LDS tile.
template <bool MAP>
__global__ __launch_bounds__(256) void tb_to_rows_kernel(const float* __restrict__ tb, int T, int first, int n_rows,
                                                         int B, int ld, float* __restrict__ rows, const int32_t* __restrict__ map) {
    __shared__ float tile[32][33];
    const int r0 = blockIdx.x * 32, b0 = blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;       // 32 x 8
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int b = b0 + ty + 8 * j, r = r0 + tx;
        tile[ty + 8 * j][tx] = (b < B && r < n_rows) ? tb[(size_t)b * T + first + r] : 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int r = r0 + ty + 8 * j, b = b0 + tx;
        if (r < n_rows && b < ld)
            if (const int row = MAP ? map[r] : r; row >= 0) rows[(size_t)row * ld + b] = tile[tx][ty + 8 * j];
    }
}

// ---------------------------------------------------------------------------------------------
// Reverse sweep of a product (AND) layer in the real semiring, first half.  The adjoint of child c of
// parent r is G[r] times the product of r's other children.  Per parent the kernel forms, per batch
// column, the product q of the non-zero children and the number z of zero ones, and replaces the
// parent's adjoint row in place by
//   P[r] = G[r] * q  (0 when z >= 2),  lowest mantissa bit = (z == 1),
// from which the by-child pass (OP_PROD_BWD) gives every child its share: P / value for a parent
// without zero children, P itself for the one zero child of a parent with z = 1.  Exact also when
// children are zero (leaves with p = 0 or p = 1); nothing is stored per edge.  A lane group of W lanes
// owns one parent row.
//   With `own` (the values of the parents themselves) the rows arrive premultiplied (OP_SUM_P,
// OP_PROD_BWD_P): G * value where the value is not zero, which is P already, and plain G where it is
// zero.  Then only the waves that hold a zero value walk the children, and only those columns change; that pass
// also raises zero_flag when it meets a zero value, and a launch that finds it down returns at once.
// ---------------------------------------------------------------------------------------------
template <int VEC, int W>
__global__ __launch_bounds__(256) void prod_parent_kernel(const int32_t* __restrict__ ptr,
                                                          const int32_t* __restrict__ child,
                                                          const float* __restrict__ below, float* __restrict__ g, int n,
                                                          int B, int ld, const float* __restrict__ own,
                                                          const int* __restrict__ zero_flag) {
    constexpr int RPW = 64 / W;
    const int lane = threadIdx.x & 63;
    const int col = ((int)blockIdx.y * W + (lane % W)) * VEC;
    if (col >= B) return;
    if (own && zero_flag && *zero_flag == 0) return;          // the pass that wrote the rows met no zero value: nothing to repair
    // the grid is capped (the launch that finds the flag down should cost as little as a launch can): a
    // workgroup takes every gridDim.x-th group of rows
    for (int64_t blk = blockIdx.x; blk * (4 * RPW) < n; blk += gridDim.x) {
    const int64_t row64 = (blk * 4 + (threadIdx.x >> 6)) * RPW + lane / W;
    if (row64 >= n) continue;
    const int row = (int)row64;
    float nv[VEC];
    if (own) {
        load_vec<VEC>(nv, own + (size_t)row * ld + col);
        bool zero_here = false;
#pragma unroll
        for (int v = 0; v < VEC; ++v) zero_here = zero_here || nv[v] == 0.0f;
        if (!__any(zero_here)) continue;
    }
    const int beg = ptr[row], end = ptr[row + 1];
    float q[VEC], z[VEC], gr[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) { q[v] = 1.0f; z[v] = 0.0f; }
    load_vec<VEC>(gr, g + (size_t)row * ld + col);
    constexpr int CH = 8;
    float x[CH][VEC];
    // 8 gathers in flight (entries past the row's end re-read its last child)
    for (int j = beg; j < end; j += CH) {
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int jj = j + i < end ? j + i : end - 1;
            load_vec<VEC>(x[i], below + (size_t)child[jj] * ld + col);
        }
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const bool live = j + i < end;
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                const bool zero = x[i][v] == 0.0f;
                z[v] += (live && zero) ? 1.0f : 0.0f;
                q[v] *= (live && !zero) ? x[i][v] : 1.0f;
            }
        }
    }
    float p[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
        const float val = z[v] >= 2.0f ? 0.0f : gr[v] * q[v];
        p[v] = __uint_as_float((__float_as_uint(val) & ~1u) | (z[v] == 1.0f ? 1u : 0u));
        if (own && nv[v] != 0.0f) p[v] = gr[v];          // premultiplied already
    }
    store_vec<VEC>(g + (size_t)row * ld + col, p);
    }
}

// ---------------------------------------------------------------------------------------------
// Leaf layer: leaf_weights[B,V] (batch-outer) -> wT[V,ld] (kept for the backward pass) and the
// literal rows of layer 0, through an LDS tile of 32 variables x 64 batch columns.  The negated
// literal of v gets wneg[b, v] when the caller supplies weights of its own for the negated literals,
// otherwise 1 - w (real semiring) or log(1 - exp(w)) (log domain).
//   16 waves per tile: there are few tiles (128 of them for 1024 variables and 256 columns), and what a wave does for a
// variable (its rows, a library logarithm and exponential, the stores) takes about a microsecond.  Four waves of eight variables
// each took 11.4 us there (now 5.7), and the leaf gradients 12.4 (5.0).
// ---------------------------------------------------------------------------------------------
constexpr int kLeafThreads = 1024;
__global__ __launch_bounds__(kLeafThreads) void leaf_fwd_kernel(const float* __restrict__ w, const float* __restrict__ wneg,
                                                       int B, int V, int ld,
                                                       const int32_t* __restrict__ pos_row,
                                                       const int32_t* __restrict__ neg_row,
                                                       float* __restrict__ wT, float* __restrict__ act0,
                                                       int log_domain) {
    __shared__ float tile[32][65];
    __shared__ float tile_neg[32][65];
    const int v0 = blockIdx.x * 32, b0 = blockIdx.y * 64;
    {
        const int vx = threadIdx.x & 31, by = threadIdx.x >> 5;
#pragma unroll
        for (int k = 0; k < 64; k += kLeafThreads / 32) {
            const int b = b0 + by + k, v = v0 + vx;
            const bool in = b < B && v < V;
            tile[vx][by + k] = in ? w[(size_t)b * V + v] : 0.0f;
            if (wneg) tile_neg[vx][by + k] = in ? wneg[(size_t)b * V + v] : 0.0f;
        }
    }
    __syncthreads();
    const int bx = threadIdx.x & 63, vy = threadIdx.x >> 6;
    const int b = b0 + bx;
    if (b >= ld) return;
#pragma unroll
    for (int k = 0; k < 32; k += kLeafThreads / 64) {
        const int v = v0 + vy + k;
        if (v >= V) break;
        const float x = tile[vy + k][bx];
        wT[(size_t)v * ld + b] = x;
        const int pr = pos_row[v], nr = neg_row[v];
        if (pr >= 0) act0[(size_t)pr * ld + b] = x;
        if (nr >= 0) {
            float y;
            if (b >= B) y = 0.0f;
            else if (wneg) y = tile_neg[vy + k][bx];
            else y = log_domain ? log1mexp_f(x) : 1.0f - x;
            act0[(size_t)nr * ld + b] = y;
        }
    }
}

// The same for small batches (ld = B <= 32), where the tile would be all but empty: a thread per (variable, column).
__global__ __launch_bounds__(256) void leaf_fwd_small_kernel(const float* __restrict__ w, const float* __restrict__ wneg,
                                                             int B, int V, const int32_t* __restrict__ pos_row,
                                                             const int32_t* __restrict__ neg_row,
                                                             float* __restrict__ wT, float* __restrict__ act0,
                                                             int log_domain) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)V * B) return;
    const int v = (int)(i / B), b = (int)(i % B);
    const float x = w[(size_t)b * V + v];
    wT[i] = x;
    const int pr = pos_row[v], nr = neg_row[v];
    if (pr >= 0) act0[(size_t)pr * B + b] = x;
    if (nr >= 0) act0[(size_t)nr * B + b] = wneg ? wneg[(size_t)b * V + v] : (log_domain ? log1mexp_f(x) : 1.0f - x);
}

__global__ void fill_row_kernel(float* row, int ld, float value) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < ld) row[b] = value;
}

// out[b, r] = top[root_pos[r], b]
__global__ void root_out_kernel(const float* __restrict__ top, const int32_t* __restrict__ root_pos,
                                int B, int R, int ld, float* __restrict__ out) {
    const int r = blockIdx.x;
    const float* row = top + (size_t)root_pos[r] * ld;
    for (int b = threadIdx.x; b < B; b += blockDim.x) out[(size_t)b * R + r] = row[b];
}

// G_top[i, b] = sum of dout[b, r] over the root columns r that read top-layer node i
// multi (or null) with the top layer's values: nodes flagged there leave in the one-gather form (encode_h)
__global__ void seed_kernel(const float* __restrict__ dout, const int32_t* __restrict__ top_ptr,
                            const int32_t* __restrict__ top_root, int B, int R, int ld,
                            float* __restrict__ g, const uint32_t* __restrict__ multi,
                            const float* __restrict__ top_values) {
    const int i = blockIdx.x;
    const bool enc = multi && ((multi[i >> 5] >> (i & 31)) & 1u);
    for (int b = threadIdx.x; b < ld; b += blockDim.x) {
        float acc = 0.0f;
        if (b < B)
            for (int t = top_ptr[i]; t < top_ptr[i + 1]; ++t) acc += dout[(size_t)b * R + top_root[t]];
        if (enc) acc = encode_h(acc, top_values[(size_t)i * ld + b]);
        g[(size_t)i * ld + b] = acc;
    }
}

// rows[r, b] = dout[b, r]: the adjoint seed as one row per root column
__global__ void seed_rows_kernel(const float* __restrict__ dout, int B, int R, int ld, float* __restrict__ rows) {
    const int r = blockIdx.x;
    for (int b = threadIdx.x; b < ld; b += blockDim.x) rows[(size_t)r * ld + b] = b < B ? dout[(size_t)b * R + r] : 0.0f;
}

// dleaf[b, v] = G0[+v, b] + G0[-v, b] * d(negated weight)/d(weight); tile transposed through LDS.
// mode 0: negated weight 1 - w, mode 1: log(1 - exp(w)), mode 2: the negated literals have weights
// of their own, so dleaf holds G0[+v, b] and dneg (may be null) receives G0[-v, b].
__global__ __launch_bounds__(kLeafThreads) void leaf_bwd_kernel(const float* __restrict__ g0, const float* __restrict__ wT,
                                                       const int32_t* __restrict__ pos_row,
                                                       const int32_t* __restrict__ neg_row, int B, int V,
                                                       int ld, int mode, float* __restrict__ dleaf,
                                                       float* __restrict__ dneg) {
    __shared__ float tile[32][65];
    __shared__ float tile_neg[32][65];
    const int v0 = blockIdx.x * 32, b0 = blockIdx.y * 64;
    {
        const int bx = threadIdx.x & 63, vy = threadIdx.x >> 6;
        const int b = b0 + bx;
#pragma unroll
        for (int k = 0; k < 32; k += kLeafThreads / 64) {
            const int v = v0 + vy + k;
            float d = 0.0f, dn = 0.0f;
            if (v < V && b < B) {
                const int pr = pos_row[v], nr = neg_row[v];
                if (pr >= 0) d = g0[(size_t)pr * ld + b];
                if (nr >= 0) {
                    const float gn = g0[(size_t)nr * ld + b];
                    if (mode == 2) dn = gn;
                    else if (gn != 0.0f) d += mode == 1 ? -gn / expm1f(-wT[(size_t)v * ld + b]) : -gn;
                }
            }
            tile[vy + k][bx] = d;
            tile_neg[vy + k][bx] = dn;
        }
    }
    __syncthreads();
    const int vx = threadIdx.x & 31, by = threadIdx.x >> 5;
#pragma unroll
    for (int k = 0; k < 64; k += kLeafThreads / 32) {
        const int b = b0 + by + k, v = v0 + vx;
        if (b < B && v < V) {
            dleaf[(size_t)b * V + v] = tile[vx][by + k];
            if (mode == 2 && dneg) dneg[(size_t)b * V + v] = tile_neg[vx][by + k];
        }
    }
}

}  // namespace klay
