// Double-precision evaluation of the same launch plans (accuracy build): one generic gather-reduce
// kernel, one or two batch columns per lane and as many rows per wave as that leaves room for, plus the small leaf / root / seed
// kernels.  Same index arrays, same order of layers and the same split-row scheme as the fp32
// kernels (paper Section 4, Alg. 1 / Appendix C, Alg. 4); exp and log are the full-precision
// library routines.  The rows are twice as long as in fp32 and OR layers pay a double-precision
// exponential per edge.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "klay_kernels.hip.h"

namespace klay {
namespace f64 {

struct PassArgs {
    const int32_t* ptr;        // [n_total + 1] CSR offsets into idx
    const uint32_t* idx;       // index entries (readable up to 16 entries past the end)
    const double* src;         // [*, ld] source rows
    const double* src2;        // OP_SOFTMAX_BWD: values of the parents, same row index as src
    const double* own;         // OP_SOFTMAX_BWD: values of the output rows
    const int32_t* seg_owner;  // output row owning segment i (rows >= n_main), may be null
    const int32_t* out_row;    // optional output row map for rows < n_main (combine pass)
    double* dst;               // output rows for rows < n_main
    double* dst_seg;           // scratch rows for rows >= n_main
    int32_t n_main;
    int32_t n_total;
    int32_t B;
    int32_t ld;
    int32_t lanes, per_wave;   // lanes per row, rows per wave
    uint32_t inverse;          // see lane_group
};

template <int OP>
__device__ __forceinline__ double identity() { return OP == OP_PROD ? 1.0 : (OP == OP_MAX ? -INFINITY : 0.0); }

// same streaming forms as the fp32 accumulate: (mx, acc) = (running max, sum of exp(x - mx))
template <int OP>
__device__ __forceinline__ void accumulate(double& acc, double& mx, double x, double y, double nc, bool weighted) {
    if (OP == OP_PROD_BWD) {       // as the fp32 form: x is an AND parent's P row (lowest bit: one zero child)
        const unsigned long long bits = (unsigned long long)__double_as_longlong(x);
        const double val = __longlong_as_double((long long)(bits & ~1ull));
        const bool one_zero = (bits & 1ull) != 0;
        const double part = one_zero ? (nc == 0.0 ? val : 0.0) : (nc != 0.0 ? val / nc : 0.0);
        acc += weighted ? x : part;
        return;
    }
    if (OP == OP_SUM) acc += x;
    else if (OP == OP_PROD) acc *= x;
    else if (OP == OP_MAX) acc = fmax(acc, x);
    else if (OP == OP_LSE) {
        const double d = x - mx;
        const double e = (x == -INFINITY) ? 0.0 : exp(-fabs(d));
        acc = (d > 0.0) ? fma(acc, e, 1.0) : acc + e;
        mx = fmax(mx, x);
    } else {
        const double wgt = !weighted ? 1.0 : ((y == -INFINITY) ? 0.0 : exp(nc - y));
        acc = fma(x, wgt, acc);
    }
}

template <int OP>
__device__ __forceinline__ double finish(double acc, double mx) {
    if (OP == OP_LSE) return (mx == -INFINITY) ? -INFINITY : mx + log(acc);
    return acc;
}

template <int VEC>
__device__ __forceinline__ void load_cols(double (&x)[VEC], const double* p) {
    if (VEC == 2) {
        typedef double v2 __attribute__((ext_vector_type(2), aligned(8)));
        const v2 t = *reinterpret_cast<const v2*>(p);
        x[0] = t.x;
        x[VEC - 1] = t.y;
    } else {
        x[0] = *p;
    }
}

// As the fp32 generic kernel: a group of a.lanes lanes per row, VEC batch columns per lane (launch_pass64 chooses; the last
// lane of an odd batch shares a column with its neighbour), offsets and entries in wide loads, four gathers in flight and,
// but for OP_SOFTMAX_BWD, four more where a row of the wave is that long.  Workgroups take the rows in turn over the XCDs (a contiguous eighth
// each, as in the fp32 kernels, leaves the longest rows to one XCD where rows are sorted by length: 37000 nodes at B = 258
// 163 against 130 us, 322000 nodes, training step at B = 395 2522 against 2243).
//   ONE: a wave has one row (more than half of its lanes), so offsets and entries are the same for all lanes and come by
// scalar loads.
template <int OP, int VEC, bool ONE>
__global__ __launch_bounds__(256) void pass_kernel(PassArgs a) {
    constexpr bool TWO = OP != OP_SOFTMAX_BWD;        // (two values per entry: four entries are enough registers)
    constexpr int STEP = TWO ? 8 : 4;
    int sub, colu;
    if (!lane_group(a, VEC, sub, colu)) return;
    const int col = colu <= a.B - VEC ? colu : a.B - VEC;
    const int wave = ONE ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : (int)(threadIdx.x >> 6);
    const int64_t row64 = ((int64_t)blockIdx.x * 4 + wave) * (ONE ? 1 : a.per_wave) + (ONE ? 0 : sub);
    if (row64 >= a.n_total) return;
    const int row = (int)row64;
    const Offsets2 range = *reinterpret_cast<const Offsets2*>(a.ptr + row);
    const int end = range.y;
    int j = range.x;
    Entries4 e0 = *reinterpret_cast<const Entries4*>(a.idx + j), e1 = *reinterpret_cast<const Entries4*>(a.idx + j + 4);
    if (e0.x == kSkip) return;                        // split row: evaluated by segments + combine
    double nc[VEC], acc[VEC], mx[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) { nc[v] = 0.0; acc[v] = identity<OP>(); mx[v] = -INFINITY; }
    if (OP == OP_SOFTMAX_BWD || OP == OP_PROD_BWD) {
        const int owner = row < a.n_main ? row : a.seg_owner[row - a.n_main];
        load_cols<VEC>(nc, a.own + (size_t)owner * a.ld + col);
    }
    for (;;) {
        double x0[4][VEC], x1[4][VEC], y0[4][VEC], y1[4][VEC];
        // entries past the row's end are valid entries of later rows (or zero padding): the gathers
        // are issued unconditionally and their data ignored
        auto gather = [&](Entries4 e, double (&x)[4][VEC], double (&y)[4][VEC]) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const size_t off = (size_t)(e[i] == kSkip ? 0u : e[i] & kIdMask) * a.ld + col;
                load_cols<VEC>(x[i], a.src + off);
                if (OP == OP_SOFTMAX_BWD) load_cols<VEC>(y[i], ((e[i] & kWeighted) ? a.src2 : a.src) + off);
            }
        };
        auto take = [&](Entries4 e, const double (&x)[4][VEC], const double (&y)[4][VEC], int live) {
            if (live <= 0) return;
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                if (OP == OP_LSE) {
                    // one maximum and one exponential per entry, four independent ones at a time
                    const double v0 = x[0][v], v1 = live > 1 ? x[1][v] : -INFINITY, v2 = live > 2 ? x[2][v] : -INFINITY,
                                 v3 = live > 3 ? x[3][v] : -INFINITY;
                    const double hi = fmax(fmax(fmax(v0, v1), fmax(v2, v3)), mx[v]);
                    const double m = fmin(fmax(hi, -1.7976931348623157e308), 1.7976931348623157e308);      // finite: no inf - inf
                    double t = (exp(v0 - m) + exp(v1 - m)) + (exp(v2 - m) + exp(v3 - m));
                    if (mx[v] != -INFINITY) t = fma(acc[v], exp(mx[v] - m), t);
                    acc[v] = t;
                    mx[v] = m;
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const double dead = OP == OP_PROD ? 1.0 : (OP == OP_MAX ? -INFINITY : 0.0);
                        accumulate<OP>(acc[v], mx[v], i < live ? x[i][v] : dead,
                                       OP == OP_SOFTMAX_BWD ? (i < live ? y[i][v] : -INFINITY) : 0.0, nc[v], (e[i] & kWeighted) != 0);
                    }
                }
            }
        };
        const bool second = TWO && (ONE ? j + 4 < end : __any(j + 4 < end)), more = ONE ? j + STEP < end : __any(j + STEP < end);
        Entries4 n0 = e0, n1 = e1;
        gather(e0, x0, y0);
        if (second) gather(e1, x1, y1);
        if (more) {
            const int at = j + STEP < end ? j + STEP : range.x;        // (a row that has ended reads its first entries again)
            n0 = *reinterpret_cast<const Entries4*>(a.idx + at);
            if (TWO) n1 = *reinterpret_cast<const Entries4*>(a.idx + at + 4);
        }
        take(e0, x0, y0, end - j);
        if (second) take(e1, x1, y1, end - j - 4);
        j += STEP;
        if (!more) break;
        e0 = n0;
        e1 = n1;
    }
    double* out;
    if (row < a.n_main) out = a.dst + (size_t)(a.out_row ? a.out_row[row] : row) * a.ld + col;
    else out = a.dst_seg + (size_t)(row - a.n_main) * a.ld + col;
    double o[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
        // (a row with nothing above -inf is -inf, also with a NaN among its children, which any other row passes on)
        if (OP == OP_LSE) o[v] = mx[v] == -1.7976931348623157e308 || mx[v] == -INFINITY ? -INFINITY : mx[v] + log(acc[v]);
        else o[v] = finish<OP>(acc[v], mx[v]);
    }
    if (VEC == 2) {
        typedef double v2 __attribute__((ext_vector_type(2), aligned(8)));
        *reinterpret_cast<v2*>(out) = v2{o[0], o[VEC - 1]};
    } else {
        *out = o[0];
    }
}

__device__ __forceinline__ double log1mexp(double x) {
    return x > -0.6931471805599453 ? log(-expm1(x)) : log1p(-exp(x));
}

// leaf layer: thread per (variable, batch column); negated literal as in the fp32 kernel
__global__ void leaf_fwd_kernel(const double* __restrict__ w, const double* __restrict__ wneg, int B, int V, int ld,
                                const int32_t* __restrict__ pos_row, const int32_t* __restrict__ neg_row,
                                double* __restrict__ wT, double* __restrict__ act0, int log_domain) {
    const int b = blockIdx.y * blockDim.x + threadIdx.x;
    const int v = blockIdx.x;
    if (b >= ld) return;
    const double x = b < B ? w[(size_t)b * V + v] : 0.0;
    wT[(size_t)v * ld + b] = x;
    const int pr = pos_row[v], nr = neg_row[v];
    if (pr >= 0) act0[(size_t)pr * ld + b] = x;
    if (nr >= 0) {
        double y;
        if (b >= B) y = 0.0;
        else if (wneg) y = wneg[(size_t)b * V + v];
        else y = log_domain ? log1mexp(x) : 1.0 - x;
        act0[(size_t)nr * ld + b] = y;
    }
}

__global__ void fill_row_kernel(double* row, int ld, double value) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < ld) row[b] = value;
}

__global__ void root_out_kernel(const double* __restrict__ top, const int32_t* __restrict__ root_pos, int B, int R,
                                int ld, double* __restrict__ out) {
    const int r = blockIdx.x;
    const double* row = top + (size_t)root_pos[r] * ld;
    for (int b = threadIdx.x; b < B; b += blockDim.x) out[(size_t)b * R + r] = row[b];
}

__global__ void seed_kernel(const double* __restrict__ dout, const int32_t* __restrict__ top_ptr,
                            const int32_t* __restrict__ top_root, int B, int R, int ld, double* __restrict__ g) {
    const int i = blockIdx.x;
    for (int b = threadIdx.x; b < ld; b += blockDim.x) {
        double acc = 0.0;
        if (b < B)
            for (int t = top_ptr[i]; t < top_ptr[i + 1]; ++t) acc += dout[(size_t)b * R + top_root[t]];
        g[(size_t)i * ld + b] = acc;
    }
}

__global__ void seed_rows_kernel(const double* __restrict__ dout, int B, int R, int ld, double* __restrict__ rows) {
    const int r = blockIdx.x;
    for (int b = threadIdx.x; b < ld; b += blockDim.x) rows[(size_t)r * ld + b] = b < B ? dout[(size_t)b * R + r] : 0.0;
}

// Real-semiring reverse sweep of a product layer, first half, as the fp32 kernel of the same name: the
// adjoint row of every AND parent is replaced in place by P = G * (product of the non-zero children),
// 0 with two or more zero children, lowest mantissa bit = exactly one zero child.  A wave per parent
// row, a lane per batch column.
__global__ __launch_bounds__(256) void prod_parent_kernel(const int32_t* __restrict__ ptr, const int32_t* __restrict__ child,
                                                          const double* __restrict__ below, double* __restrict__ g,
                                                          int n, int B, int ld) {
    const int lane = threadIdx.x & 63;
    const int col = (int)blockIdx.y * 64 + lane;
    if (col >= B) return;
    const int64_t row64 = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row64 >= n) return;
    const int row = (int)row64;
    const int beg = ptr[row], end = ptr[row + 1];
    double q = 1.0;
    int z = 0;
    for (int j = beg; j < end; ++j) {
        const double x = below[(size_t)child[j] * ld + col];
        if (x == 0.0) ++z;
        else q *= x;
    }
    const double val = z >= 2 ? 0.0 : g[(size_t)row * ld + col] * q;
    const unsigned long long bits = ((unsigned long long)__double_as_longlong(val) & ~1ull) | (z == 1 ? 1ull : 0ull);
    g[(size_t)row * ld + col] = __longlong_as_double((long long)bits);
}

// mode 0: negated weight 1 - w; mode 1: log(1 - exp(w)); mode 2: the negated literals have weights of their own
__global__ void leaf_bwd_kernel(const double* __restrict__ g0, const double* __restrict__ wT,
                                const int32_t* __restrict__ pos_row, const int32_t* __restrict__ neg_row, int B,
                                int V, int ld, int mode, double* __restrict__ dleaf, double* __restrict__ dneg) {
    const int b = blockIdx.y * blockDim.x + threadIdx.x;
    const int v = blockIdx.x;
    if (b >= B) return;
    const int pr = pos_row[v], nr = neg_row[v];
    double d = 0.0, dn = 0.0;
    if (pr >= 0) d = g0[(size_t)pr * ld + b];
    if (nr >= 0) {
        const double gn = g0[(size_t)nr * ld + b];
        if (mode == 2) dn = gn;
        else if (gn != 0.0) d += mode == 1 ? -gn / expm1(-wT[(size_t)v * ld + b]) : -gn;
    }
    dleaf[(size_t)b * V + v] = d;
    if (mode == 2 && dneg) dneg[(size_t)b * V + v] = dn;
}

}  // namespace f64
}  // namespace klay
