// Double-precision evaluation of the same launch plans (accuracy build): one generic gather-reduce
// kernel, one or two batch columns per lane and as many rows per wave as that leaves room for, persistent kernels for the narrow
// layers, plus the small leaf / root / seed kernels.  Same index arrays, same order of layers and the same split-row scheme as the fp32
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
// scalar loads, and so does the number of entries that are left: no exponential is taken for those past the end of a row of softmax terms (a library
// exponential is about forty instructions), nor, SHORT, of logsumexp terms, where a row of two takes one.  SHORT where the rows of the launch have at
// most kShortRows64 entries on average, since the branches cost longer rows more than they save (forward, us, always four / SHORT: 85000 nodes, 3.5
// entries a row, B = 33 81.6 / 80.4, B = 130 145.9 / 141.4; 160000 nodes of 5.3, B = 33 140.3 / 140.0; power-law fan-ins, 8 and 12 a row, B = 40
// 234.0 / 244.8 and 359.3 / 376.0).
template <int OP, int VEC, bool ONE, bool SHORT>
__global__ __launch_bounds__(256) void pass_kernel(PassArgs a) {
    static_assert(!SHORT || (ONE && OP == OP_LSE), "the other ops have one form");
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
                    double t;
                    if (SHORT && live == 1) t = exp(v0 - m);
                    else if (SHORT && live == 2 && mx[v] == -INFINITY) {
                        // nothing before: the larger of the two is the maximum, whose term is 1 (a NaN is the other one)
                        t = (hi == m ? 1.0 : hi > m ? INFINITY : 0.0) + exp((v0 == hi ? v1 : v0) - m);
                    } else if (SHORT && live <= 3) {
                        t = exp(v0 - m) + exp(v1 - m);
                        if (live == 3) t += exp(v2 - m);
                    } else t = (exp(v0 - m) + exp(v1 - m)) + (exp(v2 - m) + exp(v3 - m));
                    if (mx[v] != -INFINITY) t = fma(acc[v], exp(mx[v] - m), t);
                    acc[v] = t;
                    mx[v] = m;
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if (ONE && OP == OP_SOFTMAX_BWD && i >= live) break;
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

// ---------------------------------------------------------------------------------------------
// Persistent kernels for the narrow layers, as the fp32 ones (see there; same streams of runs, one column per workgroup of 16
// waves): a launch of pass_kernel over such a layer takes 4 to 7 us, of which the layer's arithmetic is a small part.  The
// exponentials cost most here (a library exponential is about forty instructions), so a group of four entries that is padding in
// all lanes is passed over, and a row of two entries takes one.
//   The reverse kernel keeps the two-gather form of the softmax adjoint (a sum of G_r exp(N_c - N_r)): the rows of even layers (OR
// nodes) are pairs (adjoint, value), those of odd layers a value that the adjoint replaces.
//   us, a launch or two for every layer and now, forward and training step: 85000 nodes in 20 layers (the top 14 of them) at B = 33
// 107 -> 84, 244 -> 203; 4500 nodes in 34 layers at B = 33 133 -> 58, 254 -> 125, at B = 512 208 -> 129, 411 -> 274; 20000 nodes
// with power-law fan-ins in 16 layers at B = 100 154 -> 96, 263 -> 188.
// ---------------------------------------------------------------------------------------------
typedef double Pair __attribute__((ext_vector_type(2)));
constexpr double kDblMax = 1.7976931348623157e308;
__device__ __forceinline__ double finite(double m) { return fmin(fmax(m, -kDblMax), kDblMax); }

template <int STEP>
__device__ __forceinline__ double fly(double x) {
    if (STEP < 4) {
        const long long b = __double_as_longlong(x);
        const float lo = klay::fly<STEP>(__int_as_float((int)b)), hi = klay::fly<STEP>(__int_as_float((int)(b >> 32)));
        return __longlong_as_double((long long)(uint32_t)__float_as_int(lo) | (long long)__float_as_int(hi) << 32);
    }
    return __shfl_xor(x, 1 << STEP);
}
template <int OP>
__device__ __forceinline__ double join(double a, double b) {
    if (OP == OP_PROD) return a * b;
    if (OP == OP_MAX || OP == OP_LSE) return fmax(a, b);          // (OP_LSE: the maxima)
    return a + b;
}
template <int OP>
__device__ __forceinline__ double col_fly(double x, int k) {
    if (k >= 1) x = join<OP>(x, fly<0>(x));
    if (k >= 2) x = join<OP>(x, fly<1>(x));
    if (k >= 3) x = join<OP>(x, fly<2>(x));
    if (k >= 4) x = join<OP>(x, fly<3>(x));
    if (k >= 5) x = join<OP>(x, fly<4>(x));
    if (k >= 6) x = join<OP>(x, fly<5>(x));
    return x;
}

// Logsumexp: m = maximum so far (of those that are no NaN), s = sum of exp(x - finite(m)); a row with nothing above -inf is -inf, a
// NaN in any other passes on (as in pass_kernel).
__device__ __forceinline__ double lse_value(double m, double s) { return m == -INFINITY ? -INFINITY : m + log(s); }

// rows of one entry, of two, of four
template <int OP>
__device__ __forceinline__ double col_one(double x) { return OP == OP_LSE || OP == OP_MAX ? fmax(x, -INFINITY) : x; }
template <int OP>
__device__ __forceinline__ double col_two(double x, double y) {
    if (OP != OP_LSE) return OP == OP_MAX ? fmax(fmax(x, y), -INFINITY) : join<OP>(x, y);
    return lse_value(fmax(fmax(x, y), -INFINITY), 1.0 + (x == y ? 1.0 : exp(-fabs(x - y))));
}
template <int OP>
__device__ __forceinline__ double col_four(double x0, double x1, double x2, double x3) {
    if (OP != OP_LSE) {
        const double x = join<OP>(join<OP>(x0, x1), join<OP>(x2, x3));
        return OP == OP_MAX ? fmax(x, -INFINITY) : x;
    }
    const double hi = fmax(fmax(fmax(x0, x1), fmax(x2, x3)), -INFINITY), m = finite(hi);
    return lse_value(hi, (exp(x0 - m) + exp(x1 - m)) + (exp(x2 - m) + exp(x3 - m)));
}

template <int OP, int KIND>
__device__ __forceinline__ void col_quarter(const double* below, uint32_t a, uint32_t b, double* out, int rows) {
    const int lane = threadIdx.x & 63;
    const double x0 = below[a & 0xFFFFu], x1 = below[a >> 16], x2 = below[b & 0xFFFFu], x3 = below[b >> 16];
    if (KIND == 0) {
        const double v[4] = {col_one<OP>(x0), col_one<OP>(x1), col_one<OP>(x2), col_one<OP>(x3)};
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (lane + 64 * i < rows) out[64 * i] = v[i];
    } else if (KIND == 1) {
        const double v0 = col_two<OP>(x0, x1), v1 = col_two<OP>(x2, x3);
        if (lane < rows) out[0] = v0;
        if (lane + 64 < rows) out[64] = v1;
    } else {
        const double v = col_four<OP>(x0, x1, x2, x3);
        if (lane < rows) out[0] = v;
    }
}

// a run of kind 0, 1 or 2
template <int OP, int KIND>
__device__ __forceinline__ void col_fwd_short(ColWalk& walk, const double* below, double* out, int rows) {
    constexpr int N = 4 >> KIND;                     // rows of a lane in a quarter of a block
    out += threadIdx.x & 63;
    for (; rows > 0; rows -= 256 * N, out += 256 * N) {
        Line w0, w1;
        walk.block(w0, w1);
        col_quarter<OP, KIND>(below, w0.x, w0.y, out, rows);
        if (rows > 64 * N) col_quarter<OP, KIND>(below, w0.z, w0.w, out + 64 * N, rows - 64 * N);
        if (rows > 128 * N) {
            col_quarter<OP, KIND>(below, w1.x, w1.y, out + 128 * N, rows - 128 * N);
            if (rows > 192 * N) col_quarter<OP, KIND>(below, w1.z, w1.w, out + 192 * N, rows - 192 * N);
        }
    }
}

// four entries of a row that takes several lanes or lines, joined to what those before gave
template <int OP>
__device__ __forceinline__ void col_long4(const double* below, uint32_t a, uint32_t b, double& m, double& s) {
    const double x0 = below[a & 0xFFFFu], x1 = below[a >> 16], x2 = below[b & 0xFFFFu], x3 = below[b >> 16];
    if (OP == OP_LSE) {
        const double hi = fmax(fmax(fmax(x0, x1), fmax(x2, x3)), m), m2 = finite(hi);
        double t = (exp(x0 - m2) + exp(x1 - m2)) + (exp(x2 - m2) + exp(x3 - m2));
        if (s != 0.0) t = fma(s, exp(m - m2), t);
        s = t;
        m = hi;
    } else {
        s = join<OP>(s, join<OP>(join<OP>(x0, x1), join<OP>(x2, x3)));
    }
}
template <int OP>
__device__ __forceinline__ void col_long(const double* below, Line w, uint32_t pads, double& m, double& s) {
    col_long4<OP>(below, w.x, w.y, m, s);
    if (__any(w.z != pads || w.w != pads)) col_long4<OP>(below, w.z, w.w, m, s);
}

template <int OP>
__device__ __forceinline__ void col_fwd_layer(ColWalk& walk, const double* below, double* here, int pad) {
    const int lane = threadIdx.x & 63;
    const uint32_t pads = (uint32_t)pad | (uint32_t)pad << 16;
    Desc table = walk.table();
    ColRun run;
    for (int i = 0; run.read(walk, table, i);) {
        double* out = here + run.slot;
        if (run.kind == 0) col_fwd_short<OP, 0>(walk, below, out, run.rows);
        else if (run.kind == 1) col_fwd_short<OP, 1>(walk, below, out, run.rows);
        else if (run.kind == 2) col_fwd_short<OP, 2>(walk, below, out, run.rows);
        else {
            const int r = lane >> run.k, per = 64 >> run.k;
            const bool writes = (lane & ((1 << run.k) - 1)) == 0;
            for (int rows = run.rows; rows > 0; rows -= per, out += per) {
                double m = -INFINITY, s = OP == OP_LSE ? 0.0 : identity<OP>();
                for (int b = 0; b < run.blocks; ++b) {
                    Line w0, w1;
                    walk.block(w0, w1);
                    col_long<OP>(below, w0, pads, m, s);
                    if (run.kind == 3) col_long<OP>(below, w1, pads, m, s);
                }
                if (OP == OP_LSE) {
                    if (run.k > 0) {
                        const double m2 = col_fly<OP_LSE>(m, run.k);
                        s = col_fly<OP_SUM>(s == 0.0 ? 0.0 : s * exp(m - finite(m2)), run.k);
                        m = m2;
                    }
                    s = lse_value(m, s);
                } else {
                    s = col_fly<OP>(s, run.k);
                }
                if (writes && r < rows) out[r] = s;
            }
        }
    }
}

// a finished layer from LDS to the column-major buffer, by one wave (stride 2: the adjoints of pairs)
template <int STRIDE>
__device__ __forceinline__ void col_move(const double* values, int n, double* __restrict__ to) {
#pragma unroll 8
    for (int i = threadIdx.x & 63; i < n; i += 64) to[i] = values[(size_t)i * STRIDE];
}

// As the fp32 kernel of this name; start: rows of the activation buffer, start_map[i] or one after another.  tb: where the values
// are kept, T doubles a column.
__global__ __launch_bounds__(kColThreads) void col_fwd_kernel(const ColLayer* __restrict__ first, int n_layers, int first_is_and,
                                                              const Line* __restrict__ blocks, int n_blocks, const Desc* __restrict__ tables,
                                                              const double* __restrict__ start, int start_rows, const int32_t* __restrict__ start_map, int ld,
                                                              int semiring, int size0, double* __restrict__ tb, int T,
                                                              const int32_t* __restrict__ root_pos, int R, double* __restrict__ out) {
    extern __shared__ double smem64[];
    double* below = smem64;
    double* here = below + size0;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int col = (int)blockIdx.x;
    const bool log_domain = semiring != 0;
    ColWalk walk;
    walk.start(blocks + (size_t)first->fwd_block[wave] * 128 + lane, tables + (size_t)first->fwd_table[wave] * kDescTable + lane);
    if (gridDim.x >= 64) {
        ColTouch<4> blocks_ahead;
        blocks_ahead.ask(blocks, 2 * n_blocks, (int)threadIdx.x, kColThreads);
        blocks_ahead.finish();
    }
    if (threadIdx.x < 2) {
        double* a = threadIdx.x == 0 ? below : here;
        a[kColPadAnd] = log_domain ? 0.0 : 1.0;
        a[kColPadOr] = log_domain ? -INFINITY : 0.0;
    }
    for (int i = threadIdx.x; i < start_rows; i += kColThreads) below[kColSlots + i] = start[(size_t)(start_map ? start_map[i] : i) * ld + col];
    double* tbc = tb + (size_t)col * T;
    for (int t = 0; t < n_layers; ++t) {
        const bool is_and = ((t & 1) == 0) == (first_is_and != 0);
        __syncthreads();
        if (wave == kColFwdWaves) {
            if (t > 0) col_move<1>(below + kColSlots, first[t - 1].n, tbc + first[t - 1].at);
        } else if (is_and) {
            if (log_domain) col_fwd_layer<OP_SUM>(walk, below, here, kColPadAnd);
            else col_fwd_layer<OP_PROD>(walk, below, here, kColPadAnd);
        } else if (semiring == 1) col_fwd_layer<OP_LSE>(walk, below, here, kColPadOr);
        else if (semiring == 2) col_fwd_layer<OP_MAX>(walk, below, here, kColPadOr);
        else col_fwd_layer<OP_SUM>(walk, below, here, kColPadOr);
        double* tmp = below; below = here; here = tmp;
    }
    __syncthreads();
    if (wave == kColFwdWaves) col_move<1>(below + kColSlots, first[n_layers - 1].n, tbc + first[n_layers - 1].at);
    for (int r = threadIdx.x; r < R; r += kColThreads) out[(size_t)col * R + r] = below[kColSlots + root_pos[r]];
}

// ---- reverse: rows of even layers are pairs, rows of odd layers single values
template <bool OR> struct ColRows;
template <> struct ColRows<true> {          // through an OR layer: from pairs into the rows of an AND layer
    using Above = Pair;
    using Here = double;
    static __device__ __forceinline__ double own(const double* at) { return *at; }
    static __device__ __forceinline__ void put(double* at, double g) { *at = g; }
    static __device__ __forceinline__ double entry(const Pair* above, uint32_t e, double own) {
        const Pair p = above[e & 0x7FFFu];
        return !(e & 0x8000u) ? p.x : p.y == -INFINITY ? 0.0 : p.x * exp(own - p.y);
    }
};
template <> struct ColRows<false> {         // through an AND layer: into pairs, whose value is there
    using Above = double;
    using Here = Pair;
    static __device__ __forceinline__ double own(const Pair*) { return 0.0; }
    static __device__ __forceinline__ void put(Pair* at, double g) { reinterpret_cast<double*>(at)[0] = g; }
    static __device__ __forceinline__ double entry(const double* above, uint32_t e, double) { return above[e & 0x7FFFu]; }
};

template <bool OR, int KIND>
__device__ __forceinline__ void col_bwd_quarter(const typename ColRows<OR>::Above* above, uint32_t a, uint32_t b, typename ColRows<OR>::Here* out, int rows) {
    using Rows = ColRows<OR>;
    constexpr int N = 4 >> KIND;
    const int lane = threadIdx.x & 63;
    const uint32_t e[4] = {a & 0xFFFFu, a >> 16, b & 0xFFFFu, b >> 16};
    double v[4], own[N];
#pragma unroll
    for (int i = 0; i < N; ++i) own[i] = Rows::own(out + (lane + 64 * i < rows ? 64 * i : -lane));
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = Rows::entry(above, e[i], own[i >> KIND]);
#pragma unroll
    for (int i = 0; i < N; ++i)
        if (lane + 64 * i < rows) Rows::put(out + 64 * i, KIND == 0 ? v[i] : KIND == 1 ? v[2 * i] + v[2 * i + 1] : (v[0] + v[1]) + (v[2] + v[3]));
}

template <bool OR, int KIND>
__device__ __forceinline__ void col_bwd_short(ColWalk& walk, const typename ColRows<OR>::Above* above, typename ColRows<OR>::Here* out, int rows) {
    constexpr int N = 4 >> KIND;
    out += threadIdx.x & 63;
    for (; rows > 0; rows -= 256 * N, out += 256 * N) {
        Line w0, w1;
        walk.block(w0, w1);
        col_bwd_quarter<OR, KIND>(above, w0.x, w0.y, out, rows);
        if (rows > 64 * N) col_bwd_quarter<OR, KIND>(above, w0.z, w0.w, out + 64 * N, rows - 64 * N);
        if (rows > 128 * N) {
            col_bwd_quarter<OR, KIND>(above, w1.x, w1.y, out + 128 * N, rows - 128 * N);
            if (rows > 192 * N) col_bwd_quarter<OR, KIND>(above, w1.z, w1.w, out + 192 * N, rows - 192 * N);
        }
    }
}

template <bool OR>
__device__ __forceinline__ double col_bwd_line(const typename ColRows<OR>::Above* above, Line w, double own) {
    using Rows = ColRows<OR>;
    constexpr uint32_t pads = (uint32_t)kColPadAnd | (uint32_t)kColPadAnd << 16;
    double s = (Rows::entry(above, w.x & 0xFFFFu, own) + Rows::entry(above, w.x >> 16, own)) + (Rows::entry(above, w.y & 0xFFFFu, own) + Rows::entry(above, w.y >> 16, own));
    if (__any(w.z != pads || w.w != pads))
        s += (Rows::entry(above, w.z & 0xFFFFu, own) + Rows::entry(above, w.z >> 16, own)) + (Rows::entry(above, w.w & 0xFFFFu, own) + Rows::entry(above, w.w >> 16, own));
    return s;
}

template <bool OR>
__device__ __forceinline__ void col_bwd_layer(ColWalk& walk, const typename ColRows<OR>::Above* above, typename ColRows<OR>::Here* here) {
    using Rows = ColRows<OR>;
    const int lane = threadIdx.x & 63;
    Desc table = walk.table();
    ColRun run;
    for (int i = 0; run.read(walk, table, i);) {
        typename Rows::Here* out = here + run.slot;
        if (run.kind == 0) col_bwd_short<OR, 0>(walk, above, out, run.rows);
        else if (run.kind == 1) col_bwd_short<OR, 1>(walk, above, out, run.rows);
        else if (run.kind == 2) col_bwd_short<OR, 2>(walk, above, out, run.rows);
        else {
            const int r = lane >> run.k, per = 64 >> run.k;
            const bool writes = (lane & ((1 << run.k) - 1)) == 0;
            for (int rows = run.rows; rows > 0; rows -= per, out += per) {
                const double own = Rows::own(out + (r < rows ? r : 0));
                double s = 0.0;
                for (int b = 0; b < run.blocks; ++b) {
                    Line w0, w1;
                    walk.block(w0, w1);
                    double t = col_bwd_line<OR>(above, w0, own);
                    if (run.kind == 3) t += col_bwd_line<OR>(above, w1, own);
                    s += t;
                }
                s = col_fly<OP_SUM>(s, run.k);
                if (writes && r < rows) Rows::put(out + r, s);
            }
        }
    }
}

// Where the reverse kernel leaves the adjoints of its last layer: the leaf gradients (wT != null, the last layer is layer 0), or,
// column-major, g_cols (T doubles a column, from `at` of a layer on).  KEEP: every layer's from the keep_from-th below the top one
// on go there.
struct ColBwdOut {
    double* g_cols;
    int32_t keep_from, n_last;
    const double* wT;           // [V, ld]
    const int32_t *pos_row, *neg_row;
    double *dleaf, *dneg;
    int32_t V, mode, ld;        // mode: as for leaf_bwd_kernel
};

// own values of a layer per thread (in registers, a step ahead): rows up to this many times 1024
constexpr int kColOwn = 10;

// Reverse sweep in the log semiring from the top layer down n_steps layers; the last one is an AND layer or layer 0.  LDS: `odd_at`
// doubles of pairs for the even layers, then the odd layers.  tb: node values; those of the rows of a step are loaded during the
// step before.
template <bool KEEP>
__global__ __launch_bounds__(kColThreads) void col_bwd_kernel(const ColLayer* __restrict__ top, int n_steps, int last_at, int top_is_and,
                                                              const Line* __restrict__ blocks, int n_blocks, const Desc* __restrict__ tables,
                                                              const double* __restrict__ dout, const int32_t* __restrict__ top_ptr,
                                                              const int32_t* __restrict__ top_root, int R, int odd_at, const double* tb, int T, ColBwdOut res) {
    extern __shared__ double smem64[];
    Pair* const even = reinterpret_cast<Pair*>(smem64);
    double* const odd = smem64 + odd_at;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int col = (int)blockIdx.x;
    const double* tbc = tb + (size_t)col * T;
    ColWalk walk;
    walk.start(blocks + (size_t)top->bwd_block[wave] * 128 + lane, tables + (size_t)top->bwd_table[wave] * kDescTable + lane);
    if (gridDim.x >= 64) {
        ColTouch<4> blocks_ahead;
        blocks_ahead.ask(blocks, 2 * n_blocks, (int)threadIdx.x, kColThreads);
        blocks_ahead.finish();
    }
    if (threadIdx.x == 0) {
        even[kColPadAnd] = Pair{0.0, 0.0};
        odd[kColPadAnd] = 0.0;
    }
    // own values of the rows of the t-th layer below the top one: how many and where (none for layer 0)
    auto own_of = [&](int t, int& n, int& at) {
        n = at = 0;
        if (t < n_steps) { n = top[-t].n; at = top[-t].at; }
        else if (t == n_steps && last_at >= 0) { n = res.n_last; at = last_at; }
    };
    auto is_odd = [&](int t) { return ((t & 1) == 0) == (top_is_and != 0); };
    auto put_own = [&](int t, int i, double v) {
        if (is_odd(t)) odd[kColSlots + i] = v;
        else reinterpret_cast<double*>(even + kColSlots + i)[1] = v;
    };
    int n, at;
    own_of(1, n, at);
    for (int i = threadIdx.x; i < n; i += kColThreads) put_own(1, i, tbc[at + i]);
    own_of(0, n, at);
    for (int i = threadIdx.x; i < n; i += kColThreads) {      // adjoint seed of the top layer
        double acc = 0.0;
        for (int j = top_ptr[i]; j < top_ptr[i + 1]; ++j) acc += dout[(size_t)col * R + top_root[j]];
        if (is_odd(0)) odd[kColSlots + i] = acc;
        else even[kColSlots + i] = Pair{acc, tbc[at + i]};
    }
    auto keep_layer = [&](int t) {
        if (t < res.keep_from) return;
        double* to = res.g_cols + (size_t)col * T + top[-t].at;
        if (is_odd(t)) col_move<1>(odd + kColSlots, top[-t].n, to);
        else col_move<2>(reinterpret_cast<const double*>(even + kColSlots), top[-t].n, to);
    };
    for (int t = 0; t < n_steps; ++t) {
        double own[kColOwn];
        own_of(t + 2, n, at);
#pragma unroll
        for (int i = 0; i < kColOwn; ++i)
            if (wave * 64 + i * kColThreads < n) own[i] = tbc[at + ((int)threadIdx.x + i * kColThreads < n ? (int)threadIdx.x + i * kColThreads : 0)];
        __syncthreads();
        if (KEEP && wave == kTopBwdWaves) keep_layer(t);
        else if (is_odd(t)) col_bwd_layer<false>(walk, odd, even);
        else col_bwd_layer<true>(walk, even, odd);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kColOwn; ++i)
            if ((int)threadIdx.x + i * kColThreads < n) put_own(t, (int)threadIdx.x + i * kColThreads, own[i]);
    }
    __syncthreads();
    if (!res.wT) {
        for (int r = threadIdx.x; r < res.n_last; r += kColThreads) res.g_cols[(size_t)col * T + last_at + r] = odd[kColSlots + r];
        return;
    }
    for (int v = threadIdx.x; v < res.V; v += kColThreads) {
        const int pr = res.pos_row[v], nr = res.neg_row[v];
        double d = pr >= 0 ? even[kColSlots + pr].x : 0.0, dn = 0.0;
        if (nr >= 0) {
            const double gn = even[kColSlots + nr].x;
            if (res.mode == 2) dn = gn;
            else if (gn != 0.0) d += res.mode == 1 ? -gn / expm1(-res.wT[(size_t)v * res.ld + col]) : -gn;
        }
        res.dleaf[(size_t)col * res.V + v] = d;
        if (res.mode == 2 && res.dneg) res.dneg[(size_t)col * res.V + v] = dn;
    }
}

// rows[r, b] (map: rows[map[r], b], where that is not negative) = cols[b, first + r] for r < n_rows, through a 32 x 33 LDS tile
__global__ __launch_bounds__(256) void cols_to_rows_kernel(const double* __restrict__ cols, int T, int first, int n_rows, int B, int ld,
                                                           double* __restrict__ rows, const int32_t* __restrict__ map) {
    __shared__ double tile[32][33];
    const int r0 = blockIdx.x * 32, b0 = blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;       // 32 x 8
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int b = b0 + ty + 8 * j, r = r0 + tx;
        tile[ty + 8 * j][tx] = (b < B && r < n_rows) ? cols[(size_t)b * T + first + r] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int r = r0 + ty + 8 * j, b = b0 + tx;
        if (r < n_rows && b < ld)
            if (const int row = map ? map[r] : r; row >= 0) rows[(size_t)row * ld + b] = tile[tx][ty + 8 * j];
    }
}

}  // namespace f64
}  // namespace klay
