// Small dense FP64 pieces of the numerical setup's factorisations, one
// wavefront each: sums by matrix instructions, the elimination of 16 columns.
// All of them round like the scalar loops they stand for (quotients: in the
// range given at div_by).
#pragma once

#include <type_traits>
#include <utility>

#include "kernels_common.hpp"

namespace gdsw {

// FP64 matrix instructions (16x16x4).  Lane l = 16 g + i holds A(i, k) and
// B(k, i) for k = g, and of the 16x16 result D(g + 4 v, i) in value v.  The
// result is that of four multiply-adds in ascending k, each rounded (checked
// bit for bit, subnormal results included), so that sums over k taken four at
// a time in ascending order have the bits of a scalar loop.  A sum over 16
// values of k: instruction q takes k = 4 q + g, a lane's four operands stand
// four columns apart.
typedef double dbl4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ dbl4 mfma_k16(const dbl4 &a, const dbl4 &b, dbl4 c) {
#pragma unroll
    for (int q = 0; q < 4; ++q) c = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q], b[q], c, 0, 0, 0);
    return c;
}

// keeps a value's computation from being moved past this point
__device__ __forceinline__ void pin(double &x) { asm volatile("" : "+v"(x)); }

// f(0), f(1), .. f(N - 1) with compile-time arguments (register arrays are
// indexed by constants from the start, whatever the unroller decides)
template <int... I, typename F>
__device__ __forceinline__ void static_for_seq(std::integer_sequence<int, I...>, F f) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F f) {
    static_for_seq(std::make_integer_sequence<int, (N > 0 ? N : 0)>{}, f);
}

// orders one wavefront's LDS accesses (no instruction: LDS is in order)
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// x / s, correctly rounded, with y = 1 / s correctly rounded (Markstein: the
// quotient's remainder is exact in one multiply-add, and adding remainder times
// y rounds once).  For |x| of at least 2^-968 or zero, where the remainder is a
// multiple of the smallest subnormal, and quotients in the normal range; below
// that (entries of a band that decay past 1e-291) the last bit may differ.
__device__ __forceinline__ double div_by(double x, double s, double y) {
    const double q = x * y;
    return __builtin_fma(__builtin_fma(-s, q, x), y, q);
}

// 1 / s for s = sqrt(d), correctly rounded: 1 / sqrt(d) from the hardware's
// estimate to about an ulp beside the square root's own chain, then two
// corrections with s itself.  The first leaves less than an ulp (the estimate's
// error, the root's rounding and the square's make up to two, from which one
// correction misses the rounding for some s); from there the second rounds
// correctly (Markstein) for every s but those with all mantissa bits set, whose
// reciprocal lies 2^-53 of itself above a power of two and is the double after it.
__device__ __forceinline__ double rcp_of_sqrt(double d, double s) {
    double y = __builtin_amdgcn_rsq(d);
    double e = __builtin_fma(-d * y, y, 1.0);
    y = __builtin_fma(y, __builtin_fma(0.375 * e, e, 0.5 * e), y);
    y = __builtin_fma(__builtin_fma(-s, y, 1.0), y, y);
    y = __builtin_fma(__builtin_fma(-s, y, 1.0), y, y);
    const bool ones = __double2loint(s) == -1 && (__double2hiint(s) & 0xfffff) == 0xfffff;
    return __hiloint2double(__double2hiint(y), __double2loint(y) | int(ones));
}

// Cholesky elimination with 16 pivots by one wavefront, a row per lane: lanes
// 0..15 hold the rows of a symmetric 16x16 block (both halves), the others
// further rows of the same 16 columns.  On return a[j] of a lane is L(row, j)
// (lanes r < 16: j < r), rounded as by the scalar loop l = a / sqrt(pivot),
// a_rc -= l_r l_c (MUL: l = a times the rounded reciprocal of sqrt(pivot)); ds
// and dy of lane j < 16 hold sqrt(pivot j) and its reciprocal.  bad: 1 + row0 + the first non-positive pivot (taken as 1), kept
// if it is set already.  The lanes above the diagonal compute values nobody
// reads, as do columns from `cols` on (fewer than 16 columns).
constexpr int EB = 16;
template <bool MUL = false>
__device__ __forceinline__ void elim16(double (&a)[EB], int lane, int row0, int &bad, double &ds, double &dy,
                                       int cols = EB) {
    asm volatile("" : "+v"(lane));   // (the lane masks are not to be kept across calls)
    ds = dy = 1.0;
    double s, y;
    auto pivot = [&](double d, int j) {
        const bool ok = d > 0.0;   // (uniform)
        bad = !ok && j < cols && bad == 0 ? 1 + row0 + j : bad;
        d = ok ? d : 1.0;
        s = sqrt(d);
        y = rcp_of_sqrt(d, s);
        if (lane == j) ds = s, dy = y;
    };
    pivot(lane_read(a[0], 0), 0);
    static_for<EB>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        const double t = MUL ? a[j] * y : div_by(a[j], s, y);
        a[j] = t;
        if constexpr (j + 1 < EB) {
            // the next pivot first: its chain runs beside the other columns
            a[j + 1] = __builtin_fma(-lane_read(t, j + 1), t, a[j + 1]);
            pivot(lane_read(a[j + 1], j + 1), j + 1);
            // (at most four multipliers held in scalar registers at a time)
            static_for<(EB - j + 1) / 4>([&](auto gc) {
                constexpr int r = j + 2 + 4 * decltype(gc)::value;
                double m[4] = {};
                static_for<4>([&](auto u) { if constexpr (r + u < EB) m[u] = lane_read(t, r + u); });
                static_for<4>([&](auto u) {
                    if constexpr (r + u < EB) a[r + u] = __builtin_fma(-m[u], t, a[r + u]);
                });
                static_for<4>([&](auto u) { if constexpr (r + u < EB) pin(a[r + u]); });
            });
        }
    });
}

// The rows below such a block: a row per lane, L(row, j) from the block's
// columns and pivots in LDS (sT: column j at 16 j, 16-byte aligned; sd:
// sqrt(pivot) and reciprocal).  The next column's values are read while one is
// in use.
template <bool MUL = false>
__device__ __forceinline__ void subst16(double (&a)[EB], const double *sT, const double *sd) {
    double m[2][EB], p[2][2];
    auto column = [&](auto jc) __attribute__((always_inline)) {
        constexpr int j = decltype(jc)::value, k = j & 1;
        p[k][0] = sd[2 * j], p[k][1] = sd[2 * j + 1];
        static_for<EB - 1 - j>([&](auto u) {
            constexpr int r = j + 1 + decltype(u)::value;
            m[k][r] = sT[EB * j + r];
        });
    };
    column(std::integral_constant<int, 0>{});
    static_for<EB>([&](auto jc) __attribute__((always_inline)) {
        constexpr int j = decltype(jc)::value, k = j & 1;
        if constexpr (j + 1 < EB) column(std::integral_constant<int, j + 1>{});
        asm volatile("" ::: "memory");   // (no reads past the next column's)
        const double t = MUL ? a[j] * p[k][1] : div_by(a[j], p[k][0], p[k][1]);
        a[j] = t;
        static_for<EB - 1 - j>([&](auto u) {
            constexpr int r = j + 1 + decltype(u)::value;
            a[r] = __builtin_fma(-m[k][r], t, a[r]);
        });
        static_for<EB - 1 - j>([&](auto u) { pin(a[j + 1 + decltype(u)::value]); });
    });
}

}  // namespace gdsw
