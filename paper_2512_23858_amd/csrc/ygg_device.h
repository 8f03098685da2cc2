// Device-side helpers shared by the kernel translation units: wave-wide reductions, order-preserving
// integer keys of floating-point values, and an fp64 exponential.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ygg {

// ---- wave-wide reductions on DPP (row shifts and row broadcasts of the 64-wide wavefront) --------
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_or_self(uint32_t v) {
    // lanes without a valid source (or outside ROW_MASK) keep their own value
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, ROW_MASK, 0xf, false);
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
    v = max(v, dpp_or_self<0xb1, 0xf>(v));   // quad_perm [1,0,3,2]
    v = max(v, dpp_or_self<0x4e, 0xf>(v));   // quad_perm [2,3,0,1]
    v = max(v, dpp_or_self<0x114, 0xf>(v));  // row_shr:4
    v = max(v, dpp_or_self<0x118, 0xf>(v));  // row_shr:8   -> lane 15 of every row holds the row maximum
    v = max(v, dpp_or_self<0x142, 0xa>(v));  // row_bcast:15 into rows 1 and 3
    v = max(v, dpp_or_self<0x143, 0xc>(v));  // row_bcast:31 into rows 2 and 3 -> lane 63 holds the maximum
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) { return ~wave_max_u32(~v); }

// ---- exchanges between the lanes of a wavefront that cost no LDS round trip -----------------------
// v from lane (lane ^ M) for M = 1, 2, 8; the mirrored lane of a group of 8 (M = 7) or 16 (M = 15).
template <int M>
__device__ __forceinline__ uint32_t row_xor(uint32_t v) {
    constexpr int ctrl = M == 1 ? 0xb1 : M == 2 ? 0x4e : M == 7 ? 0x141 : M == 8 ? 0x128 : 0x140;
    static_assert(M == 1 || M == 2 || M == 7 || M == 8 || M == 15, "a pattern of the row permutes");
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, 0xf, 0xf, true);
}
// op over aligned groups of `width` lanes (a power of two up to 64, the same in every lane); every lane gets the result.
// After the first steps all lanes of a sub-group agree, so a mirror serves where an exchange of halves is meant.
template <typename Op>
__device__ __forceinline__ float group_reduce(float v, int width, Op op) {
    auto f = [](uint32_t u) { return __uint_as_float(u); };
    const auto u = [&] { return __float_as_uint(v); };
    if (width > 1) v = op(v, f(row_xor<1>(u())));
    if (width > 2) v = op(v, f(row_xor<2>(u())));
    if (width > 4) v = op(v, f(row_xor<7>(u())));
    if (width > 8) v = op(v, f(row_xor<15>(u())));
    if (width > 16) { const auto p = __builtin_amdgcn_permlane16_swap(u(), u(), false, false); v = op(f(p[0]), f(p[1])); }
    if (width > 32) { const auto p = __builtin_amdgcn_permlane32_swap(u(), u(), false, false); v = op(f(p[0]), f(p[1])); }
    return v;
}
__device__ __forceinline__ double group_sum(double v, int width) {
    auto mk = [](uint32_t lo, uint32_t hi) { return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo)); };
    const auto lo = [&] { return (uint32_t)__double_as_longlong(v); };
    const auto hi = [&] { return (uint32_t)((uint64_t)__double_as_longlong(v) >> 32); };
    if (width > 1) v += mk(row_xor<1>(lo()), row_xor<1>(hi()));
    if (width > 2) v += mk(row_xor<2>(lo()), row_xor<2>(hi()));
    if (width > 4) v += mk(row_xor<7>(lo()), row_xor<7>(hi()));
    if (width > 8) v += mk(row_xor<15>(lo()), row_xor<15>(hi()));
    if (width > 16) {
        const auto a = __builtin_amdgcn_permlane16_swap(lo(), lo(), false, false), b = __builtin_amdgcn_permlane16_swap(hi(), hi(), false, false);
        v = mk(a[0], b[0]) + mk(a[1], b[1]);
    }
    if (width > 32) {
        const auto a = __builtin_amdgcn_permlane32_swap(lo(), lo(), false, false), b = __builtin_amdgcn_permlane32_swap(hi(), hi(), false, false);
        v = mk(a[0], b[0]) + mk(a[1], b[1]);
    }
    return v;
}
// v from lane (lane ^ M), M a power of two below 64
template <int M>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v) {
    if constexpr (M == 1 || M == 2 || M == 8) return row_xor<M>(v);
    else if constexpr (M == 4 || M == 16) return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x1f | (M << 10));
    else {
        const auto p = __builtin_amdgcn_permlane32_swap(v, v, false, false);   // {low half twice, high half twice}
        return (threadIdx.x & 32) ? p[0] : p[1];
    }
}

// order-preserving maps to unsigned integers (larger value <-> larger key; -inf is the smallest real key)
__device__ __forceinline__ uint32_t key_of(float f) {
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float float_of(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}
__device__ __forceinline__ uint64_t key_of(double d) {
    const uint64_t u = (uint64_t)__double_as_longlong(d);
    return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}
__device__ __forceinline__ double double_of(uint64_t k) {
    return __longlong_as_double((long long)((k >> 63) ? (k & 0x7fffffffffffffffull) : ~k));
}

// exp(t) in fp64 for -746 <= t <= 709 (Cody and Waite's argument reduction): k = t/ln 2 to the nearest integer, read from the low
// bits of a sum with 1.5 * 2^52; r = t - k ln 2 (two-part constant); then a polynomial of degree 12 on |r| <= ln(2)/2: the Taylor
// series of degree 18, economised (Lanczos: its terms above degree 12 replaced by Chebyshev polynomials' remainders on that interval)
// and rounded to fp64, relative error 4.3e-19 (the series itself: 5.2e-18 at degree 13; economised to degree 11: 1.6e-17); scaled by
// 2^k.  Relative error 1.4e-16 at most and 4.12e-17 on average, as with the series of degree 13 (degree 11: 1.46e-16 and 4.16e-17);
// below the underflow point the result is 0 or the smallest subnormal.  Branch-free, so independent calls interleave.  N arguments in
// step: a dependent fp64 operation takes about 20 cycles, an independent one four.
template <int N>
__device__ __forceinline__ void exp_clamped_n(const double (&t)[N], double (&e)[N]) {
    constexpr double c[] = {2.0925031338286953e-09, 2.511487021947156e-08,  2.755723946763412e-07, 2.7557224956110785e-06,
                            2.4801587366915758e-05, 0.00019841269909219843, 0.0013888888888861422, 0.008333333333309526,
                            0.04166666666666672,    0.16666666666666702,    0.5,                   1.0,
                            1.0};
    constexpr double round_at = 6755399441055744.0;   // 1.5 * 2^52
    double k[N], r[N];
    int ki[N];
#pragma unroll
    for (int i = 0; i < N; ++i) k[i] = fma(t[i], 1.4426950408889634074, round_at);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        ki[i] = (int)(uint32_t)__double_as_longlong(k[i]);
        k[i] -= round_at;
    }
#pragma unroll
    for (int i = 0; i < N; ++i) r[i] = fma(k[i], -6.93147180369123816490e-01, t[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) r[i] = fma(k[i], -1.90821492927058770002e-10, r[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) e[i] = fma(c[0], r[i], c[1]);
#pragma unroll
    for (int s = 2; s < 13; ++s) {
#pragma unroll
        for (int i = 0; i < N; ++i) e[i] = fma(e[i], r[i], c[s]);
        __builtin_amdgcn_sched_barrier(0);   // keep the series in step
    }
#pragma unroll
    for (int i = 0; i < N; ++i) e[i] = ldexp(e[i], ki[i]);
}
__device__ __forceinline__ double exp_below(double t) {
    const double a[1] = {fmax(t, -746.0)};
    double e[1];
    exp_clamped_n(a, e);
    return e[0];
}
// exp(t) for t <= 0, exactly 0 below the underflow point
__device__ __forceinline__ double exp_nonpos(double t) { return t < -745.0 ? 0.0 : exp_below(t); }

}  // namespace ygg
