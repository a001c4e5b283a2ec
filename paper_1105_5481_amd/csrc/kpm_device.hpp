// Device-side building blocks of libkpm (gfx950): 16-byte vector types,
// division by run-time constants, the Philox4x64-10 generator, double-double
// accumulation and wave/block reductions.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace kpm {

// ---------------------------------------------------------------------------
// 16-byte vector of scalars: every thread moves one such chunk per stream.
// ---------------------------------------------------------------------------
template <typename S> struct V16;
template <> struct V16<float> {
    typedef float T __attribute__((ext_vector_type(4)));
    enum { W = 4 };
};
template <> struct V16<double> {
    typedef double T __attribute__((ext_vector_type(2)));
    enum { W = 2 };
};

template <typename S>
__device__ __forceinline__ typename V16<S>::T ld16(const S *p)
{
    return *reinterpret_cast<const typename V16<S>::T *>(p);
}
template <typename S>
__device__ __forceinline__ typename V16<S>::T ld16_stream(const S *p)
{
    return __builtin_nontemporal_load(reinterpret_cast<const typename V16<S>::T *>(p));
}
template <typename S>
__device__ __forceinline__ void st16_stream(S *p, typename V16<S>::T v)
{
    __builtin_nontemporal_store(v, reinterpret_cast<typename V16<S>::T *>(p));
}

// ---------------------------------------------------------------------------
// Unsigned 32-bit division by a run-time constant d >= 1 (Granlund and
// Montgomery, "Division by invariant integers using multiplication", PLDI'94):
// with s = ceil(log2 d) and m = floor(2^32 (2^s - d) / d) + 1,
// floor(n / d) = (mulhi(m, n) + n) >> s for every 32-bit n.
// ---------------------------------------------------------------------------
struct FastDiv {
    uint32_t d, m, s, pad;
};

__host__ __device__ __forceinline__ uint32_t fdiv(uint32_t n, FastDiv f)
{
    uint32_t hi = (uint32_t)(((uint64_t)f.m * (uint64_t)n) >> 32);
    return (uint32_t)(((uint64_t)hi + (uint64_t)n) >> f.s);
}

static inline FastDiv make_fastdiv(uint32_t d)
{
    FastDiv f;
    f.d = d;
    uint32_t s = 0;
    while ((uint64_t(1) << s) < (uint64_t)d) ++s;
    f.s = s;
    f.m = (uint32_t)((((uint64_t(1) << 32) * ((uint64_t(1) << s) - (uint64_t)d)) / (uint64_t)d) + 1);
    f.pad = 0;
    return f;
}

// ---------------------------------------------------------------------------
// Philox4x64-10 (Salmon, Moraes, Dror, Shaw, "Parallel random numbers: as easy
// as 1, 2, 3", SC'11): ten rounds of two 64x64->128 multiplications with the
// round multipliers, the key bumped by the Weyl constants between rounds.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void philox4x64_10(uint64_t &c0, uint64_t &c1, uint64_t &c2, uint64_t &c3,
                                              uint64_t k0, uint64_t k1)
{
    const uint64_t M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
    const uint64_t W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        uint64_t hi0 = __umul64hi(M0, c0), lo0 = M0 * c0;
        uint64_t hi1 = __umul64hi(M1, c2), lo1 = M1 * c2;
        uint64_t n0 = hi1 ^ c1 ^ k0;
        uint64_t n2 = hi0 ^ c3 ^ k1;
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
        k0 += W0;
        k1 += W1;
    }
}

// ---------------------------------------------------------------------------
// double-double arithmetic (error-free transformations: Knuth's two-sum,
// the fma two-product; accumulation as in Ogita, Rump, Oishi, "Accurate sum
// and dot product", SIAM J. Sci. Comput. 26, 2005).
// ---------------------------------------------------------------------------
struct dd {
    double hi, lo;
};

__device__ __forceinline__ dd dd_two_sum(double a, double b)
{
    double s = a + b;
    double v = s - a;
    double e = (a - (s - v)) + (b - v);
    return dd{s, e};
}
__device__ __forceinline__ dd dd_fast_two_sum(double a, double b)
{
    double s = a + b;
    double e = b - (s - a);
    return dd{s, e};
}
__device__ __forceinline__ dd dd_add(dd x, dd y)
{
    dd s = dd_two_sum(x.hi, y.hi);
    dd t = dd_two_sum(x.lo, y.lo);
    s.lo += t.hi;
    s = dd_fast_two_sum(s.hi, s.lo);
    s.lo += t.lo;
    return dd_fast_two_sum(s.hi, s.lo);
}
// x + y inside sums of many terms, in 11 operations (dd_add takes 20): off by about 2^-106 of
// the larger term rather than of the sum, which is what the terms themselves are off by.
// Over trees and runs of partials its error is that of dd_add (random products of any size and
// sign, 2^-106 of their absolute sum for both); left unnormalised it is up to 2.8 times as much.
__device__ __forceinline__ dd dd_sum(dd x, dd y)
{
    const dd s = dd_two_sum(x.hi, y.hi);
    return dd_fast_two_sum(s.hi, s.lo + (x.lo + y.lo));
}
__device__ __forceinline__ dd dd_sum(dd x, double y)
{
    const dd s = dd_two_sum(x.hi, y);
    return dd_fast_two_sum(s.hi, s.lo + x.lo);
}
// (s, c) += x*y exactly up to the error term c, which is summed in FP64.  The two-sum of s and
// the rounded product p gives s + p = t + (s - (t - v)) + (p - v); the product's own error is
// taken in with the last term, (p - v) + (x*y - p) = x*y - v in one fma.
__device__ __forceinline__ void dot2_acc(double &s, double &c, double x, double y)
{
    const double t = s + x * y;
    const double v = t - s;
    c += (s - (t - v)) + fma(x, y, -v);
    s = t;
}
// The first product of a sum.
__device__ __forceinline__ void dot2_first(double &s, double &c, double x, double y)
{
    s = x * y;
    c = fma(x, y, -s);
}
__device__ __forceinline__ dd dd_div_d(dd x, double b)
{
    double q1 = x.hi / b;
    double p = q1 * b;
    double pe = fma(q1, b, -p);
    double r = ((x.hi - p) - pe) + x.lo;
    double q2 = r / b;
    return dd_fast_two_sum(q1, q2);
}

// ---------------------------------------------------------------------------
// lane exchanges in the vector ALU (ds_bpermute shuffles take 24 cycles each)
// ---------------------------------------------------------------------------
// (x, y) -> ([x.low, y.low], [x.high, y.high]), low / high the lower and upper 32 lanes
__device__ __forceinline__ void swap_halves(double &x, double &y)
{
    const uint64_t a = (uint64_t)__double_as_longlong(x), b = (uint64_t)__double_as_longlong(y);
    const auto l = __builtin_amdgcn_permlane32_swap((uint32_t)a, (uint32_t)b, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
    x = __longlong_as_double((long long)(((uint64_t)h[0] << 32) | l[0]));
    y = __longlong_as_double((long long)(((uint64_t)h[1] << 32) | l[1]));
}
// the same with the even and odd rows of 16 lanes
__device__ __forceinline__ void swap_rows(double &x, double &y)
{
    const uint64_t a = (uint64_t)__double_as_longlong(x), b = (uint64_t)__double_as_longlong(y);
    const auto l = __builtin_amdgcn_permlane16_swap((uint32_t)a, (uint32_t)b, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
    x = __longlong_as_double((long long)(((uint64_t)h[0] << 32) | l[0]));
    y = __longlong_as_double((long long)(((uint64_t)h[1] << 32) | l[1]));
}
// the value N lanes up within the row of 16 (a rotation)
template <int N> __device__ __forceinline__ double row_ror(double v)
{
    const uint64_t a = (uint64_t)__double_as_longlong(v);
    const uint32_t l = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)a, 0x120 + N, 0xf, 0xf, false);
    const uint32_t h = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(a >> 32), 0x120 + N, 0xf, 0xf, false);
    return __longlong_as_double((long long)(((uint64_t)h << 32) | l));
}

}  // namespace kpm
