// Kernels of libkpm for gfx950.
//
// The hot path is the fused recursion step (Eq. (rn) of Zhang et al. 2011):
//     r_{n+1} = 2 H~ r_n - r_{n-1},  written over r_{n-1},
// with the two dot products <r_{n+1}|r_{n+1}> and Re<r_{n+1}|r_n> that the
// doubling identities turn into mu_{2n+2} and mu_{2n+1}, taken from registers
// in the same pass.
//
// Layout.  Vectors are stored site-major: the R vectors (or 2R interleaved
// re/im scalars) of site i are contiguous, padded to a multiple of 16 bytes
// ("chunks").  A thread moves one 16-byte chunk per stream; a wavefront reads
// whole cache lines, and the neighbour of a site is the same chunk of the
// neighbouring site.
//
// March kernels (lattices).  The slowest lattice axis (y in 2D, z in 3D) is
// the march axis; a "plane" is the set of sites with one march coordinate and
// a "column" is one in-plane position.  A thread owns one chunk of one column
// and walks a segment of S planes, keeping the chunk of planes m-1, m, m+1 in
// registers: each vector element of r_n is fetched once per step from HBM
// (plus two halo planes per segment).  In-plane neighbours are read through
// L1/L2 from the adjacent columns, which neighbouring lanes and blocks of the
// same XCD load in the same pass.
//
// Flat kernels (CSR, and lattices on request).  Work is cut into tiles of
// 256*TPT consecutive chunks; every neighbour is loaded through the caches.
//
// A solve alone cuts the march axis into as many segments as keep the chip busy, down
// to one plane each; where a launch has blocks enough, a block walks a run of
// consecutive segments, which reads the two halo planes once per run.  The segments,
// and with them the partial sums, are the same either way.
//
// Reductions.  Each work item (march: column tile x segment; flat: tile) of a
// step leaves one partial (FP64 sums of its dot products) in a ring of
// per-step slots; a separate kernel sums the partials of a step over the items
// in a fixed order.  Results therefore do not depend on the launch grid or on
// which other instances share the launch.  The blocks of one instance walk
// its items per XCD (block b runs on XCD b mod 8 under round-robin dispatch):
// XCD x owns an eighth of them, as ItemRange says.
#pragma once

#include <type_traits>

#include "kpm_device.hpp"

#define KPM_GLOBAL __attribute__((address_space(1)))

namespace kpm {

enum OpKind { OP_REAL2 = 0, OP_REAL3 = 1, OP_SPIN2 = 2, OP_SPIN3 = 3, OP_CSR_R = 4, OP_CSR_C = 5, OP_COUNT = 6 };
enum { VEC_RADEMACHER = 0, VEC_PHASE = 1, VEC_UNIT = 2 };
enum { MODE_FLAT = 0, MODE_MARCH = 1, MODE_SMALL = 2, MODE_TB = 3, MODE_TB3 = 4 };   // how a solve runs
constexpr int BLOCK = 256;
constexpr uint32_t XCD_MIN_ITEMS = 64;   // below this an instance's items are not split per XCD
constexpr uint32_t NO_INSTANCE = 0xffffffffu;   // block-map entry of an idle block

// One solve inside a launch (device-resident table entry).
struct Inst {
    int32_t opk;
    int32_t has_diag;
    int32_t mode;
    int32_t xcd;       // items split per XCD (0 none, 1 by units, 2 by segments, 3 evenly, 4 explicit)
    int32_t alt;       // march: odd segments walk downwards
    int32_t nt;        // march: r_{n-1}/r_{n+1} accessed with non-temporal hints
    uint32_t Lx, Ly, Lz, N;
    FastDiv fLx, fLy, fC;
    uint32_t C;        // 16-byte chunks per site
    uint32_t Rs;       // scalars per site (C * W)
    uint32_t nel;      // N * C
    uint32_t tiles;    // work items per step (= partials per step)
    uint32_t nb;       // blocks given to this instance (multiple of 8)
    uint32_t block0;   // first block of this instance in the grid
    uint32_t bstride;  // its blocks are block0, block0 + bstride, ... (1, or 8 to keep them on one XCD)
    uint32_t q0, q1;   // xcd == 4: its items
    int32_t tpt;       // flat: chunks per thread per tile
    uint32_t P, Lm, S, nct, nseg;  // march: plane size, march extent, segment, column tiles, segments
    uint32_t run;      // march: consecutive segments a block walks without reloading its window
    int32_t cplx;      // data stored as interleaved complex
    int32_t M, K, R, vec;
    int32_t step0;     // recursion step n = step0 + (launch offset k)
    int32_t pslots;    // ring slots of partials
    int32_t tbh;       // temporal blocking: halo sites each side of an x-tile (= steps of the deepest pass)
    int32_t red_lo, red_n;  // dots indices [red_lo, red_lo + red_n) to reduce (k_reduce_ranges)
    uint64_t seed, instance;
    double norm;       // N R (random kinds) or R (unit vectors)
    const void *diag;  // S[N]
    const void *bond;  // S[N][dim][2]: H~_{i, i+e_ax}
    const void *hop;   // S[1]: H~_ij of the real lattice
    const int64_t *row_ptr;
    const int32_t *col;
    const void *val;   // S[nnz] or S[nnz][2]
    void *buf0, *buf1;
    void *tb2, *tb3;   // temporal blocking: buffers 2 and 3 of four (buf0, buf1 are 0 and 1)
    int32_t tbp, tbc;  // ... and which of them hold r_{step0-1}, r_{step0} (batched passes)
    int32_t tbfull, tbrem;  // batched passes of this chunk: tbfull of depth tbh, then one of depth tbrem
    uint32_t tbg, tbw; // 2D temporal blocking, few sites: chunk groups per site, chunks per group (the last may have fewer)
    uint32_t tpb;      // few sites: threads per group
    double *partial;   // [pslots][tiles][4]
    double *dots;      // [K+1][4] = (nn.hi, nn.lo, nm.hi, nm.lo)
    double *mu;        // [M]
    const uint32_t *colsite;   // column solves: the site of each column's unit start vector
};

// ---------------------------------------------------------------------------
// global-memory access with a uniform base and a 32-bit (or, for buffers of
// 4 GiB and more, 64-bit) byte offset
// ---------------------------------------------------------------------------
template <typename S, bool WIDE> struct Mem {
    typedef typename V16<S>::T T;
    typedef S S2 __attribute__((ext_vector_type(2)));
    static __device__ __forceinline__ const KPM_GLOBAL char *at(const void *b, uint32_t chunk)
    {
        if (WIDE) return (const KPM_GLOBAL char *)b + ((uint64_t)chunk << 4);
        return (const KPM_GLOBAL char *)b + (chunk << 4);
    }
    static __device__ __forceinline__ T ld(const void *b, uint32_t chunk) { return *(const KPM_GLOBAL T *)at(b, chunk); }
    static __device__ __forceinline__ T ld_nt(const void *b, uint32_t chunk)
    {
        return __builtin_nontemporal_load((const KPM_GLOBAL T *)at(b, chunk));
    }
    static __device__ __forceinline__ void st_nt(void *b, uint32_t chunk, T v)
    {
        __builtin_nontemporal_store(v, (KPM_GLOBAL T *)at(b, chunk));
    }
    // streamed access of r_{n-1} / r_{n+1}: non-temporal (NT) or cached
    template <bool NT> static __device__ __forceinline__ T ld_s(const void *b, uint32_t chunk)
    {
        if (NT) return ld_nt(b, chunk);
        return ld(b, chunk);
    }
    template <bool NT> static __device__ __forceinline__ void st_s(void *b, uint32_t chunk, T v)
    {
        if (NT) st_nt(b, chunk, v);
        else st(b, chunk, v);
    }
    static __device__ __forceinline__ void st(void *b, uint32_t chunk, T v) { *(KPM_GLOBAL T *)at(b, chunk) = v; }
    // element e of an array of S
    static __device__ __forceinline__ S lds(const void *b, uint32_t e)
    {
        if (WIDE) return *(const KPM_GLOBAL S *)((const KPM_GLOBAL char *)b + (uint64_t)e * sizeof(S));
        return *(const KPM_GLOBAL S *)((const KPM_GLOBAL char *)b + e * (uint32_t)sizeof(S));
    }
    // complex element e of an array of S pairs
    static __device__ __forceinline__ S2 ldc(const void *b, uint32_t e)
    {
        if (WIDE) return *(const KPM_GLOBAL S2 *)((const KPM_GLOBAL char *)b + (uint64_t)e * (2 * sizeof(S)));
        return *(const KPM_GLOBAL S2 *)((const KPM_GLOBAL char *)b + e * (uint32_t)(2 * sizeof(S)));
    }
};

// ---------------------------------------------------------------------------
// arithmetic policies
// FP64 follows the oracle's order with no fused operations (the library is
// compiled with -ffp-contract=off), so the FP64 vectors are bitwise equal to
// a plain sequential evaluation.  FP32 uses fma freely.
// ---------------------------------------------------------------------------
template <typename S> struct Arith;
template <> struct Arith<double> {
    typedef V16<double>::T T;
    static __device__ __forceinline__ T mac(T acc, double h, T v) { return acc + h * v; }
    static __device__ __forceinline__ void cmul(double &ar, double &ai, double hr, double hi, double vr, double vi)
    {
        ar = hr * vr - hi * vi;
        ai = hr * vi + hi * vr;
    }
    static __device__ __forceinline__ void cmac(double &ar, double &ai, double hr, double hi, double vr, double vi)
    {
        ar = ar + (hr * vr - hi * vi);
        ai = ai + (hr * vi + hi * vr);
    }
};
template <> struct Arith<float> {
    typedef V16<float>::T T;
    static __device__ __forceinline__ T mac(T acc, float h, T v)
    {
        T hv = h;
        return __builtin_elementwise_fma(hv, v, acc);
    }
    static __device__ __forceinline__ void cmul(float &ar, float &ai, float hr, float hi, float vr, float vi)
    {
        ar = fmaf(hr, vr, -hi * vi);
        ai = fmaf(hr, vi, hi * vr);
    }
    static __device__ __forceinline__ void cmac(float &ar, float &ai, float hr, float hi, float vr, float vi)
    {
        ar = fmaf(hr, vr, fmaf(-hi, vi, ar));
        ai = fmaf(hr, vi, fmaf(hi, vr, ai));
    }
};

// 2 v - w in one rounding (2 v is exact, so this is the value of the two operations)
template <typename T> __device__ __forceinline__ T two_minus(T v, T w)
{
    return __builtin_elementwise_fma((T)(2), v, -w);
}

// Dot-product accumulators: (sum, error) pairs in FP64 for FP64 vectors; for
// FP32 vectors the products are exact in FP64 and a plain FP64 sum suffices.
// (x0 + x1, x2 + x3) are the two sums.
template <typename S> struct Dots;
template <> struct Dots<double> {
    double s0 = 0.0, c0 = 0.0, s1 = 0.0, c1 = 0.0;
    static constexpr int NV = 4;   // values save() keeps
    __device__ __forceinline__ Dots() {}
    __device__ __forceinline__ explicit Dots(const double (&h)[NV][BLOCK])
        : s0(h[0][threadIdx.x]), c0(h[1][threadIdx.x]), s1(h[2][threadIdx.x]), c1(h[3][threadIdx.x]) {}
    __device__ __forceinline__ void save(double (&h)[NV][BLOCK]) const
    {
        h[0][threadIdx.x] = s0;
        h[1][threadIdx.x] = c0;
        h[2][threadIdx.x] = s1;
        h[3][threadIdx.x] = c1;
    }
    __device__ __forceinline__ void add(V16<double>::T o, V16<double>::T v)
    {
#pragma unroll
        for (int l = 0; l < 2; ++l) {
            dot2_acc(s0, c0, o[l], o[l]);
            dot2_acc(s1, c1, o[l], v[l]);
        }
    }
    __device__ __forceinline__ void first(V16<double>::T o, V16<double>::T v)   // add() to empty sums
    {
        dot2_first(s0, c0, o[0], o[0]);
        dot2_first(s1, c1, o[0], v[0]);
        dot2_acc(s0, c0, o[1], o[1]);
        dot2_acc(s1, c1, o[1], v[1]);
    }
    __device__ __forceinline__ void norm_only(V16<double>::T o)
    {
#pragma unroll
        for (int l = 0; l < 2; ++l) dot2_acc(s0, c0, o[l], o[l]);
    }
    __device__ __forceinline__ void cross_only(V16<double>::T o, V16<double>::T v)
    {
#pragma unroll
        for (int l = 0; l < 2; ++l) dot2_acc(s1, c1, o[l], v[l]);
    }
    __device__ __forceinline__ double x0() const { return s0; }
    __device__ __forceinline__ double x1() const { return c0; }
    __device__ __forceinline__ double x2() const { return s1; }
    __device__ __forceinline__ double x3() const { return c1; }
    static constexpr bool DD = true;
};
template <> struct Dots<float> {
    double s0 = 0.0, s1 = 0.0;
    static constexpr int NV = 2;
    __device__ __forceinline__ Dots() {}
    __device__ __forceinline__ explicit Dots(const double (&h)[NV][BLOCK]) : s0(h[0][threadIdx.x]), s1(h[1][threadIdx.x]) {}
    __device__ __forceinline__ void save(double (&h)[NV][BLOCK]) const
    {
        h[0][threadIdx.x] = s0;
        h[1][threadIdx.x] = s1;
    }
    __device__ __forceinline__ void add(V16<float>::T o, V16<float>::T v)
    {
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            double a = (double)o[l];
            s0 = fma(a, a, s0);
            s1 = fma(a, (double)v[l], s1);
        }
    }
    __device__ __forceinline__ void first(V16<float>::T o, V16<float>::T v) { add(o, v); }
    __device__ __forceinline__ void norm_only(V16<float>::T o)
    {
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            double a = (double)o[l];
            s0 = fma(a, a, s0);
        }
    }
    __device__ __forceinline__ double x0() const { return s0; }
    __device__ __forceinline__ double x1() const { return 0.0; }
    __device__ __forceinline__ double x2() const { return s1; }
    __device__ __forceinline__ double x3() const { return 0.0; }
    static constexpr bool DD = false;
};
// The dot products of each vector of a chunk by itself (NV vectors): for FP64 vectors two
// (sum, error) pairs each, for FP32 vectors two sums.  value(k): vector k / V1, value k % V1 of
// V1 = 4 or 2.
template <typename S, bool CPLX> struct ColDots;
template <bool CPLX> struct ColDots<float, CPLX> {
    static constexpr int NV = CPLX ? 2 : 4, V1 = 2;
    double s[NV][2] = {};
    __device__ __forceinline__ void add(V16<float>::T o, V16<float>::T v)
    {
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            double *a = s[CPLX ? l / 2 : l];
            a[0] = fma((double)o[l], (double)o[l], a[0]);
            a[1] = fma((double)o[l], (double)v[l], a[1]);
        }
    }
    __device__ __forceinline__ double value(int k) const { return s[k / 2][k % 2]; }
};
template <bool CPLX> struct ColDots<double, CPLX> {
    static constexpr int NV = CPLX ? 1 : 2, V1 = 4;
    Dots<double> d[NV];
    __device__ __forceinline__ void add(V16<double>::T o, V16<double>::T v)
    {
#pragma unroll
        for (int l = 0; l < 2; ++l) {
            Dots<double> &a = d[CPLX ? 0 : l];
            dot2_acc(a.s0, a.c0, o[l], o[l]);
            dot2_acc(a.s1, a.c1, o[l], v[l]);
        }
    }
    __device__ __forceinline__ double value(int k) const
    {
        const Dots<double> &a = d[k / 4];
        return k % 4 == 0 ? a.x0() : (k % 4 == 1 ? a.x1() : (k % 4 == 2 ? a.x2() : a.x3()));
    }
};

// ---------------------------------------------------------------------------
// sums over a wavefront
// ---------------------------------------------------------------------------
// Two sums (x0 + x1, x2 + x3; double-doubles when DD, else x0 and x2 alone) of up to four
// accumulators.  A level of the tree adds each lane's value and that of the lane 32, 16, 8, 4,
// 2 or 1 away.  At the first three the two lanes hand each other half of what they have: the
// lower 32 lanes go on with the first sum, the upper 32 with the second; the even rows of 16
// lanes with one accumulator of a pair, the odd ones with the other; the lower and upper 8 lanes
// of a row with the first and second pair.  Four accumulators so take ten additions of 11
// operations, and no exchange goes through the LDS.  (With ds_bpermute shuffles it was 48 of 20
// and 192 shuffles of 24 cycles, most of a step of the few-site solves.)  An accumulator's
// tree, and so its bits, are the same whatever others share the exchanges.
template <bool DD> __device__ __forceinline__ dd wave_add(dd x, dd y)
{
    if (DD) return dd_sum(x, y);
    return dd{x.hi + y.hi, 0.0};
}
template <bool DD, int N> __device__ __forceinline__ dd wave_ror(dd p)
{
    return dd{row_ror<N>(p.hi), DD ? row_ror<N>(p.lo) : 0.0};
}
template <bool DD> __device__ __forceinline__ dd wave_halves(dd p, dd q)
{
    swap_halves(p.hi, q.hi);
    if (DD) swap_halves(p.lo, q.lo);
    return wave_add<DD>(p, q);
}
template <bool DD> __device__ __forceinline__ dd wave_rows(dd p, dd q)
{
    swap_rows(p.hi, q.hi);
    if (DD) swap_rows(p.lo, q.lo);
    return wave_add<DD>(p, q);
}
template <bool DD> struct WaveSums {
    dd r{0.0, 0.0}, t{0.0, 0.0};   // the last accumulator or pair; the first pair
    // accumulator k = 0 .. 3, in order (k the same in every lane)
    __device__ __forceinline__ void add(int k, double x0, double x1, double x2, double x3)
    {
        const dd h = wave_halves<DD>(dd{x0, x1}, dd{x2, x3});
        if ((k & 1) == 0) r = h;
        else if (k == 1) t = wave_rows<DD>(r, h);
        else r = wave_rows<DD>(r, h);
    }
    template <typename A> __device__ __forceinline__ void add(int k, const A &d) { add(k, d.x0(), d.x1(), d.x2(), d.x3()); }
    // the sums of the n accumulators added: accumulator k as four doubles (hi, lo, hi, lo) at dst + k * pitch
    __device__ __forceinline__ void finish(int n, double *dst, size_t pitch)
    {
        dd u = n == 2 ? t : r;
        if (n & 1) u = wave_rows<DD>(u, u);
        const dd v = n == 1 ? u : t;
        const int lane = threadIdx.x & 63;
        const bool up = (lane & 8) != 0;
        const dd keep{up ? u.hi : v.hi, up ? u.lo : v.lo}, give{up ? v.hi : u.hi, up ? v.lo : u.lo};
        dd p = wave_add<DD>(keep, wave_ror<DD, 8>(give));
        p = wave_add<DD>(p, wave_ror<DD, 4>(p));   // valid in lanes 4 .. 7 of each 8,
        p = wave_add<DD>(p, wave_ror<DD, 2>(p));   // ... 6 and 7,
        p = wave_add<DD>(p, wave_ror<DD, 1>(p));   // ... 7
        const int k = ((lane >> 4) & 1) + ((lane >> 3) & 1) * 2;
        if ((lane & 7) == 7 && k < n) {
            double *o = dst + (size_t)k * pitch + ((lane & 32) >> 4);
            o[0] = p.hi;
            o[1] = p.lo;
        }
    }
};
template <bool DD>
__device__ __forceinline__ void wave_reduce_store(double x0, double x1, double x2, double x3, double *dst)
{
    WaveSums<DD> s;
    s.add(0, x0, x1, x2, x3);
    s.finish(1, dst, 0);
}
template <typename A> __device__ __forceinline__ void wave_reduce_store(const A &d, double *dst)
{
    wave_reduce_store<A::DD>(d.x0(), d.x1(), d.x2(), d.x3(), dst);
}

// Sum (x0 + x1, x2 + x3) over the block in a fixed order, stored as four doubles
// (hi, lo, hi, lo) at dst; thread 0 adds the waves' first sums, thread 1 the second.
template <bool DD, int NT = BLOCK>
__device__ __forceinline__ void block_reduce_store(double x0, double x1, double x2, double x3, double *dst)
{
    __shared__ double red[NT / 64][4];
    wave_reduce_store<DD>(x0, x1, x2, x3, red[threadIdx.x >> 6]);
    __syncthreads();
    if (threadIdx.x < 2) {
        const int o = threadIdx.x * 2;
        dd a{red[0][o], red[0][o + 1]};
#pragma unroll
        for (int k = 1; k < NT / 64; ++k) {
            if (DD) a = dd_sum(a, dd{red[k][o], red[k][o + 1]});
            else a.hi += red[k][o];
        }
        dst[o] = a.hi;
        dst[o + 1] = a.lo;
    }
    __syncthreads();
}
template <int NT = BLOCK, typename A> __device__ __forceinline__ void block_reduce_store(const A &d, double *dst)
{
    block_reduce_store<A::DD, NT>(d.x0(), d.x1(), d.x2(), d.x3(), dst);
}

// The block's sums of `n` segments from their waves' (red[k][wave]), added in the order of
// block_reduce_store: segment k's four doubles go to dst + k * pitch.
constexpr int RUN_MAX = 4;   // segments per run
template <bool DD>
__device__ __forceinline__ void reduce_run(const double (&red)[RUN_MAX][BLOCK / 64][4], uint32_t n, double *dst,
                                           size_t pitch)
{
    if (threadIdx.x >= 2 * n) return;
    const uint32_t k = threadIdx.x >> 1, o = (threadIdx.x & 1u) * 2;
    dd a{red[k][0][o], red[k][0][o + 1]};
#pragma unroll
    for (int w = 1; w < BLOCK / 64; ++w) {
        if (DD) a = dd_sum(a, dd{red[k][w][o], red[k][w][o + 1]});
        else a.hi += red[k][w][o];
    }
    dst[k * pitch + o] = a.hi;
    dst[k * pitch + o + 1] = a.lo;
}

// ---------------------------------------------------------------------------
// mapping of an instance's blocks to its work items
// ---------------------------------------------------------------------------
// Work items of an instance handled by block `block` of the launch.  An item is (unit, seg)
// with unit a column tile (march), tile (flat) or tile of a blocked pass.  Local item it, for
// it = first, first + stride, ... below count, is the one that at() names; the kernels and the
// host check take it from there, so that every split covers every item once.  XCD split (block b
// runs on XCD b mod 8):
//   xcd == 2: XCD x owns segments [x*segs/8, (x+1)*segs/8) of every unit, so a
//             whole plane stays in one L2;
//   xcd == 1: XCD x owns units [x*units/8, (x+1)*units/8) of every segment;
//   xcd == 3: XCD x owns the x-th eighth of all items in the order of seg, then unit
//             (equal to one item, whatever the units and segments);
//   xcd == 4: this table entry covers items [q0, q1) of its instance, in that order;
//   xcd == 0: no split.
class ItemRange {
    uint32_t ub, nu, sb, base;   // first unit, units, first segment; offset in their items

public:
    uint32_t first, stride, count;
    __host__ __device__ __forceinline__ ItemRange(const Inst &I, uint32_t block, uint32_t units, uint32_t segs)
        : ub(0), nu(units), sb(0), base(0)
    {
        const uint32_t bl = (block - I.block0) / I.bstride;
        uint32_t ns = segs;
        first = bl;
        stride = I.nb;
        if (I.xcd == 4) {
            base = I.q0;
            count = I.q1 - I.q0;
            return;
        }
        if (I.xcd) {
            const uint32_t x8 = bl & 7u;
            first = bl >> 3;
            stride = I.nb >> 3;
            if (I.xcd == 3) {
                const uint64_t all = (uint64_t)units * segs;
                base = (uint32_t)((all * x8) >> 3);
                count = (uint32_t)((all * (x8 + 1)) >> 3) - base;
                return;
            }
            if (I.xcd == 2) {
                sb = (uint32_t)(((uint64_t)segs * x8) >> 3);
                ns = (uint32_t)(((uint64_t)segs * (x8 + 1)) >> 3) - sb;
            } else {
                ub = (uint32_t)(((uint64_t)units * x8) >> 3);
                nu = (uint32_t)(((uint64_t)units * (x8 + 1)) >> 3) - ub;
            }
        }
        count = nu * ns;
    }
    // unit and segment of local item `it`
    __host__ __device__ __forceinline__ void at(uint32_t it, uint32_t &unit, uint32_t &sg) const
    {
        const uint32_t q = base + it, sl = q / nu;
        sg = sb + sl;
        unit = ub + (q - sl * nu);
    }
};
// The block's items of an instance of the given mode.  A march item is a run of I.run segments.
__host__ __device__ __forceinline__ ItemRange item_range(const Inst &I, int mode, uint32_t block)
{
    switch (mode) {
    case MODE_MARCH: return ItemRange(I, block, I.nct, (I.nseg + I.run - 1) / I.run);
    case MODE_TB: return ItemRange(I, block, I.nct * I.tbg, I.nseg);
    case MODE_TB3: return ItemRange(I, block, I.nct * I.C, I.nseg);
    default: return ItemRange(I, block, I.tiles, 1);
    }
}

// ---------------------------------------------------------------------------
// start vectors
// ---------------------------------------------------------------------------
// The four Philox words for site i and vectors 4*rq .. 4*rq+3.
__device__ __forceinline__ void start_words(uint64_t seed, uint64_t instance, uint32_t i, uint32_t rq, uint64_t w[4])
{
    uint64_t c0 = i, c1 = rq, c2 = instance, c3 = 0;
    philox4x64_10(c0, c1, c2, c3, seed, 4);
    w[0] = c0; w[1] = c1; w[2] = c2; w[3] = c3;
}
// Random phases: xi = e^{i phi}, phi = 2 pi k / 2^30 with k = word >> 34,
// formed as the ordered product (ascending j) of w_j = e^{2 pi i 2^j / 2^30}
// over the set bits of k.  The factors are computed on the host from the
// half-angle recurrence with IEEE operations only and placed in constant
// memory, so the phases are reproducible bit for bit on any IEEE machine.
constexpr int PHASE_BITS = 30;
__constant__ double kpm_phase_w[PHASE_BITS][2];

// The phases of NC vectors at once, k[l] = the top PHASE_BITS bits of their
// words: every lane runs through all PHASE_BITS factors (uniform, so they come
// from scalar loads) and takes the product z * w_j only where bit j of its k is
// set, so the factors multiply in ascending j as defined above.  z starts at 1:
// 1 * w_j gives w_j exactly (w_j has no zero of negative sign), the first
// factor itself, and k = 0 gives 1.
template <int NC>
__device__ __forceinline__ void phase_products(const uint32_t (&k)[NC], double (&zr)[NC], double (&zi)[NC])
{
#pragma unroll
    for (int l = 0; l < NC; ++l) {
        zr[l] = 1.0;
        zi[l] = 0.0;
    }
#pragma unroll 2
    for (int j = 0; j < PHASE_BITS; ++j) {
        const double wr = kpm_phase_w[j][0], wi = kpm_phase_w[j][1];
#pragma unroll
        for (int l = 0; l < NC; ++l) {
            const double tr = zr[l] * wr - zi[l] * wi;
            const double ti = zr[l] * wi + zi[l] * wr;
            const bool set = (k[l] >> j) & 1u;
            zr[l] = set ? tr : zr[l];
            zi[l] = set ? ti : zi[l];
        }
    }
}

// (re, im) of xi_{r,i} given its Philox word.
__device__ __forceinline__ void start_value(int vec, uint64_t word, uint64_t instance, uint32_t N, uint32_t i,
                                            uint32_t r, double &re, double &im)
{
    if (vec == VEC_RADEMACHER) {
        re = (word >> 63) ? -1.0 : 1.0;
        im = 0.0;
    } else if (vec == VEC_PHASE) {
        const uint32_t k[1] = {(uint32_t)(word >> (64 - PHASE_BITS))};
        double zr[1], zi[1];
        phase_products<1>(k, zr, zi);
        re = zr[0];
        im = zi[0];
    } else {
        uint64_t j = (instance + (uint64_t)r) % (uint64_t)N;
        re = (j == (uint64_t)i) ? 1.0 : 0.0;
        im = 0.0;
    }
}

// Chunk c of site i of the start block.
template <typename S>
__device__ __forceinline__ typename V16<S>::T start_chunk(const Inst &I, uint32_t i, uint32_t c)
{
    typedef typename V16<S>::T T;
    constexpr int W = V16<S>::W;
    const uint32_t k0 = c * W;                  // first scalar of the chunk
    const uint32_t r0 = I.cplx ? k0 / 2 : k0;   // first vector of the chunk (all in one Philox block)
    uint64_t w[4] = {0, 0, 0, 0};
    if (I.vec != VEC_UNIT) start_words(I.seed, I.instance, i, r0 / 4, w);
    T v;
    if (I.cplx && I.vec == VEC_PHASE) {
        // the chunk's W / 2 phases in one pass over the factors
        constexpr int NC = W / 2;
        uint32_t k[NC];
        double zr[NC], zi[NC];
#pragma unroll
        for (int l = 0; l < NC; ++l) k[l] = (uint32_t)(w[(r0 + l) & 3] >> (64 - PHASE_BITS));
        phase_products<NC>(k, zr, zi);
#pragma unroll
        for (int l = 0; l < NC; ++l) {
            const bool in = r0 + l < (uint32_t)I.R;
            v[2 * l] = in ? (S)zr[l] : (S)0;
            v[2 * l + 1] = in ? (S)zi[l] : (S)0;
        }
    } else if (I.cplx) {
#pragma unroll
        for (int l = 0; l < W / 2; ++l) {
            const uint32_t r = r0 + l;
            double re = 0.0, im = 0.0;
            if (r < (uint32_t)I.R) start_value(I.vec, w[r & 3], I.instance, I.N, i, r, re, im);
            v[2 * l] = (S)re;
            v[2 * l + 1] = (S)im;
        }
    } else {
#pragma unroll
        for (int l = 0; l < W; ++l) {
            const uint32_t r = r0 + l;
            double re = 0.0, im = 0.0;
            if (r < (uint32_t)I.R) start_value(I.vec, w[r & 3], I.instance, I.N, i, r, re, im);
            v[l] = (S)re;
        }
    }
    return v;
}

// r_0 into buf0 and the partials of <r_0|r_0>, over the same work items as the
// recursion step of the instance's mode.
template <typename S, bool WIDE>
__global__ __launch_bounds__(BLOCK) void k_init(const Inst *__restrict__ tab, const uint32_t *__restrict__ bmap)
{
    typedef Mem<S, WIDE> G;
    const uint32_t h = bmap ? bmap[blockIdx.x] : 0u;
    if (h == NO_INSTANCE) return;
    const Inst I = tab[h];
    if (I.step0 != 0) return;
    double *part = I.partial;   // slot 0
    if (I.mode == MODE_MARCH) {
        const ItemRange ir = item_range(I, MODE_MARCH, blockIdx.x);
        const uint32_t PC = I.P * I.C;
        for (uint32_t it = ir.first; it < ir.count; it += ir.stride) {
            uint32_t ct, rn;
            ir.at(it, ct, rn);
            const uint32_t e = ct * BLOCK + threadIdx.x;
            for (uint32_t sg = rn * I.run; sg < min((rn + 1) * I.run, I.nseg); ++sg) {
                Dots<S> acc;
                if (e < PC) {
                    const uint32_t p = fdiv(e, I.fC), c = e - p * I.C;
                    const uint32_t m0 = sg * I.S, m1 = min(m0 + I.S, I.Lm);
                    for (uint32_t m = m0; m < m1; ++m) {
                        const uint32_t i = p + I.P * m;
                        const auto v = start_chunk<S>(I, i, c);
                        G::st(I.buf0, i * I.C + c, v);
                        acc.norm_only(v);
                    }
                }
                block_reduce_store(acc, part + (size_t)(sg * I.nct + ct) * 4);
            }
        }
    } else {
        const ItemRange ir = item_range(I, MODE_FLAT, blockIdx.x);
        for (uint32_t it = ir.first; it < ir.count; it += ir.stride) {
            uint32_t t, sg;
            ir.at(it, t, sg);
            Dots<S> acc;
            for (int u = 0; u < I.tpt; ++u) {
                const uint32_t e = t * (uint32_t)(BLOCK * I.tpt) + (uint32_t)(u * BLOCK) + threadIdx.x;
                if (e < I.nel) {
                    const uint32_t i = fdiv(e, I.fC), c = e - i * I.C;
                    const auto v = start_chunk<S>(I, i, c);
                    G::st(I.buf0, e, v);
                    acc.norm_only(v);
                }
            }
            block_reduce_store(acc, part + (size_t)t * 4);
        }
    }
}

// ---------------------------------------------------------------------------
// operator application on one chunk, in the oracle's slot order
// (diagonal, -x, +x, -y, +y[, -z, +z])
// ---------------------------------------------------------------------------
// Real hopping: a = d*v + h*(v_-x) + h*(v_+x) + ...
template <typename S, int NS>
__device__ __forceinline__ typename V16<S>::T apply_real(bool hd, S d, S h, typename V16<S>::T v,
                                                         const typename V16<S>::T (&nb)[NS])
{
    typedef Arith<S> A;
    typename V16<S>::T a;
    if (hd) {
        a = d * v;
        a = A::mac(a, h, nb[0]);
    } else {
        a = h * nb[0];
    }
#pragma unroll
    for (int s = 1; s < NS; ++s) a = A::mac(a, h, nb[s]);
    return a;
}
// Complex hopping: slot s has coefficient (hr[s], hi[s]).
template <typename S, int NS>
__device__ __forceinline__ typename V16<S>::T apply_cplx(bool hd, S d, typename V16<S>::T v,
                                                         const typename V16<S>::T (&nb)[NS], const S (&hr)[NS],
                                                         const S (&hi)[NS])
{
    typedef Arith<S> A;
    constexpr int W = V16<S>::W;
    typename V16<S>::T out;
#pragma unroll
    for (int l = 0; l < W / 2; ++l) {
        S ar, ai;
        if (hd) {
            ar = d * v[2 * l];
            ai = d * v[2 * l + 1];
            A::cmac(ar, ai, hr[0], hi[0], nb[0][2 * l], nb[0][2 * l + 1]);
        } else {
            A::cmul(ar, ai, hr[0], hi[0], nb[0][2 * l], nb[0][2 * l + 1]);
        }
#pragma unroll
        for (int s = 1; s < NS; ++s) A::cmac(ar, ai, hr[s], hi[s], nb[s][2 * l], nb[s][2 * l + 1]);
        out[2 * l] = ar;
        out[2 * l + 1] = ai;
    }
    return out;
}

// Column solves: the sums of each vector over the block's threads, to dst[column][4].  The
// threads of chunk c of their site are C apart; the values go through the LDS.  As many threads
// of a wave as there are take one sum together (with one each, two sites on a 64^3 lattice
// waited for 256 additions in a row: 27.3 us per step).
template <typename A, int NB>
__device__ __forceinline__ void column_sums(const Inst &I, const A &acc, double (&lds)[NB][BLOCK], uint32_t ct, double *dst)
{
#pragma unroll
    for (int k = 0; k < NB; ++k) lds[k][threadIdx.x] = acc.value(k);
    __syncthreads();
    const uint32_t C = I.C, c0 = ct * BLOCK - fdiv(ct * BLOCK, I.fC) * C;   // the chunk of thread 0
    const uint32_t Q = C * A::NV * 2;   // sums: two of each vector
    uint32_t lp = 6;                    // log2 of the threads per sum: at most half the block's for all
    while (lp > 0 && Q << lp > BLOCK / 2) --lp;
    const uint32_t P = 1u << lp, part = threadIdx.x & (P - 1);
    for (uint32_t q = threadIdx.x >> lp; q < Q; q += BLOCK >> lp) {
        const uint32_t c = q / (A::NV * 2), v = (q / 2) % A::NV, o = q & 1u, col = c * A::NV + v;
        const uint32_t k = v * A::V1 + o * (A::V1 / 2);
        dd a{0.0, 0.0};
        for (uint32_t t = (c < c0 ? c + C - c0 : c - c0) + part * C; t < BLOCK; t += P * C) {
            if constexpr (A::V1 == 4) a = dd_sum(a, dd{lds[k][t], lds[k + 1][t]});
            else a = dd_sum(a, lds[k][t]);
        }
        for (uint32_t off = P >> 1; off > 0; off >>= 1)
            a = dd_sum(a, dd{__shfl_xor(a.hi, (int)off, 64), __shfl_xor(a.lo, (int)off, 64)});
        if (part == 0 && col < (uint32_t)I.R) {
            dst[col * 4 + 2 * o] = a.hi;
            dst[col * 4 + 2 * o + 1] = a.lo;
        }
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// the fused recursion step, march form (lattices)
// ---------------------------------------------------------------------------
// COLS: the dot products of every vector by itself (unit start vectors at chosen sites, R of
// them in one solve), one partial per item and column; an item is one segment.
template <typename S, int OPK, bool WIDE, bool NT, bool COLS = false>
__global__ __launch_bounds__(BLOCK) void k_step_march(const Inst *__restrict__ tab,
                                                      const uint32_t *__restrict__ bmap, int32_t k)
{
    typedef typename V16<S>::T T;
    typedef Mem<S, WIDE> G;
    typedef typename Mem<S, WIDE>::S2 S2;
    constexpr bool D3 = (OPK == OP_REAL3 || OPK == OP_SPIN3);
    constexpr bool SPIN = (OPK == OP_SPIN2 || OPK == OP_SPIN3);
    constexpr int DIM = D3 ? 3 : 2;
    constexpr int NS = 2 * DIM;
    const uint32_t h = bmap ? bmap[blockIdx.x] : 0u;
    if (h == NO_INSTANCE) return;
    const Inst I = tab[h];
    const int32_t n = I.step0 + k;
    if (n < 0 || n >= I.K) return;
    const void *cur = (n & 1) ? I.buf1 : I.buf0;
    void *nxt = (n & 1) ? I.buf0 : I.buf1;
    const bool first = (n == 0);
    const bool hd = I.has_diag;
    S hop = 0;
    if (!SPIN) hop = G::lds(I.hop, 0);
    double *part = I.partial + (size_t)((n + 1) % I.pslots) * I.tiles * 4 * (COLS ? (uint32_t)I.R : 1u);
    const uint32_t C = I.C, P = I.P, Lx = I.Lx, Ly = I.Ly, Lm = I.Lm;
    const uint32_t PC = P * C;
    typedef std::conditional_t<COLS, ColDots<S, SPIN>, Dots<S>> Acc;
    __shared__ double red[COLS ? 1 : RUN_MAX][BLOCK / 64][4];   // wave sums of the run's segments
    // a thread's sums of the even segment of a pair, reduced with the odd one's (in the LDS:
    // four more VGPRs would cost the FP32 3D spin kernel one of its 7 waves per SIMD; all four
    // segments of a run reduced at its end measured 1-4% slower)
    __shared__ double held[COLS ? ColDots<S, SPIN>::NV * ColDots<S, SPIN>::V1 : Dots<S>::NV][BLOCK];
    const ItemRange ir = item_range(I, MODE_MARCH, blockIdx.x);
    for (uint32_t it = ir.first; it < ir.count; it += ir.stride) {
        uint32_t ct, rn;
        ir.at(it, ct, rn);
        const uint32_t e = ct * BLOCK + threadIdx.x;
        const bool active = e < PC;
        const uint32_t p = active ? fdiv(e, I.fC) : 0u, c = active ? e - p * C : 0u;
        uint32_t x = p, y = 0;
        if constexpr (D3) {
            y = fdiv(p, I.fLx);
            x = p - y * Lx;
        }
        const uint32_t pxm = (x == 0) ? p + (Lx - 1) : p - 1;
        const uint32_t pxp = (x == Lx - 1) ? p - (Lx - 1) : p + 1;
        uint32_t pym = 0, pyp = 0;
        if constexpr (D3) {
            pym = (y == 0) ? p + (Ly - 1) * Lx : p - Lx;
            pyp = (y == Ly - 1) ? p - (Ly - 1) * Lx : p + Lx;
        }
        const uint32_t s0 = rn * I.run, s1 = min(s0 + I.run, I.nseg);
        const uint32_t r0 = s0 * I.S, r1 = min(s1 * I.S, Lm);   // planes of the run
        // Odd segments march downwards, so that two adjacent segments reach
        // their common boundary planes at about the same time and the second
        // read of a halo plane hits in L2.  (Runs of several segments march upwards.)
        const bool down = I.alt && (s0 & 1u) != 0;
        const uint32_t mfirst = down ? r1 - 1 : r0;
        const uint32_t mbefore = down ? ((r1 == Lm) ? 0 : r1) : ((r0 == 0) ? Lm - 1 : r0 - 1);
        // window: vb = plane behind (in march order), v0 = current plane
        T vb = G::ld(cur, (p + P * mbefore) * C + c);
        T v0 = G::ld(cur, (p + P * mfirst) * C + c);
        // march-axis bond linking plane mbefore and mfirst (H~_{(m-1), m} stored at plane m-1)
        S2 bb = {0, 0};
        if (SPIN) bb = G::ldc(I.bond, (p + P * (down ? mfirst : mbefore)) * DIM + (DIM - 1));
        for (uint32_t sg = s0; sg < s1; ++sg) {
            Acc acc;
            const uint32_t m0 = sg * I.S, m1 = min(m0 + I.S, Lm);
            if (active)
                for (uint32_t s_ = 0; s_ < m1 - m0; ++s_) {
                    const uint32_t m = down ? m1 - 1 - s_ : m0 + s_;
                    const uint32_t ma = down ? ((m == 0) ? Lm - 1 : m - 1) : ((m + 1 == Lm) ? 0 : m + 1);  // plane ahead
                    const uint32_t i = p + P * m;
                    const uint32_t ch = i * C + c;
                    const T va = G::ld(cur, (p + P * ma) * C + c);
                    T nb[NS];
                    nb[0] = G::ld(cur, (pxm + P * m) * C + c);
                    nb[1] = G::ld(cur, (pxp + P * m) * C + c);
                    if constexpr (D3) {
                        nb[2] = G::ld(cur, (pym + P * m) * C + c);
                        nb[3] = G::ld(cur, (pyp + P * m) * C + c);
                    }
                    // slots -march, +march in the fixed order
                    nb[NS - 2] = down ? va : vb;
                    nb[NS - 1] = down ? vb : va;
                    T prev;
                    if (!first) prev = G::template ld_s<NT>(nxt, ch);
                    const S d = hd ? G::lds(I.diag, i) : (S)0;
                    T out;
                    if (!SPIN) {
                        out = apply_real<S, NS>(hd, d, hop, v0, nb);
                    } else {
                        S hr[NS], hi[NS];
                        const S2 bxm = G::ldc(I.bond, (pxm + P * m) * DIM + 0);
                        const S2 bxp = G::ldc(I.bond, i * DIM + 0);
                        hr[0] = bxm[0]; hi[0] = -bxm[1];
                        hr[1] = bxp[0]; hi[1] = bxp[1];
                        if constexpr (D3) {
                            const S2 bym = G::ldc(I.bond, (pym + P * m) * DIM + 1);
                            const S2 byp = G::ldc(I.bond, i * DIM + 1);
                            hr[2] = bym[0]; hi[2] = -bym[1];
                            hr[3] = byp[0]; hi[3] = byp[1];
                        }
                        // the other march-axis bond: H~_{m, m+1} (up) lives at plane m,
                        // H~_{m-1, m} (down) at plane m-1 = the plane ahead
                        const S2 ba = G::ldc(I.bond, (p + P * (down ? ma : m)) * DIM + (DIM - 1));
                        const S2 bminus = down ? ba : bb;   // H~_{m-1,m}: conjugated for slot -march
                        const S2 bplus = down ? bb : ba;    // H~_{m,m+1}
                        hr[NS - 2] = bminus[0]; hi[NS - 2] = -bminus[1];
                        hr[NS - 1] = bplus[0]; hi[NS - 1] = bplus[1];
                        out = apply_cplx<S, NS>(hd, d, v0, nb, hr, hi);
                        bb = ba;
                    }
                    if (!first) out = two_minus(out, prev);
                    G::template st_s<NT>(nxt, ch, out);
                    acc.add(out, v0);
                    vb = v0;
                    v0 = va;
                }
            if constexpr (COLS) {
                column_sums(I, acc, held, ct, part + (size_t)(sg * I.nct + ct) * I.R * 4);
            } else {
                const uint32_t k = sg - s0, w = threadIdx.x >> 6;
                if (!(k & 1u) && sg + 1 < s1) {
                    acc.save(held);
                } else {
                    WaveSums<Dots<S>::DD> ws;
                    if (k & 1u) {
                        ws.add(0, Dots<S>(held));
                        ws.add(1, acc);
                        ws.finish(2, red[k - 1][w], BLOCK / 64 * 4);
                    } else {
                        ws.add(0, acc);
                        ws.finish(1, red[k][w], 0);
                    }
                }
            }
        }
        if constexpr (!COLS) {
            __syncthreads();
            reduce_run<Dots<S>::DD>(red, s1 - s0, part + (size_t)(s0 * I.nct + ct) * 4, (size_t)I.nct * 4);
            __syncthreads();
        }
    }
}

// ---------------------------------------------------------------------------
// the fused recursion step, flat form (CSR; lattices on request)
// ---------------------------------------------------------------------------
// CSR rows are walked CSR_AHEAD entries at a time: their columns and values first, then
// the gathers of r_n, all in flight together (each entry used to wait for its column, then
// for its gather: a chain of 2 nnz/N latencies with a wave's only loads).  A lane past its
// row's end, or at the stored diagonal, gathers nothing: a clamped gather repeated the last
// one from the L2 (100000 rows of 13, FP64 R = 16: 60 -> 72 us).  Entries are added in
// stored order.  Once enough waves run, the gathers are bound by the lines that the
// Infinity Cache delivers; groups of chunks per XCD, so that a group's r_n fits the L2,
// paid more for their narrower gathers than they saved, and non-temporal loads of the
// entries lost the lines that neighbouring rows share.  us per step, 1 -> 4 -> 8 entries
// at one chunk per thread and tile (before: 1 entry at four):
//   100000 rows of 13, complex FP32, R = 16     30.9 -> 29.1 -> 28.1   (45.7)
//   the same in FP64                            60.6 -> 61.2 -> 55.5   (60.1)
//   200000 rows of 17, complex FP32, R = 8     100.2 -> 74.4 -> 70.3   (70.3)
//   30000 rows of 13, complex FP32, R = 16      14.1 ->  9.9 -> 10.2   (38.0)
// The last four or fewer of a row take half as many loads: eight at a time alone, then four
// at the end (before):
//   500000 rows of 3, FP64, R = 8               34.6 -> 32.4   (31.6)
//   500000 rows of 9, FP32, R = 8               29.1 -> 24.6   (28.4)
//   100000 rows of 21, FP32, R = 16             35.8 -> 32.9   (62.4)
constexpr int CSR_AHEAD = 8;
// H~ r on chunk e, r read through ld(chunk index); v receives the chunk itself.
template <typename S, int OPK, bool WIDE, typename LD>
__device__ __forceinline__ typename V16<S>::T flat_apply(const Inst &I, uint32_t e, S hop, const LD &ld,
                                                         typename V16<S>::T &v)
{
    typedef typename V16<S>::T T;
    typedef Mem<S, WIDE> G;
    typedef typename Mem<S, WIDE>::S2 S2;
    typedef Arith<S> A;
    constexpr int W = V16<S>::W;
    const uint32_t C = I.C;
    const uint32_t i = fdiv(e, I.fC);
    const uint32_t c = e - i * C;
    v = ld(e);
    T out;
    if constexpr (OPK <= OP_SPIN3) {
        constexpr bool D3 = (OPK == OP_REAL3 || OPK == OP_SPIN3);
        constexpr bool SPIN = (OPK == OP_SPIN2 || OPK == OP_SPIN3);
        constexpr int DIM = D3 ? 3 : 2;
        constexpr int NS = 2 * DIM;
        const uint32_t Lx = I.Lx, Ly = I.Ly;
        const uint32_t yq = fdiv(i, I.fLx);
        const uint32_t x = i - yq * Lx;
        uint32_t y = yq, z = 0;
        if constexpr (D3) {
            z = fdiv(yq, I.fLy);
            y = yq - z * Ly;
        }
        uint32_t nbi[NS];
        nbi[0] = (x == 0) ? i + (Lx - 1) : i - 1;
        nbi[1] = (x == Lx - 1) ? i - (Lx - 1) : i + 1;
        nbi[2] = (y == 0) ? i + (Ly - 1) * Lx : i - Lx;
        nbi[3] = (y == Ly - 1) ? i - (Ly - 1) * Lx : i + Lx;
        if constexpr (D3) {
            const uint32_t Pz = Lx * Ly, Lz = I.Lz;
            nbi[4] = (z == 0) ? i + (Lz - 1) * Pz : i - Pz;
            nbi[5] = (z == Lz - 1) ? i - (Lz - 1) * Pz : i + Pz;
        }
        T nb[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) nb[s] = ld(nbi[s] * C + c);
        const bool hd = I.has_diag;
        const S d = hd ? G::lds(I.diag, i) : (S)0;
        if (!SPIN) {
            out = apply_real<S, NS>(hd, d, hop, v, nb);
        } else {
            S hr[NS], hi[NS];
#pragma unroll
            for (int ax = 0; ax < DIM; ++ax) {
                const S2 bm = G::ldc(I.bond, nbi[2 * ax] * DIM + ax);
                const S2 bp = G::ldc(I.bond, i * DIM + ax);
                hr[2 * ax] = bm[0]; hi[2 * ax] = -bm[1];
                hr[2 * ax + 1] = bp[0]; hi[2 * ax + 1] = bp[1];
            }
            out = apply_cplx<S, NS>(hd, d, v, nb, hr, hi);
        }
    } else {
        // CSR: the diagonal d_i first, then the off-diagonal entries in stored order
        const int64_t kb = I.row_ptr[i], ke = I.row_ptr[i + 1];
        const S d = G::lds(I.diag, i);
        T a;
#pragma unroll
        for (int l = 0; l < W; ++l) a[l] = d * v[l];
        // entries kk .. kk + n - 1 (n a constant), as many of them as the row has
        auto entries = [&](int64_t kk, auto n) {
            constexpr int AHEAD = decltype(n)::value;
            uint32_t jj[AHEAD];
            S2 h[AHEAD];
            T vj[AHEAD];
#pragma unroll
            for (int z = 0; z < AHEAD; ++z) {
                const int64_t o = min(kk + z, ke - 1);
                jj[z] = kk + z < ke ? (uint32_t)I.col[o] : i;   // i: an entry not added
                if constexpr (OPK == OP_CSR_R) h[z] = S2{((const S *)I.val)[o], (S)0};
                else h[z] = ((const S2 *)I.val)[o];
            }
#pragma unroll
            for (int z = 0; z < AHEAD; ++z) {
                vj[z] = (T)(S)0;
                if (jj[z] != i) vj[z] = ld(jj[z] * C + c);
            }
#pragma unroll
            for (int z = 0; z < AHEAD; ++z) {
                if (jj[z] == i) continue;
                if constexpr (OPK == OP_CSR_R) {
                    a = A::mac(a, h[z][0], vj[z]);
                } else {
#pragma unroll
                    for (int l = 0; l < W / 2; ++l) {
                        S ar = a[2 * l], ai = a[2 * l + 1];
                        A::cmac(ar, ai, h[z][0], h[z][1], vj[z][2 * l], vj[z][2 * l + 1]);
                        a[2 * l] = ar;
                        a[2 * l + 1] = ai;
                    }
                }
            }
        };
        int64_t kk = kb;
        for (; ke - kk > CSR_AHEAD / 2; kk += CSR_AHEAD) entries(kk, std::integral_constant<int, CSR_AHEAD>());
        if (kk < ke) entries(kk, std::integral_constant<int, CSR_AHEAD / 2>());
        out = a;
    }
    return out;
}

template <typename S, int OPK, bool WIDE>
__global__ __launch_bounds__(BLOCK) void k_step_flat(const Inst *__restrict__ tab, const uint32_t *__restrict__ bmap,
                                                     int32_t k)
{
    const uint32_t h = bmap ? bmap[blockIdx.x] : 0u;
    if (h == NO_INSTANCE) return;
    const Inst I = tab[h];
    const int32_t n = I.step0 + k;
    if (n < 0 || n >= I.K) return;
    const void *cur = (n & 1) ? I.buf1 : I.buf0;
    void *nxt = (n & 1) ? I.buf0 : I.buf1;
    const bool first = (n == 0);
    S hop = 0;
    if (OPK == OP_REAL2 || OPK == OP_REAL3) hop = Mem<S, WIDE>::lds(I.hop, 0);
    double *part = I.partial + (size_t)((n + 1) % I.pslots) * I.tiles * 4;
    const ItemRange ir = item_range(I, MODE_FLAT, blockIdx.x);
    for (uint32_t it = ir.first; it < ir.count; it += ir.stride) {
        uint32_t t, sg;
        ir.at(it, t, sg);
        Dots<S> acc;
        for (int u = 0; u < I.tpt; ++u) {
            const uint32_t e = t * (uint32_t)(BLOCK * I.tpt) + (uint32_t)(u * BLOCK) + threadIdx.x;
            if (e < I.nel) {
                typename V16<S>::T v;
                auto out = flat_apply<S, OPK, WIDE>(I, e, hop, [&](uint32_t q) { return Mem<S, WIDE>::ld(cur, q); }, v);
                if (!first) out = two_minus(out, Mem<S, WIDE>::ld_nt(nxt, e));
                Mem<S, WIDE>::st_nt(nxt, e, out);
                acc.add(out, v);
            }
        }
        block_reduce_store(acc, part + (size_t)t * 4);
    }
}

// ---------------------------------------------------------------------------
// solves of few sites: a site's vectors in the LDS of one workgroup
// ---------------------------------------------------------------------------
// The vectors of a solve are independent, so a solve of few sites runs as one
// workgroup per group of tbw of its C chunks, each with r_{n-1}, r_n of all N sites in
// the LDS (2 * N * tbw * 16 bytes), many steps per launch and one block barrier per
// step.  A thread owns EPT = 1 or 2 chunks for the whole launch: their r_n and r_{n-1},
// diagonal, neighbour indices (16 bits each) and bonds stay in registers, so a step
// reads the neighbours from the LDS and writes one chunk.  (EPT = 0: more chunks per
// thread, taken from the LDS and placed anew each step.)
// Dots are summed per wave for four steps at once and then over the waves,
// by waves 0 and 1 while the others go on; each step leaves one partial per group.
//
// What bounds it: the chain of one step (LDS reads, the stencil, the sums, the barrier).
// us per step of whole solves of 128 steps, launches included; before: one 1024-thread
// workgroup for all chunks and a whole wave sum per wave and step where they fitted, else a
// launch per step: 32 x 32 sites FP64 R = 8 5.7 -> 1.3, R = 32 7.9 -> 1.3; 10^3 spin FP32
// R = 16 10.5 -> 1.2; 12^3 spin FP64 R = 16 13.8 -> 3.1; 64 x 64 FP32 R = 4 3.5 -> 2.9.
constexpr uint32_t SMALL_BLOCK = 1024;
constexpr uint32_t SMALL_WAVES = SMALL_BLOCK / 64;
constexpr uint32_t SMALL_EPT = 2;     // most chunks per thread kept in registers

// Steps step0 + n0 .. step0 + n1 - 1 (at most to K) of each instance of the table; n0 < 0 draws
// r_0 first and starts at step 0.  A solve that does not end with the launch leaves r_{n-1},
// r_n in buf0 / buf1 (r_m in buffer m & 1) and takes them from there in the next.
template <typename S, int OPK, int EPT>
__global__ __launch_bounds__(SMALL_BLOCK) void k_solve_small(const Inst *__restrict__ tab, int32_t n0, int32_t n1)
{
    typedef typename V16<S>::T T;
    typedef Mem<S, false> G;
    typedef typename Mem<S, false>::S2 S2;
    typedef Arith<S> A;
    constexpr int W = V16<S>::W;
    constexpr bool CSR = OPK >= OP_CSR_R;
    constexpr bool D3 = (OPK == OP_REAL3 || OPK == OP_SPIN3);
    constexpr bool SPIN = (OPK == OP_SPIN2 || OPK == OP_SPIN3);
    constexpr int DIM = D3 ? 3 : 2;
    constexpr int NS = 2 * DIM;
    constexpr int NE = EPT ? EPT : 1;   // EPT = 0: any number of chunks, their values in the LDS alone
    extern __shared__ __align__(16) char kpm_lds[];
    __shared__ double red[2][4][SMALL_WAVES][4];
    const Inst I = tab[blockIdx.x];
    const uint32_t g = blockIdx.y;
    if (g >= I.tbg) return;
    const int32_t na = I.step0 + max(n0, 0), nz = min(I.step0 + n1, I.K);
    if (n0 >= 0 && na >= nz) return;
    const uint32_t C = I.C, cg0 = g * I.tbw, ng = min(I.tbw, C - cg0), ne = I.N * ng, tpb = I.tpb;
    const uint32_t tid = threadIdx.x, w = tid >> 6, nw = tpb >> 6;
    const bool alive = tid < tpb;   // the other waves only keep the barriers
    auto lb = [&](int32_t m) { return reinterpret_cast<T *>(kpm_lds) + ((m & 1) ? ne : 0u); };   // where r_m is
    S hop = 0;
    if (OPK == OP_REAL2 || OPK == OP_REAL3) hop = G::lds(I.hop, 0);
    const bool hd = CSR || I.has_diag;
    auto div_ng = [&](uint32_t e) { return ng == 1 ? e : e / ng; };
    T v[NE], pv[NE];
    S d[NE];
    uint32_t site[NE];
    uint32_t nbx[NE][EPT ? DIM : NS];   // neighbours' LDS elements, two per word where they are kept
    // bonds in registers, but for two FP64 chunks per thread (96 VGPRs of bonds alone in 3D)
    constexpr bool KEEP = SPIN && !(EPT == 2 && sizeof(S) == 8);
    S2 bnd[NE][KEEP ? NS : 1];
    uint32_t sbm[NE][SPIN && !KEEP ? DIM : 1];   // else the sites of the backward ones
    // diagonal, neighbours and bonds of chunk e into the registers of slot u
    auto place = [&](int u, uint32_t e) {
        const uint32_t i = div_ng(e), cl = e - i * ng;
        site[u] = i;
        d[u] = hd ? G::lds(I.diag, i) : (S)0;
        if constexpr (!CSR) {
            const uint32_t Lx = I.Lx, Ly = I.Ly;
            const uint32_t yq = fdiv(i, I.fLx), x = i - yq * Lx;
            uint32_t y = yq, z = 0;
            if constexpr (D3) {
                z = fdiv(yq, I.fLy);
                y = yq - z * Ly;
            }
            uint32_t nb[6];
            nb[0] = (x == 0) ? i + (Lx - 1) : i - 1;
            nb[1] = (x == Lx - 1) ? i - (Lx - 1) : i + 1;
            nb[2] = (y == 0) ? i + (Ly - 1) * Lx : i - Lx;
            nb[3] = (y == Ly - 1) ? i - (Ly - 1) * Lx : i + Lx;
            nb[4] = nb[5] = i;
            if constexpr (D3) {
                const uint32_t P = Lx * Ly, Lz = I.Lz;
                nb[4] = (z == 0) ? i + (Lz - 1) * P : i - P;
                nb[5] = (z == Lz - 1) ? i - (Lz - 1) * P : i + P;
            }
#pragma unroll
            for (int k = 0; k < DIM; ++k) {
                const uint32_t m = nb[2 * k] * ng + cl, q = nb[2 * k + 1] * ng + cl;   // below 2^16
                if constexpr (EPT) {
                    nbx[u][k] = m | (q << 16);
                } else {
                    nbx[u][2 * k] = m;
                    nbx[u][2 * k + 1] = q;
                }
            }
            if constexpr (SPIN) {
#pragma unroll
                for (int ax = 0; ax < DIM; ++ax) {
                    if constexpr (KEEP) {
                        const S2 m = G::ldc(I.bond, nb[2 * ax] * DIM + ax);
                        bnd[u][2 * ax] = S2{m[0], -m[1]};
                        bnd[u][2 * ax + 1] = G::ldc(I.bond, i * DIM + ax);
                    } else {
                        sbm[u][ax] = nb[2 * ax];
                    }
                }
            }
        }
    };
    // r_n of chunk e: drawn, or left by the last launch (with r_{n-1} in buffer na & 1 ^ 1)
    Dots<S> acc;
    auto first_value = [&](uint32_t e) {
        const uint32_t i = div_ng(e), c = cg0 + e - i * ng;
        if (n0 >= 0) return G::ld((na & 1) ? I.buf1 : I.buf0, i * C + c);
        const T x = start_chunk<S>(I, i, c);
        acc.norm_only(x);
        return x;
    };
    auto before = [&](uint32_t e) {
        const uint32_t i = div_ng(e);
        return (n0 >= 0 && na > 0) ? G::ld((na & 1) ? I.buf0 : I.buf1, i * C + cg0 + e - i * ng) : (T)(S)0;
    };
    if constexpr (EPT == 0) {
        if (alive)
            for (uint32_t e = tid; e < ne; e += tpb) {
                lb(na)[e] = first_value(e);
                lb(na + 1)[e] = before(e);
            }
    } else {
#pragma unroll
        for (int u = 0; u < EPT; ++u) {
            const uint32_t e = tid + (uint32_t)u * tpb;
            if (!alive || e >= ne) continue;
            place(u, e);
            v[u] = first_value(e);
            pv[u] = before(e);
            lb(na)[e] = v[u];
        }
    }
    const size_t pitch = (size_t)I.tiles * 4;
    double *const part = I.partial + (size_t)g * 4;
    if (n0 < 0) {   // <r_0|r_0>
        if (alive) wave_reduce_store(acc, red[0][0][w]);
        __syncthreads();
        if (tid < 2) {
            dd a{0.0, 0.0};
            for (uint32_t k = 0; k < nw; ++k) a = dd_sum(a, dd{red[0][0][k][2 * tid], red[0][0][k][2 * tid + 1]});
            part[2 * tid] = a.hi;
            part[2 * tid + 1] = a.lo;
        }
    }
    __syncthreads();   // r_n complete
    // the sums over the waves of steps nq .. (at most four, `m` of them), from red[half]: rows of
    // 16 lanes of waves 0 and 1, one row per step and sum
    auto flush = [&](int32_t nq, int32_t m, int half) {
        for (uint32_t h = w; h < 2; h += nw) {
            const uint32_t lane = tid & 63, q = 2 * h + (lane >> 5), o = ((lane >> 4) & 1u) * 2, k = lane & 15;
            dd a{0.0, 0.0};
            if ((int32_t)q < m && k < nw) a = dd{red[half][q][k][o], red[half][q][k][o + 1]};
            a = dd_sum(a, dd{row_ror<8>(a.hi), row_ror<8>(a.lo)});
            a = dd_sum(a, dd{row_ror<4>(a.hi), row_ror<4>(a.lo)});
            a = dd_sum(a, dd{row_ror<2>(a.hi), row_ror<2>(a.lo)});
            a = dd_sum(a, dd{row_ror<1>(a.hi), row_ror<1>(a.lo)});
            if ((int32_t)q < m && k == 0) {
                double *dst = part + (size_t)((nq + (int32_t)q + 1) % I.pslots) * pitch;
                dst[o] = a.hi;
                dst[o + 1] = a.lo;
            }
        }
    };
    WaveSums<Dots<S>::DD> ws;   // of the last steps, four together
    for (int32_t n = na; n < nz; ++n) {
        const int32_t j = n - na;          // steps of this launch so far
        const int q = j & 3, half = (j >> 2) & 1;
        const T *cur = lb(n);
        T *nxt = lb(n + 1);
        Dots<S> a2;
        // r_{n+1} of chunk e, whose place is in slot u, from r_n = x and r_{n-1} = y
        auto next = [&](int u, uint32_t e, T x, T y) {
            T out;
            if constexpr (!CSR) {
                T nb[NS];
#pragma unroll
                for (int k = 0; k < DIM; ++k) {
                    nb[2 * k] = cur[EPT ? nbx[u][k] & 0xffffu : nbx[u][EPT ? k : 2 * k]];
                    nb[2 * k + 1] = cur[EPT ? nbx[u][k] >> 16 : nbx[u][EPT ? k : 2 * k + 1]];
                }
                if constexpr (!SPIN) {
                    out = apply_real<S, NS>(hd, d[u], hop, x, nb);
                } else {
                    S hr[NS], hi[NS];
#pragma unroll
                    for (int k = 0; k < NS; ++k) {
                        if constexpr (KEEP) {
                            hr[k] = bnd[u][k][0];
                            hi[k] = bnd[u][k][1];
                        } else {
                            const S2 b = G::ldc(I.bond, ((k & 1) ? site[u] : sbm[u][k / 2]) * DIM + k / 2);
                            hr[k] = b[0];
                            hi[k] = (k & 1) ? b[1] : -b[1];
                        }
                    }
                    out = apply_cplx<S, NS>(hd, d[u], x, nb, hr, hi);
                }
            } else {
                const uint32_t i = site[u], cl = e - i * ng;
#pragma unroll
                for (int l = 0; l < W; ++l) out[l] = d[u] * x[l];
                for (int64_t kk = I.row_ptr[i]; kk < I.row_ptr[i + 1]; ++kk) {
                    const uint32_t jj = (uint32_t)I.col[kk];
                    if (jj == i) continue;
                    const T vj = cur[jj * ng + cl];
                    if constexpr (OPK == OP_CSR_R) {
                        out = A::mac(out, ((const S *)I.val)[kk], vj);
                    } else {
                        const S hr = ((const S *)I.val)[2 * kk], hi = ((const S *)I.val)[2 * kk + 1];
#pragma unroll
                        for (int l = 0; l < W / 2; ++l) {
                            S ar = out[2 * l], ai = out[2 * l + 1];
                            A::cmac(ar, ai, hr, hi, vj[2 * l], vj[2 * l + 1]);
                            out[2 * l] = ar;
                            out[2 * l + 1] = ai;
                        }
                    }
                }
            }
            if (n > 0) out = two_minus(out, y);
            nxt[e] = out;
            if (EPT && u == 0) a2.first(out, x);
            else a2.add(out, x);
            return out;
        };
        if (alive) {
            if constexpr (EPT == 0) {
                for (uint32_t e = tid; e < ne; e += tpb) {
                    place(0, e);
                    next(0, e, cur[e], nxt[e]);
                }
            } else {
#pragma unroll
                for (int u = 0; u < EPT; ++u) {
                    const uint32_t e = tid + (uint32_t)u * tpb;
                    if (e >= ne) continue;
                    const T out = next(u, e, v[u], pv[u]);
                    pv[u] = v[u];
                    v[u] = out;
                }
            }
            ws.add(q, a2);
            if (q == 3 || n + 1 == nz) ws.finish(q + 1, red[half][0][w], SMALL_WAVES * 4);
        }
        // step n's LDS writes before step n + 1 reads them, and its reads before they are overwritten
        __syncthreads();
        if (alive && (q == 3 || n + 1 == nz)) flush(n - q, q + 1, half);
    }
    if (nz < I.K && alive)
        for (uint32_t e = tid; e < ne; e += tpb) {
            const uint32_t i = div_ng(e), at = i * C + cg0 + e - i * ng;
            G::st((nz & 1) ? I.buf1 : I.buf0, at, lb(nz)[e]);
            if (nz > 0) G::st((nz & 1) ? I.buf0 : I.buf1, at, lb(nz + 1)[e]);
        }
}

// ---------------------------------------------------------------------------
// reduction of the per-item partials and the moments
// ---------------------------------------------------------------------------
// Block (x, h): dots index idx = step0 + 1 + klo + x of instance h, for x < nk.
__global__ __launch_bounds__(BLOCK) void k_reduce(const Inst *__restrict__ tab, int32_t klo, int32_t nk)
{
    const Inst *I = tab + blockIdx.y;
    if ((int32_t)blockIdx.x >= nk) return;
    const int32_t idx = I->step0 + 1 + klo + (int32_t)blockIdx.x;
    if (idx < 0 || idx > I->K) return;
    const double *p = I->partial + (size_t)(idx % I->pslots) * I->tiles * 4;
    dd a{0.0, 0.0}, b{0.0, 0.0};
    for (uint32_t t = threadIdx.x; t < I->tiles; t += BLOCK) {
        a = dd_sum(a, dd{p[(size_t)t * 4 + 0], p[(size_t)t * 4 + 1]});
        b = dd_sum(b, dd{p[(size_t)t * 4 + 2], p[(size_t)t * 4 + 3]});
    }
    block_reduce_store<true>(a.hi, a.lo, b.hi, b.lo, I->dots + (size_t)idx * 4);
}

// Block (x, h): dots index red_lo + x of instance h, for x < red_n.
__global__ __launch_bounds__(BLOCK) void k_reduce_ranges(const Inst *__restrict__ tab)
{
    const Inst *I = tab + blockIdx.y;
    if ((int32_t)blockIdx.x >= I->red_n) return;
    const int32_t idx = I->red_lo + (int32_t)blockIdx.x;
    if (idx < 0 || idx > I->K) return;
    const double *p = I->partial + (size_t)(idx % I->pslots) * I->tiles * 4;
    dd a{0.0, 0.0}, b{0.0, 0.0};
    for (uint32_t t = threadIdx.x; t < I->tiles; t += BLOCK) {
        a = dd_sum(a, dd{p[(size_t)t * 4 + 0], p[(size_t)t * 4 + 1]});
        b = dd_sum(b, dd{p[(size_t)t * 4 + 2], p[(size_t)t * 4 + 3]});
    }
    block_reduce_store<true>(a.hi, a.lo, b.hi, b.lo, I->dots + (size_t)idx * 4);
}

// mu_0 = S_nn[0]/norm, mu_1 = S_nm[1]/norm,
// mu_{2n} = (2 S_nn[n] - S_nn[0])/norm, mu_{2n+1} = (2 S_nm[n+1] - S_nm[1])/norm,
// formed in double-double and rounded once.
__global__ __launch_bounds__(BLOCK) void k_moments(const Inst *__restrict__ tab)
{
    const Inst *I = tab + blockIdx.y;
    const int32_t m = blockIdx.x * BLOCK + threadIdx.x;
    if (m >= I->M) return;
    const double *D = I->dots;
    dd v;
    if (m == 0) {
        v = dd{D[0], D[1]};
    } else if (m == 1) {
        v = dd{D[4 + 2], D[4 + 3]};
    } else if ((m & 1) == 0) {
        const int n = m / 2;
        v = dd_add(dd{2.0 * D[n * 4 + 0], 2.0 * D[n * 4 + 1]}, dd{-D[0], -D[1]});
    } else {
        const int n1 = m / 2 + 1;
        v = dd_add(dd{2.0 * D[n1 * 4 + 2], 2.0 * D[n1 * 4 + 3]}, dd{-D[4 + 2], -D[4 + 3]});
    }
    const dd q = dd_div_d(v, I->norm);
    I->mu[m] = q.hi + q.lo;
}

// ---------------------------------------------------------------------------
// column solves: unit start vectors e_{site[r]}, r < R, dots [R][K + 1][4]
// ---------------------------------------------------------------------------
template <typename S> __global__ __launch_bounds__(BLOCK) void k_cols_init(const Inst *__restrict__ tab)
{
    constexpr int W = V16<S>::W;
    const Inst I = tab[0];
    for (uint64_t e = (uint64_t)blockIdx.x * BLOCK + threadIdx.x; e < I.nel; e += (uint64_t)gridDim.x * BLOCK) {
        const uint32_t i = fdiv((uint32_t)e, I.fC), c = (uint32_t)e - i * I.C;
        typename V16<S>::T v;
#pragma unroll
        for (int l = 0; l < W; ++l) {
            const uint32_t k = c * W + l, r = I.cplx ? k / 2 : k;
            v[l] = (r < (uint32_t)I.R && (!I.cplx || (k & 1u) == 0) && I.colsite[r] == i) ? (S)1 : (S)0;
        }
        ((typename V16<S>::T *)I.buf0)[e] = v;
    }
}
// Dots indices lo .. lo + gridDim.x - 1 of sixteen columns (blockIdx.y): eight threads per sum
// over the items, their sums added in order.
__global__ __launch_bounds__(BLOCK) void k_cols_reduce(const Inst *__restrict__ tab, int32_t lo)
{
    const Inst *I = tab;
    const int32_t idx = lo + (int32_t)blockIdx.x;
    const uint32_t R = (uint32_t)I->R, tl = threadIdx.x >> 5, pr = threadIdx.x & 31u;
    const uint32_t col = blockIdx.y * 16 + (pr >> 1), o = (pr & 1u) * 2;
    __shared__ double red[8][32][2];
    dd a{0.0, 0.0};
    if (col < R) {
        const double *p = I->partial + (size_t)(idx % I->pslots) * I->tiles * R * 4 + col * 4 + o;
        for (uint32_t t = tl; t < I->tiles; t += 8) a = dd_sum(a, dd{p[(size_t)t * R * 4], p[(size_t)t * R * 4 + 1]});
    }
    red[tl][pr][0] = a.hi;
    red[tl][pr][1] = a.lo;
    __syncthreads();
    if (tl == 0 && col < R) {
        for (int k = 1; k < 8; ++k) a = dd_sum(a, dd{red[k][pr][0], red[k][pr][1]});
        double *d = I->dots + ((size_t)col * (I->K + 1) + idx) * 4 + o;
        d[0] = a.hi;
        d[1] = a.lo;
    }
}
// mu[column][m] as k_moments forms them, <r_0|r_0> = 1.
__global__ __launch_bounds__(BLOCK) void k_cols_moments(const Inst *__restrict__ tab)
{
    const Inst *I = tab;
    const int32_t m = blockIdx.x * BLOCK + threadIdx.x;
    if (m >= I->M) return;
    const double *D = I->dots + (size_t)blockIdx.y * (I->K + 1) * 4;
    dd v{1.0, 0.0};
    if (m == 1) {
        v = dd{D[4 + 2], D[4 + 3]};
    } else if (m > 1 && (m & 1) == 0) {
        v = dd_add(dd{2.0 * D[(m / 2) * 4 + 0], 2.0 * D[(m / 2) * 4 + 1]}, dd{-1.0, 0.0});
    } else if (m > 1) {
        v = dd_add(dd{2.0 * D[(m / 2 + 1) * 4 + 2], 2.0 * D[(m / 2 + 1) * 4 + 3]}, dd{-D[4 + 2], -D[4 + 3]});
    }
    I->mu[(size_t)blockIdx.y * I->M + m] = v.hi + v.lo;
}

}  // namespace kpm
