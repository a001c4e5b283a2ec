// Lanczos estimate of the spectral interval of H~ (FP64).
//
// The rescaling H~ = (H - b)/a of Sec. II-A needs an interval that encloses
// the spectrum; Gershgorin's discs always do but can be loose (spin hopping,
// disorder).  The Lanczos three-term process (Golub and Van Loan, Matrix
// Computations, Sec. 10.1) gives Ritz values that converge to the extreme
// eigenvalues from inside; padded by their residual bounds and a relative
// margin, and clipped to Gershgorin, they give a tighter interval.
//
// One start vector in the solve layout with R = 1: one 16-byte chunk per site
// holding (re, im) for a complex operator or (value, 0) for a real one.
//   v_0 = xi / ||xi||;  for j = 0, 1, ...:
//     u = H~ v_j,  alpha_j = Re <v_j|u>,
//     w = (u - alpha_j v_j) - beta_{j-1} v_{j-1}   (last term absent for j = 0),
//     beta_j = ||w||,  v_{j+1} = w / beta_j        (0 if beta_j = 0)
// Two launches per step: the vectors are kept as w_j and divided by their norm where
// they are read, and each kernel sums the partial dots of the one before it itself, every
// block all of them (at most LZ_BLOCKS) in the same order.  A step is a handful of
// launches' latency: with the sums and the division in launches of their own it took
// 27 us at 64^3 sites (five launches), the tridiagonal solve on one thread 870 us; the
// whole interval with k = 100 went from 3.6 to 1.8 ms (20^3: 32 to 13 us per step).
// The scalars stay on the device, in the instance's dots array, as
// double-double sums (each used rounded to a double):
//   index 0       <xi|xi>
//   index 2j + 1  (0, Re<u|v_j>)         alpha_j = the second sum
//   index 2j + 2  (||w||^2, 0)           beta_j = sqrt(the first sum)
#pragma once

namespace kpm {

constexpr int LZ_KMAX = 512;       // Lanczos steps per call (LDS of the tridiagonal solve)
constexpr double LZ_BREAKDOWN = 1e-12;

constexpr uint32_t LZ_BLOCKS = 2048;   // most blocks (= partial dots) per launch

// Chunks [base, end) of the block's XCD (block b runs on XCD b mod 8) and its first one and
// stride: neighbouring rows and planes of a large lattice meet in one L2.
struct LzRange {
    uint32_t first, stride, end;
};
__device__ __forceinline__ LzRange lz_range(uint32_t nel)
{
    if (gridDim.x % 8) return LzRange{blockIdx.x * BLOCK + threadIdx.x, gridDim.x * BLOCK, nel};
    const uint32_t x = blockIdx.x & 7u, base = (uint32_t)(((uint64_t)nel * x) >> 3);
    return LzRange{base + (blockIdx.x >> 3) * BLOCK + threadIdx.x, (gridDim.x >> 3) * BLOCK,
                   (uint32_t)(((uint64_t)nel * (x + 1)) >> 3)};
}

// The sum of the blocks' partials `part` ([blocks][2]), the same in every thread.
__device__ __forceinline__ double lz_total(const double *part, uint32_t blocks, double &lo)
{
    __shared__ double sum[4];
    double a = 0.0, b = 0.0;
    for (uint32_t t = threadIdx.x; t < blocks; t += BLOCK) {
        const dd s = dd_sum(dd{a, b}, dd{part[2 * t], part[2 * t + 1]});
        a = s.hi;
        b = s.lo;
    }
    block_reduce_store<true>(a, b, 0.0, 0.0, sum);
    const dd s = dd_fast_two_sum(sum[0], sum[1]);
    lo = s.lo;
    return s.hi;
}
// y / ||w||, or 0
__device__ __forceinline__ V16<double>::T lz_unit(V16<double>::T y, double nrm)
{
#pragma unroll
    for (int l = 0; l < 2; ++l) y[l] = nrm > 0.0 ? y[l] / nrm : 0.0;
    return y;
}

// The first sum at dots index idx, a pair, rounded to a double.
__device__ __forceinline__ double lz_norm2(const Inst &I, int32_t idx)
{
    return I.dots[(size_t)idx * 4] + I.dots[(size_t)idx * 4 + 1];
}

// u = H~ v_j, v_j = w / ||w||, and the partials of Re<u|v_j> in pout.  ||w||^2 is the sum of
// `pin` (j > 0; block 0 leaves it at dots index 2j) or dots index 0.
template <int OPK, bool WIDE>
__global__ __launch_bounds__(BLOCK) void k_lz_matvec(const Inst *__restrict__ tab, const void *w, void *u, int32_t j,
                                                     const double *pin, double *pout)
{
    typedef Mem<double, WIDE> G;
    typedef V16<double>::T T;
    const Inst I = tab[0];
    double n2 = lz_norm2(I, 0), lo = 0.0;
    if (j > 0) {
        n2 = lz_total(pin, gridDim.x, lo);
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            I.dots[(size_t)(2 * j) * 4 + 0] = n2;
            I.dots[(size_t)(2 * j) * 4 + 1] = lo;
        }
    }
    const double nrm = sqrt(n2);
    double hop = 0.0;
    if (OPK == OP_REAL2 || OPK == OP_REAL3) hop = G::lds(I.hop, 0);
    Dots<double> acc;
    const LzRange r = lz_range(I.nel);
    for (uint32_t e = r.first; e < r.end; e += r.stride) {
        T v;
        const T out = flat_apply<double, OPK, WIDE>(I, e, hop, [&](uint32_t q) { return lz_unit(G::ld(w, q), nrm); }, v);
        G::st(u, e, out);
        acc.cross_only(out, v);
    }
    __shared__ double sum[4];
    block_reduce_store(acc, sum);
    if (threadIdx.x < 2) pout[2 * blockIdx.x + threadIdx.x] = sum[2 + threadIdx.x];
}

// w_{j+1} = (u - alpha_j v_j) - beta_{j-1} v_{j-1}, written over w_{j-1} (wp), and the partials
// of its squared norm in pout; alpha_j is the sum of pin (block 0 leaves it at dots index
// 2j + 1).
template <bool WIDE>
__global__ __launch_bounds__(BLOCK) void k_lz_update(const Inst *__restrict__ tab, const void *u, const void *w,
                                                     void *wp, int32_t j, const double *pin, double *pout)
{
    typedef Mem<double, WIDE> G;
    typedef V16<double>::T T;
    const Inst I = tab[0];
    double lo;
    const double al = lz_total(pin, gridDim.x, lo);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        I.dots[(size_t)(2 * j + 1) * 4 + 2] = al;
        I.dots[(size_t)(2 * j + 1) * 4 + 3] = lo;
    }
    const double nrm = sqrt(lz_norm2(I, 2 * j));                      // of w_j: beta_{j-1} for j > 0
    const double nrp = j > 0 ? sqrt(lz_norm2(I, 2 * j - 2)) : 0.0;    // of w_{j-1}
    Dots<double> acc;
    const LzRange r = lz_range(I.nel);
    for (uint32_t e = r.first; e < r.end; e += r.stride) {
        const T uu = G::ld(u, e), vv = lz_unit(G::ld(w, e), nrm);
        T x;
#pragma unroll
        for (int l = 0; l < 2; ++l) x[l] = uu[l] - al * vv[l];
        if (j > 0) {
            const T pp = lz_unit(G::ld(wp, e), nrp);
#pragma unroll
            for (int l = 0; l < 2; ++l) x[l] = x[l] - nrm * pp[l];
        }
        G::st(wp, e, x);
        acc.norm_only(x);
    }
    __shared__ double sum[4];
    block_reduce_store(acc, sum);
    if (threadIdx.x < 2) pout[2 * blockIdx.x + threadIdx.x] = sum[threadIdx.x];
}

// ---------------------------------------------------------------------------
// the k x k tridiagonal matrix: extreme eigenpairs and the padded interval
// ---------------------------------------------------------------------------
// Number of eigenvalues of T below x: negative pivots of the LDL^T
// factorisation of T - x I (Sturm count).
__device__ inline int lz_count_below(const double *al, const double *b2, int m, double x, double pivmin)
{
    int c = 0;
    double q = al[0] - x;
    if (fabs(q) < pivmin) q = -pivmin;
    if (q < 0.0) ++c;
    for (int i = 1; i < m; ++i) {
        q = (al[i] - x) - b2[i - 1] / q;
        if (fabs(q) < pivmin) q = -pivmin;
        if (q < 0.0) ++c;
    }
    return c;
}

// Eigenvalue number `which` (0 = smallest) of T: the adjacent doubles between which the
// count passes it, found by LZ_SECTIONS lanes counting at as many points of the interval
// at once (seven rounds for 49 bits), the last few by bisection.  All lanes of the group
// (`lane` < LZ_SECTIONS, one group of waves per eigenvalue) call it; `below`: LDS of the group.
constexpr int LZ_SECTIONS = 128;
__device__ inline double lz_section(const double *al, const double *b2, int m, int which, double lo, double hi,
                                    double pivmin, int lane, int *below)
{
    for (int round = 0; round < 7; ++round) {
        const double h = (hi - lo) / (double)(LZ_SECTIONS + 1);
        const double x = fmin(fmax(lo + h * (double)(lane + 1), lo), hi);
        below[lane] = lz_count_below(al, b2, m, x, pivmin) >= which + 1 ? 1 : 0;
        __syncthreads();
        int first = LZ_SECTIONS;   // the first point at or above the eigenvalue
        for (int t = LZ_SECTIONS - 1; t >= 0; --t)
            if (below[t]) first = t;
        const double nlo = first > 0 ? fmin(fmax(lo + h * (double)first, lo), hi) : lo;
        const double nhi = first < LZ_SECTIONS ? fmin(fmax(lo + h * (double)(first + 1), lo), hi) : hi;
        lo = nlo;
        hi = nhi;
        __syncthreads();
    }
    for (int it = 0; it < 256; ++it) {
        const double mid = 0.5 * (lo + hi);
        if (mid <= lo || mid >= hi) break;   // adjacent doubles
        if (lz_count_below(al, b2, m, mid, pivmin) >= which + 1) hi = mid;
        else lo = mid;
    }
    return 0.5 * (lo + hi);
}

// |last component| of the unit eigenvector of T for the eigenvalue theta:
// two steps of inverse iteration, each a solve with T - theta I factored by
// Gaussian elimination with partial pivoting (tridiagonal form, one extra
// superdiagonal from the row interchanges).  Work arrays of length m in LDS.
__device__ inline double lz_last_component(const double *al, const double *be, int m, double theta, double tnorm,
                                           double *d, double *dl, double *du, double *du2, unsigned char *piv,
                                           double *x)
{
    if (m == 1) return 1.0;
    for (int i = 0; i < m; ++i) {
        d[i] = al[i] - theta;
        du2[i] = 0.0;
        x[i] = 1.0;
    }
    for (int i = 0; i + 1 < m; ++i) {
        dl[i] = be[i];
        du[i] = be[i];
    }
    for (int i = 0; i + 1 < m; ++i) {
        if (fabs(d[i]) >= fabs(dl[i])) {
            piv[i] = 0;
            if (d[i] != 0.0) {
                const double f = dl[i] / d[i];
                dl[i] = f;
                d[i + 1] = d[i + 1] - f * du[i];
            } else {
                dl[i] = 0.0;
            }
        } else {
            piv[i] = 1;
            const double f = d[i] / dl[i];
            d[i] = dl[i];
            dl[i] = f;
            const double tmp = du[i];
            du[i] = d[i + 1];
            d[i + 1] = tmp - f * d[i + 1];
            if (i + 2 < m) {
                du2[i] = du[i + 1];
                du[i + 1] = -f * du[i + 1];
            }
        }
    }
    const double tiny = 2.220446049250313e-16 * (tnorm > 0.0 ? tnorm : 1.0);
    for (int i = 0; i < m; ++i)
        if (d[i] == 0.0) d[i] = tiny;
    for (int pass = 0; pass < 2; ++pass) {
        for (int i = 0; i + 1 < m; ++i) {
            if (!piv[i]) {
                x[i + 1] = x[i + 1] - dl[i] * x[i];
            } else {
                const double tmp = x[i];
                x[i] = x[i + 1];
                x[i + 1] = tmp - dl[i] * x[i];
            }
        }
        x[m - 1] = x[m - 1] / d[m - 1];
        x[m - 2] = (x[m - 2] - du[m - 2] * x[m - 1]) / d[m - 2];
        for (int i = m - 3; i >= 0; --i) x[i] = ((x[i] - du[i] * x[i + 1]) - du2[i] * x[i + 2]) / d[i];
        double s = 0.0;
        for (int i = 0; i < m; ++i) s = fmax(s, fabs(x[i]));
        double n2 = 0.0;
        for (int i = 0; i < m; ++i) {
            x[i] = x[i] / s;
            n2 = n2 + x[i] * x[i];
        }
        const double n = sqrt(n2);
        for (int i = 0; i < m; ++i) x[i] = x[i] / n;
    }
    return fabs(x[m - 1]);
}

// out[0..1]  E_lo, E_hi of H (padded, mapped by E = a lambda + b, clipped)
// out[2..3]  theta_min, theta_max (Ritz values of H~)
// out[4..5]  r_min, r_max (residual bounds, units of H~)
// out[6]     m, the number of Lanczos steps used (a breakdown stops early)
// out[8 + j], out[8 + k + j]  alpha_j, beta_j for j < k
// The lower and the upper half of the block work on the two ends of the spectrum.
__global__ __launch_bounds__(2 * LZ_SECTIONS) void k_lz_tridiag(const Inst *__restrict__ tab, int32_t k, double pad,
                                                                double a, double b, double clamp_lo, double clamp_hi,
                                                                const double *pin, uint32_t blocks, double *out)
{
    __shared__ double al[LZ_KMAX], be[LZ_KMAX], b2[LZ_KMAX];
    __shared__ double d[2][LZ_KMAX], dl[2][LZ_KMAX], du[2][LZ_KMAX], du2[2][LZ_KMAX], x[2][LZ_KMAX];
    __shared__ unsigned char piv[2][LZ_KMAX];
    __shared__ int below[2][LZ_SECTIONS];
    __shared__ double th[2], res[2];
    const Inst I = tab[0];
    double lo;
    const double last = lz_total(pin, blocks, lo);   // ||w_k||^2
    for (int j = threadIdx.x; j < k; j += blockDim.x) {
        al[j] = I.dots[(size_t)(2 * j + 1) * 4 + 2];
        be[j] = sqrt(j + 1 < k ? I.dots[(size_t)(2 * j + 2) * 4 + 0] : last);
        b2[j] = be[j] * be[j];
        out[8 + j] = al[j];
        out[8 + k + j] = be[j];
    }
    __syncthreads();
    const int side = threadIdx.x / LZ_SECTIONS, lane = threadIdx.x % LZ_SECTIONS;
    int m = k;
    bool stop = false;
    double scale = 0.0;
    for (int j = 0; j < k; ++j) {
        scale = fmax(scale, fmax(fabs(al[j]), be[j]));
        if (be[j] <= LZ_BREAKDOWN * scale) {
            m = j + 1;
            stop = true;
            break;
        }
    }
    // Gershgorin interval of T brackets every eigenvalue
    double glo = al[0], ghi = al[0], tnorm = 0.0;
    for (int i = 0; i < m; ++i) {
        const double r = (i > 0 ? be[i - 1] : 0.0) + (i + 1 < m ? be[i] : 0.0);
        glo = fmin(glo, al[i] - r);
        ghi = fmax(ghi, al[i] + r);
        tnorm = fmax(tnorm, fabs(al[i]) + r);
    }
    const double pivmin = 1e-290 * fmax(1.0, tnorm * tnorm);
    const double margin = 4.440892098500626e-16 * (tnorm > 0.0 ? tnorm : 1.0) + pivmin;
    glo -= margin;
    ghi += margin;
    const double theta = lz_section(al, b2, m, side ? m - 1 : 0, glo, ghi, pivmin, lane, below[side]);
    const double blast = stop ? 0.0 : be[m - 1];
    if (lane == 0) {
        th[side] = theta;
        res[side] = blast > 0.0 ? blast * lz_last_component(al, be, m, theta, tnorm, d[side], dl[side], du[side],
                                                            du2[side], piv[side], x[side])
                                : 0.0;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    const double width = th[1] - th[0];
    const double e_lo = th[0] - fmax(res[0], pad * width);
    const double e_hi = th[1] + fmax(res[1], pad * width);
    out[0] = fmax(a * e_lo + b, clamp_lo);
    out[1] = fmin(a * e_hi + b, clamp_hi);
    out[2] = th[0];
    out[3] = th[1];
    out[4] = res[0];
    out[5] = res[1];
    out[6] = (double)m;
    out[7] = 0.0;
}

}  // namespace kpm
