// trbt_tridiag.hip -- the lowest nev eigenpairs of a real symmetric
// tridiagonal matrix T = diag(d) + subdiag(e) on AMD Instinct MI355X
// (gfx950): the tridiagonal step of the two-stage solver (Eq. 2stage_solve),
// between the bulge chasing and the back-transformation.  Only the wanted
// eigenvectors are computed.
//
// Method (the classical pair; the paper's solver is divide and conquer, which
// reaches the same eigenpairs):
//   * eigenvalue i by multisection on the Sturm count: the number of sign changes
//     in the leading principal minors of T - x I equals the number of
//     eigenvalues below x; the interval starts from the Gershgorin bounds and is
//     cut into 17 (33, 65) by as many lanes less one per eigenvalue until it is no
//     wider than a few ulps of its end points;
//   * eigenvector i by inverse iteration with that eigenvalue, one thread per
//     vector: Gaussian elimination with partial pivoting, a half step from a
//     fixed pseudo-random vector (the back substitution alone, as in EISPACK's
//     tinvit) and a full step; a pivot below a floor is raised to it, in L and U
//     alike (so that rows equal to within rounding weigh the same in a cluster's
//     vectors).
// Accuracy: residual ||T x - lambda x|| ~ eps ||T||; the angle between
// computed eigenvectors of eigenvalues a gap apart ~ eps ||T|| / gap.
// Eigenvalues closer than 1e-6 ||T|| to their predecessor form a cluster:
// its vectors (each an inverse iterate from a different start, so together
// spanning the cluster's invariant subspace) are orthonormalised by modified
// Gram-Schmidt, one workgroup per cluster, so (near-)degenerate eigenvalues
// get an orthonormal basis of their subspace.

#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "trbt.h"
#include "trbt_device.h"
#include "trbt_lanes.h"

namespace {

constexpr int TD_THREADS = 64;
// eigenvalues closer than this times ||T|| to their predecessor are one
// cluster, whose vectors are orthonormalised together afterwards; outside
// clusters the angle error of inverse iteration is below about eps / TD_CLUSTER
constexpr double TD_CLUSTER = 1e-6;

// e2[k] = (s e[k])^2, re[k] = 1 / (s e[k]) (0 for 0) with s the power of
// two that brings ||T|| into [1/2, 1) (as far as s is a number); bounds[0..1] = Gershgorin
// interval of the scaled T, bounds[2] = norm estimate (max row sum) of T, bounds[3] = s.
// One workgroup.
__global__ __launch_bounds__(256) void k_td_prep(int64_t n, const double* __restrict__ d,
                                                 const double* __restrict__ e,
                                                 double* __restrict__ e2,
                                                 double* __restrict__ re,
                                                 double* __restrict__ bounds)
{
    __shared__ double lo_s[256], hi_s[256], nm_s[256];
    double lo = INFINITY, hi = -INFINITY, nm = 0.0;
    for (int64_t k = threadIdx.x; k < n; k += 256) {
        const double a = k > 0 ? fabs(e[k - 1]) : 0.0, b = k + 1 < n ? fabs(e[k]) : 0.0;
        lo = fmin(lo, d[k] - a - b);
        hi = fmax(hi, d[k] + a + b);
        nm = fmax(nm, fabs(d[k]) + a + b);
    }
    lo_s[threadIdx.x] = lo;
    hi_s[threadIdx.x] = hi;
    nm_s[threadIdx.x] = nm;
    for (int h = 128; h > 0; h /= 2) {
        __syncthreads();
        if (threadIdx.x < h) {
            const int o = threadIdx.x + h;
            lo_s[threadIdx.x] = fmin(lo_s[threadIdx.x], lo_s[o]);
            hi_s[threadIdx.x] = fmax(hi_s[threadIdx.x], hi_s[o]);
            nm_s[threadIdx.x] = fmax(nm_s[threadIdx.x], nm_s[o]);
        }
    }
    __syncthreads();
    lo = lo_s[0];
    hi = hi_s[0];
    nm = nm_s[0] > 0.0 ? nm_s[0] : 1.0;
    int ex;
    (void)frexp(nm, &ex);
    const double s = ldexp(1.0, ex < -1022 ? 1022 : -ex);
    if (threadIdx.x == 0) {
        const double eps = 2.220446049250313e-16;
        lo *= s;
        hi *= s;
        const double pad = 2.0 * eps * fmax(fabs(lo), fabs(hi)) + 2.0 * eps * n * (nm_s[0] * s) + 1e-300;
        bounds[0] = lo - pad;
        bounds[1] = hi + pad;
        bounds[2] = nm;
        bounds[3] = s;
    }
    for (int64_t k = threadIdx.x; k + 1 < n; k += 256) {
        const double es = e[k] * s;
        e2[k] = es * es;
        re[k] = es != 0.0 ? 1.0 / es : 0.0;
    }
}

// The number of eigenvalues of the scaled T below x: sign changes in the sequence
// of its leading principal minors p_k = (d_k - x) p_{k-1} - e_{k-1}^2 p_{k-2}
// (the pivots of LDL^T are their ratios; each computed p_k is that of a T with
// off-diagonals changed by a few ulps).  One FMA is all that a step waits
// for, where the pivots need a division each (350 clocks a step, 16.7 ms for the
// 4096 lowest at n = 8192; now 57 and 2.7, most of them waits for the scalar
// loads of d and e^2).
//
// The last two minors are brought back to [1/2, 1) every TD_CHUNK steps; none grows by
// more than 3 a step.  They may vanish, though: a zero minor before a zero
// off-diagonal (x an eigenvalue of a block that is coupled to nothing) leaves only
// zeros, and many small factors leave the range.  A count in which a chunk ends with
// both below TD_SMALL, so that rounding at the end of the range might matter, is
// done again by the pivots (a branch inside the loop, to do the one chunk again,
// takes 3.3 ms for the 2.7 at n = 8192, where no chunk is: the loads made ahead are
// waited for at it).  Otherwise a minor that is exactly zero counts once whichever
// sign it gets, its neighbours' signs being opposite.
constexpr int TD_CHUNK = 8;
constexpr int TD_EXMIN = -664;   // of TD_SMALL
constexpr double TD_SMALL = 1e-200, TD_PIVMIN = 1e-290;

// The same count by the pivots t_k = d_k - x - e_{k-1}^2 / t_{k-1}, a zero one counted as
// negative
__device__ inline int td_count_pivots(int n, const double* __restrict__ d,
                                      const double* __restrict__ e2, double s, double x)
{
    int cnt = 0;
    double t = INFINITY;
#pragma unroll 1
    for (int k = 0; k < n; ++k) {
        t = fma(d[k], s, -x) - (k > 0 ? e2[k - 1] / t : 0.0);
        if (fabs(t) < TD_PIVMIN) t = -TD_PIVMIN;
        cnt += t < 0.0;
    }
    return cnt;
}

__device__ inline int td_count(int n, const double* __restrict__ d,
                               const double* __restrict__ e2, double s, double x)
{
    double q = 1.0, p = fma(d[0], s, -x);   // p_{k-1}, p_k
    unsigned bits = (unsigned)(__builtin_bit_cast(uint64_t, p) >> 63);   // signs, newest lowest
    int cnt = (int)bits;
    auto step = [&](double dk, double ek) {
        const double r = fma(fma(dk, s, -x), p, -(ek * q));
        q = p;
        p = r;
        bits = __builtin_amdgcn_alignbit(bits, (unsigned)(__builtin_bit_cast(uint64_t, r) >> 32), 31);
    };
    // whole chunks, each loaded (scalar loads: the same for every lane) while the
    // one before is worked on
    struct Chunk {
        double d[TD_CHUNK], e[TD_CHUNK];
    };
    auto load = [&](Chunk& c, int k) {
#pragma unroll
        for (int i = 0; i < TD_CHUNK; ++i) {
            c.d[i] = d[k + i];
            c.e[i] = e2[k - 1 + i];
        }
    };
    int least = 0;   // exponent of the largest minor at the chunks' ends, the smallest of them
    auto work = [&](const Chunk& c) {
#pragma unroll
        for (int i = 0; i < TD_CHUNK; ++i) step(c.d[i], c.e[i]);
        const int ex = __builtin_amdgcn_frexp_exp(fmax(fabs(p), fabs(q)));
        cnt += __builtin_popcount((bits ^ (bits >> 1)) & ((1u << TD_CHUNK) - 1));
        least = ex < least ? ex : least;   // (two zeros stay zeros to the end)
        p = __builtin_amdgcn_ldexp(p, -ex);
        q = __builtin_amdgcn_ldexp(q, -ex);
    };
    const int m = (n - 1) / TD_CHUNK;
    Chunk a, b;
    if (m > 0) load(a, 1);
    int j = 0;
    for (; j + 2 < m; j += 2) {
        load(b, 1 + (j + 1) * TD_CHUNK);
        __builtin_amdgcn_sched_barrier(0);   // (or the loads would sink to their use)
        work(a);
        load(a, 1 + (j + 2) * TD_CHUNK);
        __builtin_amdgcn_sched_barrier(0);
        work(b);
    }
    if (j < m) work(a);
    if (j + 1 < m) {
        load(b, 1 + (j + 1) * TD_CHUNK);
        work(b);
    }
    for (int k = 1 + m * TD_CHUNK; k < n; ++k) {
        step(d[k], e2[k - 1]);
        cnt += (bits ^ (bits >> 1)) & 1;
    }
    if (least < TD_EXMIN || fmax(fabs(p), fabs(q)) < TD_SMALL)
        return td_count_pivots(n, d, e2, s, x);
    return cnt;
}

// eigenvalue i (0-based, ascending) of the scaled T by multisection: MS consecutive lanes share
// one eigenvalue and evaluate the Sturm count at MS interior points of its
// interval, x_k = lo + (hi - lo)(k+1)/(MS+1); the new interval is
// [x_{k*-1}, x_{k*}] for the first point k* with count > i, read from the
// group's bits of a wave ballot (every lane of the group computes the same
// end points from the same formula).
template <int MS>
__global__ __launch_bounds__(TD_THREADS) void k_td_bisect(int64_t n, int64_t nev,
                                                          const double* __restrict__ d,
                                                          const double* __restrict__ e2,
                                                          const double* __restrict__ bounds,
                                                          double* __restrict__ w)
{
    const int64_t gid = (int64_t)blockIdx.x * TD_THREADS + threadIdx.x;
    const int64_t i = gid / MS;
    const int k = (int)(gid % MS);
    const int gbit = (threadIdx.x & 63) & ~(MS - 1);   // the group's first lane in the wave
    if (i >= nev) return;   // whole groups leave together
    double lo = bounds[0], hi = bounds[1];
    const double s = bounds[3];
    const double eps = 2.220446049250313e-16;
    // invariant: count(lo) <= i < count(hi)
    for (int it = 0; it < 100; ++it) {
        if (hi - lo <= 4.0 * eps * fmax(fabs(lo), fabs(hi)) + 1e-290) break;
        const double step = (hi - lo) / (MS + 1);
        const double x = lo + step * (k + 1);
        const bool above = td_count((int)n, d, e2, s, x) > i;
        const uint64_t grp = (__ballot(above) >> gbit) & (~0ull >> (64 - MS));
        double nlo = lo, nhi = hi;
        if (grp) {
            const int ks = __builtin_ctzll(grp);
            nhi = lo + step * (ks + 1);
            if (ks > 0) nlo = lo + step * ks;
        } else {
            nlo = lo + step * MS;
        }
        if (nlo == lo && nhi == hi) break;   // no representable progress
        lo = nlo;
        hi = nhi;
    }
    if (k == 0) w[i] = 0.5 * (lo + hi) / s;
}

// a fixed pseudo-random start in [-1, 1): a 32-bit integer hash (two rounds of
// multiply and xorshift, Wellons' "lowbias32") of (vector, row)
__device__ inline double td_start(uint32_t i, uint32_t r)
{
    uint32_t z = i * 0x9E3779B9u + r * 0x85EBCA77u + 0x7F4A7C15u;
    z ^= z >> 16;
    z *= 0x7FEB352Du;
    z ^= z >> 15;
    z *= 0x846CA68Bu;
    z ^= z >> 16;
    return (double)(int)z * (1.0 / 2147483648.0);
}

// 1 / x from the hardware estimate by two Newton steps (x far from the ends of
// the range)
__device__ inline double td_recip(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
}

// The shift of vector i's inverse iteration (of the scaled T), and the floor of
// its pivots.  Pivots below the floor are raised to it, a change of T by no more:
// eps ||T||, what rounding may change anyway.  But an eigenvalue that is small beside
// its distance to its neighbours (they are found to full relative accuracy) keeps
// what the rounding of its own rows leaves it: entries over many orders of
// magnitude (1e-40 .. 1) otherwise give it pivots of other eigenvalues raised to the
// same floor, and vectors that depend on each other (a third of such matrices had
// residuals up to ||T||).  Eigenvalues equal to rounding get a shift that is not one
// of them, so that all of their vectors come up alike: repeated diagonals -2 .. 2
// coupled by 1e-12 had wrong vectors in 44 of 300 matrices without it, 3 with it.
struct TdShift {
    double lam, floor;
};

__device__ inline TdShift td_shift(int64_t i, int64_t nev, const double* __restrict__ w,
                                   const double* __restrict__ bounds)
{
    const double eps = 2.220446049250313e-16, s = bounds[3], full = eps * (bounds[2] * s);
    const double gap = fmin(i > 0 ? w[i] - w[i - 1] : INFINITY,
                            i + 1 < nev ? w[i + 1] - w[i] : INFINITY);
    const double lam = w[i] * s;
    if (gap > 1e-3 * fabs(w[i])) return {lam, fmax(eps * fabs(lam), 1e-100)};
    return {gap * s < 64.0 * full ? lam + 2.0 * full : lam, full};
}

// Eigenvector i by inverse iteration on the scaled T - lambda I, one thread per
// vector, everything row-major across the vectors (a wave reads and writes
// consecutive addresses).  The LU factorisation with partial pivoting keeps one
// number per row and a bit:
//   row k not swapped with k+1 (bit 0): V = 1 / pivot; the multiplier is e_k V,
//     U's row (pivot, b_k, 0);
//   swapped (bit 1): V = the multiplier; U's row (e_k, d_{k+1} - lambda, e_{k+1});
// b_k = e_k, or -V_{k-1} e_k after a swap.  Everything else comes from d and e,
// the same for all vectors.  Rows are swapped only for a pivot e_k that needs no
// raising, so that U's pivot is e_k itself.  Should small pivots (and a small
// floor) overflow, it is done again with the floor eps ||T||.
//
// Passes over the rows: the factorisation; a first half step U x = y with a
// fixed pseudo-random y (a start b = L y, as good as a random b, and the
// forward substitution is saved); a full step from it; the norm and the sign
// are taken along with the second backward substitution and applied as the
// vectors are transposed into Z.  A pass runs TD_CH rows at a time with the next
// rows' loads already issued: nev threads are few (64 waves at nev = 4096), so
// the issue of one wave per SIMD and its waits bound it.  n = 8192, nev = 4096:
// 4.2 ms (19.1 with five numbers per row, a division in every substitution and
// separate norm passes).
constexpr int TD_CH = 16;

__global__ __launch_bounds__(TD_THREADS) void k_td_invit(int64_t n64, int64_t nev,
                                                         const double* __restrict__ d,
                                                         const double* __restrict__ e,
                                                         const double* __restrict__ re,
                                                         const double* __restrict__ bounds,
                                                         const double* __restrict__ w,
                                                         double* __restrict__ X,
                                                         double* __restrict__ V,
                                                         uint32_t* __restrict__ B,
                                                         double* __restrict__ sc)
{
    const int64_t i = (int64_t)blockIdx.x * TD_THREADS + threadIdx.x;
    if (i >= nev) return;
    const int n = (int)n64;
    const double s = bounds[3], eps = 2.220446049250313e-16, full = eps * (bounds[2] * s);
    const TdShift shift = td_shift(i, nev, w, bounds);
    const double lam = shift.lam;
    X += i;
    V += i;
    B += i;
    auto ev = [&](int k) { return k >= 0 && k + 1 < n ? e[k] * s : 0.0; };
    auto dv = [&](int k) { return k < n ? fma(d[k], s, -lam) : 0.0; };

    // ---- factorisation.  The current row (to become U's row k, or to be swapped
    // with row k+1) has a in column k and b in column k+1; tiny is its pivot's floor.
    auto factor = [&](double base) {
        double a = dv(0), b = ev(0), tiny = base;
        uint32_t bits = 0;
        auto row = [&](int k, double sub, double dn, double en) {
            const bool swap = fabs(sub) >= tiny && fabs(a) < fabs(sub);
            double x = swap ? sub : a;
            if (fabs(x) < tiny) x = copysign(tiny, x);
            const double r = td_recip(x);
            const double l = (swap ? a : sub) * r;
            V[(int64_t)k * nev] = swap ? l : r;
            bits |= (uint32_t)swap << (k & 31);
            tiny = fma(eps, fabs(swap ? b : l * b), base);
            a = swap ? fma(-l, dn, b) : fma(-l, b, dn);
            b = swap ? -l * en : en;
        };
        int k = 0;
        for (; k + TD_CH + 1 < n; k += TD_CH) {
            double dc[TD_CH], ec[TD_CH + 1];
#pragma unroll
            for (int t = 0; t < TD_CH; ++t) {
                dc[t] = d[k + 1 + t];
                ec[t] = e[k + t];
            }
            ec[TD_CH] = e[k + TD_CH];
#pragma unroll
            for (int t = 0; t < TD_CH; ++t) row(k + t, ec[t] * s, fma(dc[t], s, -lam), ec[t + 1] * s);
            if (k & 16) {
                B[(int64_t)(k >> 5) * nev] = bits;
                bits = 0;
            }
        }
        for (; k < n; ++k) {
            row(k, ev(k), dv(k + 1), ev(k + 1));
            if ((k & 31) == 31 || k + 1 == n) {
                B[(int64_t)(k >> 5) * nev] = bits;
                bits = 0;
            }
        }
    };

    const int nc = (n + TD_CH - 1) / TD_CH;   // chunks of TD_CH rows; a word of B holds two
    struct Chunk {
        double v[TD_CH + 1];   // V of the rows and (backward) of the row before
        double y[TD_CH];
        uint32_t bits, prev;
    };
    auto load = [&](Chunk& c, int q, bool before, bool withy) {
        q = q < 0 ? 0 : q >= nc ? nc - 1 : q;
        const int k0 = q * TD_CH;
#pragma unroll
        for (int t = 0; t < TD_CH; ++t) {
            const int64_t k = k0 + t < n ? k0 + t : n - 1;
            c.v[t + 1] = V[k * nev];
            if (withy) c.y[t] = X[k * nev];
        }
        c.bits = B[(int64_t)(k0 >> 5) * nev];
        if (before) {
            const int64_t k = k0 > 0 ? k0 - 1 : 0;
            c.v[0] = V[k * nev];
            c.prev = B[(k >> 5) * nev];
        }
    };

    // ---- backward substitution U x = y, in place; y random in the first
    double ss = 0.0, big = 0.0, sg = 1.0, x1 = 0.0, x2 = 0.0;
    auto back = [&](const Chunk& c, int q, auto first, auto edge) {
        constexpr bool FIRST = decltype(first)::value, EDGE = decltype(edge)::value;
        const int k0 = q * TD_CH;
        const uint32_t cb = c.bits >> (k0 & 31);                 // bit t: row k0 + t
        const uint32_t pb = EDGE && k0 == 0 ? 0 : c.prev >> ((k0 - 1) & 31) & 1;
        double dc[TD_CH], ec[TD_CH + 1], rc[TD_CH];
#pragma unroll
        for (int t = 0; t < TD_CH; ++t) {   // rows' d_{k+1}, e_k, 1/e_k
            const int k = k0 + t;
            dc[t] = EDGE ? (k + 1 < n ? d[k + 1] : 0.0) : d[k + 1];
            ec[t] = EDGE ? (k + 1 < n ? e[k] : 0.0) : e[k];
            rc[t] = EDGE ? (k + 1 < n ? re[k] : 0.0) : re[k];
        }
        ec[TD_CH] = EDGE ? (k0 + TD_CH + 1 < n ? e[k0 + TD_CH] : 0.0) : e[k0 + TD_CH];
#pragma unroll
        for (int t = TD_CH - 1; t >= 0; --t) {
            const int k = k0 + t;
            if (EDGE && k >= n) continue;
            const bool sw = cb >> t & 1, swp = t > 0 ? cb >> (t > 0 ? t - 1 : 0) & 1 : pb;
            const double ek = ec[t] * s;
            const double b = swp ? -c.v[t] * ek : ek;
            const double u1 = sw ? fma(dc[t], s, -lam) : b, u2 = sw ? ec[t + 1] * s : 0.0;
            const double ri = sw ? rc[t] : c.v[t + 1];
            const double y = FIRST ? td_start((uint32_t)i, (uint32_t)k) : c.y[t];
            const double x = fma(-u1, x1, fma(-u2, x2, y)) * ri;
            X[(int64_t)k * nev] = x;
            ss = fma(x, x, ss);
            if (!FIRST) {   // the largest entry's sign, the first row's of equal ones
                const bool up = fabs(x) >= big;
                big = up ? fabs(x) : big;
                sg = up ? (x < 0.0 ? -1.0 : 1.0) : sg;
            }
            x2 = x1;
            x1 = x;
        }
    };
    auto back_any = [&](const Chunk& c, int q, auto first) {
        if (q > 0 && (q + 1) * TD_CH + 1 < n) back(c, q, first, std::false_type{});
        else back(c, q, first, std::true_type{});
    };
    auto backward = [&](auto first) {
        constexpr bool FIRST = decltype(first)::value;
        ss = x1 = x2 = 0.0;
        Chunk a, b;
        load(a, nc - 1, true, !FIRST);
        for (int q = nc - 1; q >= 0; q -= 2) {
            load(b, q - 1, true, !FIRST);
            back_any(a, q, first);
            load(a, q - 2, true, !FIRST);
            if (q > 0) back_any(b, q - 1, first);
        }
    };
    // ---- forward substitution: row swaps and multipliers on x / ||x||, in place
    // (row k of the result is written once row k+1 has been read)
    auto forward = [&]() {
        const double inv = 1.0 / sqrt(ss);
        double carry = 0.0;
        bool sw = false;   // of row k-1
        double l = 0.0;
        auto forw = [&](const Chunk& c, int q, auto edge) {
            constexpr bool EDGE = decltype(edge)::value;
            const int k0 = q * TD_CH;
            const uint32_t cb = c.bits >> (k0 & 31);
            double ec[TD_CH];
#pragma unroll
            for (int t = 0; t < TD_CH; ++t) ec[t] = EDGE ? (k0 + t + 1 < n ? e[k0 + t] : 0.0) : e[k0 + t];
#pragma unroll
            for (int t = 0; t < TD_CH; ++t) {
                const int k = k0 + t;
                if (EDGE && k >= n) continue;
                const double x = c.y[t] * inv;
                if (!EDGE || k > 0) X[(int64_t)(k - 1) * nev] = sw ? x : carry;
                carry = sw ? fma(-l, x, carry) : fma(-l, carry, x);   // (k = 0: x)
                sw = cb >> t & 1;
                l = sw ? c.v[t + 1] : ec[t] * s * c.v[t + 1];
            }
        };
        auto forw_any = [&](const Chunk& c, int q) {
            if (q > 0 && (q + 1) * TD_CH < n) forw(c, q, std::false_type{});
            else forw(c, q, std::true_type{});
        };
        Chunk a, b;
        load(a, 0, false, true);
        for (int q = 0; q < nc; q += 2) {
            load(b, q + 1, false, true);
            forw_any(a, q);
            load(a, q + 2, false, true);
            if (q + 1 < nc) forw_any(b, q + 1);
        }
        X[(int64_t)(n - 1) * nev] = carry;
    };

    double base = shift.floor;
    for (int tries = 0; tries < 2; ++tries, base = full) {
        factor(base);
        backward(std::true_type{});
        forward();
        big = 0.0;
        backward(std::false_type{});
        if (ss > 0.0 && ss < 1e300) break;
    }
    sc[i] = sg / sqrt(ss);
}

// Modified Gram-Schmidt over each cluster of size >= 2 (one workgroup per
// eigenvalue index; only cluster starts with a successor in the cluster do
// work).  Vectors in the output Z (column-major, vector j = Z[j * ldz ..],
// contiguous, so the workgroup's threads read consecutive rows), already
// unit.
//
// A vector of which the subtractions leave less than TD_LEFT (of its square)
// held little that its predecessors did not: what is left of it carries their
// rounding, 1 / sqrt(TD_LEFT) times as large.  It gets one more step of inverse
// iteration from there, with the factors that k_td_invit left, which brings up
// what belongs to its eigenvalue, and is orthonormalised again.  (Four equal
// random blocks joined by 1e-20 .. 1e-8: 8 of 100 had residuals over 1e-13 ||T||,
// up to 8e-12; none with it.  Of 256 random vectors that span a cluster about 3
// need it.  A spectrum of pairs, n = 4096, nev = 2048: 4.5 ms with, 3.2 without.)
constexpr int TD_OT = 256;          // threads
constexpr double TD_LEFT = 1e-2;
constexpr int TD_TRIES = 3;

struct TdStage {   // TD_OT rows on their way through LDS
    double x[TD_OT], v[TD_OT + 1], d[TD_OT], e[TD_OT + 1], re[TD_OT];
    int sw[TD_OT + 1];
};

// x <- (T - lambda I)^{-1} z (scaled T), by the factors V, B of that vector: the
// workgroup moves the rows, one thread runs the two substitutions.
__device__ inline void td_solve(int n, int64_t nev, const double* __restrict__ d,
                                const double* __restrict__ e, const double* __restrict__ re,
                                double s, double lam, const double* __restrict__ V,
                                const uint32_t* __restrict__ B, const double* __restrict__ z,
                                double* __restrict__ x, TdStage& S)
{
    const int tid = threadIdx.x;
    auto swapped = [&](int k) { return k >= 0 && k < n && (B[(int64_t)(k >> 5) * nev] >> (k & 31) & 1); };
    auto ev = [&](int k) { return k + 1 < n ? e[k] * s : 0.0; };
    const int last = (n - 1) / TD_OT * TD_OT;
    double carry = 0.0, l = 0.0;
    int sw = 0;   // of the row before
    for (int k0 = 0; k0 <= last; k0 += TD_OT) {
        const int k = k0 + tid;
        if (k < n) {
            S.x[tid] = z[k];
            S.v[tid] = V[(int64_t)k * nev];
            S.e[tid] = ev(k);
            S.sw[tid] = swapped(k);
        }
        __syncthreads();
        if (tid == 0) {
            for (int t = 0; t < TD_OT && k0 + t < n; ++t) {
                const double y = S.x[t];
                S.x[t] = sw ? y : carry;   // of row k0 + t - 1
                carry = sw ? fma(-l, y, carry) : fma(-l, carry, y);
                sw = S.sw[t];
                l = sw ? S.v[t] : S.e[t] * S.v[t];
            }
        }
        __syncthreads();
        if (k > 0 && k < n) x[k - 1] = S.x[tid];
    }
    if (tid == 0) x[n - 1] = carry;
    double x1 = 0.0, x2 = 0.0;
    for (int k0 = last; k0 >= 0; k0 -= TD_OT) {
        const int k = k0 + tid;
        __syncthreads();
        if (k < n) {
            S.x[tid] = x[k];
            S.v[tid + 1] = V[(int64_t)k * nev];
            S.d[tid] = k + 1 < n ? fma(d[k + 1], s, -lam) : 0.0;
            S.re[tid] = k + 1 < n ? re[k] : 0.0;
            S.sw[tid + 1] = swapped(k);
        }
        S.e[tid] = ev(k);
        if (tid == 0) {
            S.e[TD_OT] = ev(k0 + TD_OT);
            S.v[0] = k0 > 0 ? V[(int64_t)(k0 - 1) * nev] : 0.0;
            S.sw[0] = swapped(k0 - 1);
        }
        __syncthreads();
        if (tid == 0) {
            for (int t = (n - k0 < TD_OT ? n - k0 : TD_OT) - 1; t >= 0; --t) {
                const bool su = S.sw[t + 1];
                const double u1 = su ? S.d[t] : S.sw[t] ? -S.v[t] * S.e[t] : S.e[t];
                const double u2 = su ? S.e[t + 1] : 0.0;
                const double xk = fma(-u1, x1, fma(-u2, x2, S.x[t])) * (su ? S.re[t] : S.v[t + 1]);
                S.x[t] = xk;
                x2 = x1;
                x1 = xk;
            }
        }
        __syncthreads();
        if (k < n) x[k] = S.x[tid];
    }
    __syncthreads();
}

__global__ __launch_bounds__(TD_OT) void k_td_ortho(int64_t n, int64_t nev,
                                                    const double* __restrict__ d,
                                                    const double* __restrict__ e,
                                                    const double* __restrict__ re,
                                                    const double* __restrict__ w,
                                                    const double* __restrict__ bounds,
                                                    const double* __restrict__ V,
                                                    const uint32_t* __restrict__ B,
                                                    double* __restrict__ X,
                                                    double* __restrict__ Z, int64_t ldz)
{
    // one partial per wave, double-buffered by call parity: outside td_solve each
    // thread only ever touches its own rows of Z (r = tid mod TD_OT), so the sums
    // are the only exchange, and one barrier per sum suffices (a wave can reach
    // the next sum's writes only after every wave has passed this one's barrier)
    __shared__ double red[2][4];
    __shared__ TdStage S;
    const int64_t i = blockIdx.x;
    const double thr = TD_CLUSTER * bounds[2];
    if (i > 0 && w[i] - w[i - 1] <= thr) return;            // not a cluster start
    if (i + 1 >= nev || w[i + 1] - w[i] > thr) return;       // a single eigenvalue
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    int parity = 0;
    auto block_sum = [&](double v) {
        v = wave_sum(v);
        if (lane == 0) red[parity][wv] = v;
        __syncthreads();
        const double s = (red[parity][0] + red[parity][1]) + (red[parity][2] + red[parity][3]);
        parity ^= 1;
        return s;
    };
    auto square = [&](const double* v) {
        double p = 0.0;
        for (int64_t r = tid; r < n; r += TD_OT) p = fma(v[r], v[r], p);
        return block_sum(p);
    };
    for (int64_t j = i + 1; j < nev && w[j] - w[j - 1] <= thr; ++j) {
        double* __restrict__ zj = Z + j * ldz;
        // takes z_i .. z_{j-1} out of z_j; what is left of its square
        auto reduce = [&]() {
            for (int64_t m = i; m < j; ++m) {
                const double* __restrict__ zm = Z + m * ldz;
                double p = 0.0;
                for (int64_t r = tid; r < n; r += TD_OT) p = fma(zj[r], zm[r], p);
                const double dt = block_sum(p);
                for (int64_t r = tid; r < n; r += TD_OT) zj[r] = fma(-dt, zm[r], zj[r]);
            }
            return square(zj);
        };
        for (int tries = 0;; ++tries) {
            // once, and again where little of the (unit) vector was left: what the
            // subtractions leave is orthogonal to eps over that little
            const double first = reduce();
            double left = first < TD_LEFT ? reduce() : first;
            if (!(left > 0.0)) {   // nothing: another start
                for (int64_t r = tid; r < n; r += TD_OT)
                    zj[r] = td_start((uint32_t)(nev + j), (uint32_t)r);
                left = reduce();
            }
            const double inv = 1.0 / sqrt(left);
            for (int64_t r = tid; r < n; r += TD_OT) zj[r] *= inv;
            if (first >= TD_LEFT || tries == TD_TRIES) break;
            double* __restrict__ xj = X + j * n;   // (the iterates are in Z by now)
            __syncthreads();
            td_solve((int)n, nev, d, e, re, bounds[3], td_shift(j, nev, w, bounds).lam,
                     V + j, B + j, zj, xj, S);
            const double ss = square(xj);
            if (!(ss > 0.0 && ss < 1e300)) break;
            const double xinv = 1.0 / sqrt(ss);
            for (int64_t r = tid; r < n; r += TD_OT) zj[r] = xj[r] * xinv;
        }
    }
}

// row-major X (n x nev) -> column-major Z (ldz), vector c times sc[c]
__global__ __launch_bounds__(256) void k_td_out(int64_t n, int64_t nev,
                                                const double* __restrict__ X,
                                                const double* __restrict__ sc,
                                                double* __restrict__ Z, int64_t ldz)
{
    __shared__ double tile[32][33];
    const int64_t r0 = (int64_t)blockIdx.x * 32, c0 = (int64_t)blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int q = ty; q < 32; q += 8) {
        const int64_t r = r0 + q, c = c0 + tx;
        if (r < n && c < nev) tile[q][tx] = X[r * nev + c];
    }
    __syncthreads();
    for (int q = ty; q < 32; q += 8) {
        const int64_t c = c0 + q, r = r0 + tx;
        if (r < n && c < nev) Z[c * ldz + r] = tile[tx][q] * sc[c];
    }
}

struct TdLayout {
    size_t e2 = 0, bounds = 0, x = 0, f = 0, p = 0, total = 0;
};

size_t tdal(size_t v) { return (v + 255) / 256 * 256; }

TdLayout td_layout(int64_t n, int64_t nev)
{
    TdLayout L;
    size_t off = 0;
    L.e2 = off;
    off = tdal(off + (size_t)(n > 1 ? n - 1 : 1) * 8);
    L.bounds = off;
    off = tdal(off + 4 * 8);
    L.x = off;
    off = tdal(off + (size_t)n * nev * 8);
    L.f = off;
    off = tdal(off + (size_t)n * nev * 4 * 8);
    L.p = off;
    off = tdal(off + (size_t)n * nev);
    L.total = off;
    return L;
}

}  // namespace

extern "C" {

int trbt_tridiag_eigh_workspace_bytes(int64_t n, int64_t nev, size_t* bytes)
{
    if (n < 0) return -1;
    if (nev < 0 || nev > n) return -2;
    if (!bytes) return -3;
    *bytes = (n > 0 && nev > 0) ? td_layout(n, nev).total : 0;
    return TRBT_SUCCESS;
}

int trbt_tridiag_eigh_d(int64_t n, int64_t nev, const double* d, const double* e, double* w,
                        double* Z, int64_t ldz, void* work, size_t work_bytes, void* stream)
{
    if (n < 0) return -1;
    if (nev < 0 || nev > n) return -2;
    if (nev > 0 && !d) return -3;
    if (nev > 0 && n > 1 && !e) return -4;
    if (nev > 0 && !w) return -5;
    if (nev > 0 && !Z) return -6;
    if (ldz < (n > 1 ? n : 1)) return -7;
    if (work && ((uintptr_t)work % TRBT_WORK_ALIGN)) return -8;
    if (nev == 0) return TRBT_SUCCESS;
    const TdLayout L = td_layout(n, nev);
    if (!work || work_bytes < L.total) return TRBT_ERR_WORKSPACE;
    int rc = check_device();
    if (rc) return rc;
    hipStream_t st = (hipStream_t)stream;
    char* ws = (char*)work;
    double* e2 = (double*)(ws + L.e2);
    double* bounds = (double*)(ws + L.bounds);
    double* X = (double*)(ws + L.x);
    // of the factors' n x nev x 4: V, then 1/e (n) and the vectors' scales (nev)
    double* V = (double*)(ws + L.f);
    double* re = V + (size_t)n * nev;
    double* sc = re + (size_t)n * nev;
    uint32_t* B = (uint32_t*)(ws + L.p);   // a bit per row and vector, of the n x nev bytes
    hipLaunchKernelGGL(k_td_prep, dim3(1), dim3(256), 0, st, n, d, e, e2, re, bounds);
    // lanes per eigenvalue: more lanes need fewer rounds (14, 11, 9 for 16, 32, 64),
    // and their waves are free while SIMDs stand idle (whole calls, ms: nev =
    // 400 of 400 0.298, 0.290, 0.274; 2000 of 4000 3.01, 3.00, 3.25; 4096 of
    // 8192 6.9, 7.4, 8.5; 12000 of 12000 13.9, 15.9, 20.7)
    auto bisect = [&](auto kern, int ms) {
        hipLaunchKernelGGL(kern, dim3((unsigned)((nev * ms + TD_THREADS - 1) / TD_THREADS)),
                           dim3(TD_THREADS), 0, st, n, nev, d, (const double*)e2,
                           (const double*)bounds, w);
    };
    if (nev <= 512) bisect(k_td_bisect<64>, 64);
    else if (nev <= 2048) bisect(k_td_bisect<32>, 32);
    else bisect(k_td_bisect<16>, 16);
    hipLaunchKernelGGL(k_td_invit, dim3((unsigned)((nev + TD_THREADS - 1) / TD_THREADS)),
                       dim3(TD_THREADS), 0, st, n, nev, d, e, (const double*)re,
                       (const double*)bounds, (const double*)w, X, V, B, sc);
    hipLaunchKernelGGL(k_td_out, dim3((unsigned)((n + 31) / 32), (unsigned)((nev + 31) / 32)),
                       dim3(256), 0, st, n, nev, (const double*)X, (const double*)sc, Z, ldz);
    hipLaunchKernelGGL(k_td_ortho, dim3((unsigned)nev), dim3(TD_OT), 0, st, n, nev,
                       d, e, (const double*)re, (const double*)w, (const double*)bounds,
                       (const double*)V, (const uint32_t*)B, X, Z, ldz);
    return hipGetLastError() == hipSuccess ? TRBT_SUCCESS : TRBT_ERR_HIP;
}

}  // extern "C"
