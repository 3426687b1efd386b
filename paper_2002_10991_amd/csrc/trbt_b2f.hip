// trbt_b2f.hip -- band-to-full eigenvector back-transformation on gfx950:
// C = P^* Y (Sec. 2.1, Eq. 2stage_bkwd2), the step after the
// tridiagonal-to-banded one, with P^* = H_0 H_1 ... H_{J-1} the Householder
// reflectors of the full-to-band reduction B = P A P^* (Eq. 2stage_fwd1):
// one reflector per column j = 0 .. n-nbw-2, acting on rows [j+nbw, n).
//
// Unlike the stage-2 reflectors (length <= nbw, a few per column of Z),
// these are long, so the update is GEMM-rich: PW consecutive reflectors
// form a panel, H_{j0} ... H_{j0+PW-1} = I - V T V^H (forward compact WY,
// T upper triangular), and the panels are applied last to first:
//     W = V^H Z,  W' = T W,  Z <- Z - V W'     (rows [j0+nbw, n) of Z).
//
// Kernels:
//  * k_b2f_gram (four workgroups per panel): the Gram matrix V^H V on FP64
//    MFMA, into the workspace.
//  * k_b2f_tfac (one workgroup per panel): T from it, in its place.
//  * k_b2f_apply (one workgroup per strip of 16 columns of Z, 8 waves): for
//    every panel p from the last to the first, the waves walk the panel's rows
//    in 16-row blocks (block b to wave b mod 8).  A block is loaded once into
//    MFMA accumulators, updated with panel p (Z -= V_p W'_p, W'_p in LDS),
//    stored, and -- while still in registers -- contracted with the next
//    panel's reflectors, W_{p-1} += V_{p-1}^H Z.  So each panel reads and
//    writes its rows of Z once.  The waves' partial W_{p-1} are summed in wave
//    order through LDS (bitwise reproducible), multiplied by T_{p-1} on MFMA
//    into W'_{p-1}, and the next panel starts.
//
// What bounds it: the strips re-read the reflectors, every element twice, from
// L2; at 16 columns that is 4 flops a byte real and 8 complex.  L2 reads (counted at 128
// bytes): real n = 8192, nev = 4096 10.7 TB/s over the chip, 17 bytes a clock and CU;
// complex n = 32768, nev = 8192 7.5 TB/s, half of them from beyond the XCD's L2.
// Skipping those loads
// (a timing-only variant) took 10.3 and 125 ms where the kernel takes 14.1
// and 159 (real n = 8192, complex n = 16384, nev = 4096; the matrix
// instructions alone 7.7 and 112).  Wider strips would halve the reads and leave
// half of the CUs without one at nev = 4096; more waves on a strip than one
// workgroup holds would need memory to add their W in.  The form before (real
// panels of 64, loads just ahead of their use, T in one serial workgroup
// per panel): 26.6 and 319 ms, 2.1 and 6.8 of them for T (now 0.2 and 1.2).
//
// Register layout of v_mfma_f64_16x16x4_f64 (A lane i+16k = A[i][k], B lane
// j+16k = B[k][j], D lane j+16g element e = D[g+4e][j]): a tile in accumulator
// layout is the B operand of four chunks as it stands, element e the chunk whose
// four rows lane groups 0..3 hold in it.

#include <hip/hip_runtime.h>

#include <stdint.h>

#include <mutex>
#include <type_traits>

#include "trbt.h"
#include "trbt_device.h"

namespace {

constexpr int B2F_UNIT = 64;       // reflectors per 64 x 64 unit of the workspace
constexpr int B2F_NW = 8;          // waves per workgroup
constexpr int B2F_HDR = 256;       // workspace header: fault word (unused here), step counters
constexpr int B2F_ROUND = 256;     // workgroups the chip holds at a time (CUs; locality only)
constexpr int B2F_STEPS = 56;      // step counters, from byte 32 of the header
constexpr uint64_t B2F_STEP_TICKS = 5000;   // 50 us of the 100 MHz wall clock

// Reflectors per panel: a pass over Z reads and writes it once per panel, so a
// real panel of 64 would ask for 16 flop per byte of Z, the rate at which
// memory and the matrix cores take the same time; 128 halves that traffic.
// Complex elements carry four times the flops for twice the bytes.
template <bool CPLX>
struct B2F {
    static constexpr int PW = CPLX ? 64 : 128;
    static constexpr int PT = PW / 16;              // 16 x 16 tiles across a panel
    static constexpr int NC = CPLX ? 2 : 1;
    static constexpr int TILE = 256 * NC;           // doubles per tile
    static constexpr int64_t TP = (int64_t)PW / B2F_UNIT * B2F_UNIT * B2F_UNIT * NC;   // per panel
};

// T (and before it the Gram matrix) of a panel in its part of the workspace:
// the tiles (a, b), a <= b, of the upper triangle, each stored as the four A
// operand chunks of v_mfma_f64_16x16x4_f64 (chunk c, lane i + 16k: element
// [i][4c + k]; complex: the imaginary parts 256 doubles on).  Two diagonal
// tiles share one: that of an even b in its strictly upper part, that of the odd
// b + 1 transposed in the strictly lower part; the diagonal is tau.  So a
// panel of 128 takes 28 + 4 tiles, the two 64 x 64 units it has, and the first
// 64 columns the first unit alone (all a short last panel has).
__host__ __device__ constexpr int b2f_tile(int a, int b)   // a < b
{
    const int m = b / 2;
    return 2 * m * m + (b % 2 ? 2 * m : 0) + a;
}
__host__ __device__ constexpr int b2f_diag_tile(int b) { return 2 * (b / 2) * (b / 2) + 4 * (b / 2) + 1; }

// position of element [i][j] in a tile
__device__ inline int b2f_pos(int i, int j) { return (j >> 2) * 64 + i + 16 * (j & 3); }

__host__ __device__ inline int64_t b2f_reflectors(int64_t n, int nbw)
{
    return (nbw >= 1 && n - nbw - 1 > 0) ? n - nbw - 1 : 0;
}

template <bool CPLX>
__host__ __device__ inline int64_t b2f_panels(int64_t J)
{
    return (J + B2F<CPLX>::PW - 1) / B2F<CPLX>::PW;
}

// one stored element: real or complex (interleaved re, im)
template <bool CPLX>
struct Elt;
template <>
struct Elt<false> {
    double re;
    static constexpr double im = 0.0;
};
template <>
struct Elt<true> {
    double re, im;
};

template <bool CPLX>
__device__ inline Elt<CPLX> ld_elt(const double* __restrict__ p, int64_t idx)
{
    Elt<CPLX> e;
    if constexpr (CPLX) {
        const d2 v = *reinterpret_cast<const d2*>(p + 2 * idx);
        e.re = v.x;
        e.im = v.y;
    } else {
        e.re = p[idx];
    }
    return e;
}

template <bool CPLX>
__device__ inline void st_elt(double* __restrict__ p, int64_t idx, double re, double im)
{
    if constexpr (CPLX) {
        d2 v;
        v.x = re;
        v.y = im;
        *reinterpret_cast<d2*>(p + 2 * idx) = v;
    } else {
        (void)im;
        p[idx] = re;
    }
}

// element (row r, reflector j) of the stored reflectors, or 0 where the
// reflector has no entry (rows above its start j+nbw, rows >= n): a load from
// a clamped address inside the n x J array and a select.  Reflectors j >= J
// give those of J-1; T has zeros in their rows and columns.
template <bool CPLX>
__device__ inline Elt<CPLX> v_sel(const double* __restrict__ V, int64_t ldv, int64_t n,
                                  int nbw, int64_t J, int64_t r, int64_t j)
{
    const bool ok = r >= j + nbw && r < n;
    const int64_t rr = r < n ? r : n - 1, jj = j < J ? j : J - 1;
    Elt<CPLX> e = ld_elt<CPLX>(V, rr + jj * ldv);
    e.re = ok ? e.re : 0.0;
    if constexpr (CPLX) e.im = ok ? e.im : 0.0;
    return e;
}

// D += conj(A) B or, with NEG, D -= A B, on FP64 MFMA (complex: four products).
template <bool CPLX>
__device__ inline void mma_conj(Elt<CPLX> a, double br, double bi, Tile<CPLX>& d)
{
    d.re = mfma(a.re, br, d.re);
    if constexpr (CPLX) {
        d.im = mfma(a.re, bi, d.im);
        d.re = mfma(a.im, bi, d.re);
        d.im = mfma_n<1>(a.im, br, d.im);
    }
}

template <bool CPLX>
__device__ inline void mma_sub(Elt<CPLX> a, double br, double bi, Tile<CPLX>& d)
{
    d.re = mfma_n<1>(a.re, br, d.re);
    if constexpr (CPLX) {
        d.im = mfma_n<1>(a.re, bi, d.im);
        d.re = mfma(a.im, bi, d.re);
        d.im = mfma_n<1>(a.im, br, d.im);
    }
}

template <bool CPLX>
__device__ inline void mma_add(Elt<CPLX> a, double br, double bi, Tile<CPLX>& d)
{
    d.re = mfma(a.re, br, d.re);
    if constexpr (CPLX) {
        d.im = mfma(a.re, bi, d.im);
        d.re = mfma_n<1>(a.im, bi, d.re);
        d.im = mfma(a.im, br, d.im);
    }
}

template <bool CPLX>
__device__ inline Tile<CPLX> tile0()
{
    Tile<CPLX> t;
    t.re = d4{0.0, 0.0, 0.0, 0.0};
    if constexpr (CPLX) t.im = t.re;
    return t;
}

template <bool CPLX>
__device__ inline double imag(const Tile<CPLX>& t, int e)
{
    if constexpr (CPLX) return t.im[e];
    else return 0.0;
}

// --------------------------------------------------------------------------
// k_b2f_gram: the tiles a <= b of G = V^H V of panel blockIdx.x, strictly upper
// part, into the panel's part of the workspace.  blockIdx.y = 0, 1: the
// diagonal quads (a, b both in the first, second half of the tiles); 2, 3: a
// in the first half, b in the two quarters of the second (one workgroup per
// panel and a quarter of its tiles fills the chip at a few thousand
// reflectors).  The waves take the 16-row blocks in turn and are summed as a
// tree in a fixed order.
//
// Rows in registers: lane i + 16g holds rows r0+4g .. r0+4g+3 of column i, one
// 32-byte read.  Element e of the four lane groups is then rows r0+4g+e:
// any four rows may form a chunk of the contraction, so the chunk e of A (conj V)
// and of B (V) is the same register.
// --------------------------------------------------------------------------
template <bool CPLX, int NA, int NB, bool DIAG>
__device__ inline void gram_part(int64_t n, int nbw, const double* __restrict__ V, int64_t ldv,
                                 int64_t J, int64_t j0, int a0, int b0, double* __restrict__ Tp,
                                 double* red)
{
    constexpr int NT = DIAG ? NA * (NA + 1) / 2 : NA * NB;
    constexpr int NC = B2F<CPLX>::NC;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i16 = lane & 15, g4 = lane >> 4;
    Tile<CPLX> acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = tile0<CPLX>();
    const int64_t lo = j0 + 16 * (DIAG ? a0 : b0) + nbw;   // first row of the part's products
    for (int64_t r0 = (lo & ~(int64_t)15) + 16 * w; r0 < n; r0 += 16 * B2F_NW) {
        Elt<CPLX> x[NA + (DIAG ? 0 : NB)][4];
        const int64_t jl = j0 + 16 * (DIAG ? a0 + NA : b0 + NB) - 1;   // the part's last reflector
        if (r0 >= jl + nbw && r0 + 16 <= n && jl < J) {
#pragma unroll
            for (int t = 0; t < NA + (DIAG ? 0 : NB); ++t) {
                const int64_t j = j0 + 16 * (t < NA ? a0 + t : b0 + t - NA) + i16;
#pragma unroll
                for (int e = 0; e < 4; ++e) x[t][e] = ld_elt<CPLX>(V, r0 + 4 * g4 + e + j * ldv);
            }
        } else {
#pragma unroll
            for (int t = 0; t < NA + (DIAG ? 0 : NB); ++t) {
                const int64_t j = j0 + 16 * (t < NA ? a0 + t : b0 + t - NA) + i16;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    x[t][e] = v_sel<CPLX>(V, ldv, n, nbw, J, r0 + 4 * g4 + e, j);
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            int t = 0;
#pragma unroll
            for (int b = 0; b < (DIAG ? NA : NB); ++b)
#pragma unroll
                for (int a = 0; a < (DIAG ? b + 1 : NA); ++a, ++t) {
                    const Elt<CPLX> v = x[DIAG ? b : NA + b][e];
                    mma_conj<CPLX>(x[a][e], v.re, v.im, acc[t]);
                }
        }
    }
    // sum the waves: 4..7 onto 0..3, 2..3 onto 0..1, 1 onto 0
#pragma unroll
    for (int h = B2F_NW / 2; h > 0; h /= 2) {
        __syncthreads();
        if (w >= h && w < 2 * h) {
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    double* q = red + (((w - h) * NT + t) * NC * 4 + e) * 64 + lane;
                    q[0] = acc[t].re[e];
                    if constexpr (CPLX) q[256] = acc[t].im[e];
                }
        }
        __syncthreads();
        if (w < h) {
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double* q = red + ((w * NT + t) * NC * 4 + e) * 64 + lane;
                    acc[t].re[e] += q[0];
                    if constexpr (CPLX) acc[t].im[e] += q[256];
                }
        }
    }
    if (w == 0) {
        int t = 0;
#pragma unroll
        for (int b = 0; b < (DIAG ? NA : NB); ++b)
#pragma unroll
            for (int a = 0; a < (DIAG ? b + 1 : NA); ++a, ++t) {
                const int ta = a0 + a, tb = b0 + b;
                const bool dg = DIAG && a == b;
                double* tp = Tp + (int64_t)(dg ? b2f_diag_tile(tb) : b2f_tile(ta, tb)) *
                                      B2F<CPLX>::TILE;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int i = g4 + 4 * e, j = i16;   // element [i][j] of the tile
                    if (dg && i >= j) continue;
                    const int pos = dg && (tb & 1) ? b2f_pos(j, i) : b2f_pos(i, j);
                    tp[pos] = acc[t].re[e];
                    if constexpr (CPLX) tp[256 + pos] = acc[t].im[e];
                }
            }
    }
}

template <bool CPLX>
__global__ __launch_bounds__(64 * B2F_NW) void k_b2f_gram(int64_t n, int nbw,
                                                          const double* __restrict__ V,
                                                          int64_t ldv, double* __restrict__ Tw)
{
    constexpr int H = B2F<CPLX>::PT / 2, Q = H / 2;
    constexpr int RT = H * (H + 1) / 2 > H * Q ? H * (H + 1) / 2 : H * Q;
    __shared__ double red[B2F_NW / 2 * RT * B2F<CPLX>::TILE];
    const int64_t J = b2f_reflectors(n, nbw);
    const int64_t j0 = (int64_t)blockIdx.x * B2F<CPLX>::PW;
    double* Tp = Tw + blockIdx.x * B2F<CPLX>::TP;
    const int y = blockIdx.y;
    // (a short last panel has room for the first 64 columns only, and no others)
    if (y > 0 && j0 + 16 * H >= J) return;
    if (y < 2) gram_part<CPLX, H, H, true>(n, nbw, V, ldv, J, j0, H * y, H * y, Tp, red);
    else gram_part<CPLX, H, Q, false>(n, nbw, V, ldv, J, j0, 0, H + Q * (y - 2), Tp, red);
}

// --------------------------------------------------------------------------
// k_b2f_tfac: T of panel blockIdx.x in place of its Gram matrix: the forward
// compact-WY factor T = (I + D N)^{-1} D with D = diag(tau) and N the strictly
// upper part of G (the same T as the column recursion T[0:q, q] =
// -tau_q T[0:q, 0:q] G[0:q, q], also for tau = 0).  One wave per 16 columns b:
// the diagonal tiles by back substitution, one lane per column, then tile by
// tile upwards T[a][b] = -T[a][a] sum_{a<c<=b} N[a][c] T[c][b] on FP64 MFMA (a
// result tile is the next product's B operand as it stands).
// --------------------------------------------------------------------------
template <bool CPLX>
__global__ __launch_bounds__(64 * B2F<CPLX>::PT) void k_b2f_tfac(int64_t n, int nbw,
                                                                 const double* __restrict__ tau,
                                                                 double* __restrict__ Tw)
{
    using B = B2F<CPLX>;
    constexpr int PT = B::PT, NC = B::NC, TILE = B::TILE, NS = PT * PT / 2;
    const int64_t J = b2f_reflectors(n, nbw);
    const int64_t j0 = (int64_t)blockIdx.x * B::PW;
    double* __restrict__ Tp = Tw + blockIdx.x * B::TP;
    __shared__ double N[NS * TILE];
    __shared__ double Td[PT][16][17][NC];
    const int lane = threadIdx.x & 63, i16 = lane & 15, g4 = lane >> 4;
    const int b = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool half = j0 + 8 * PT >= J;   // a short last panel: the first half of the tiles
    const int ns = half ? PT * PT / 8 : NS;
    for (int x = threadIdx.x; x < ns * TILE; x += 64 * PT) N[x] = Tp[x];
    __syncthreads();
    const bool act = !half || b < PT / 2;
    if (act && lane < 16) {
        const double* S = N + b2f_diag_tile(b) * TILE;
        const int p = lane;
        for (int i = 15; i >= 0; --i) {
            const int64_t q = j0 + 16 * b + i;
            Elt<CPLX> u{};
            if (q < J) u = ld_elt<CPLX>(tau, q);
            double tr = u.re, ti = u.im;
            if (i < p) {
                double wr = 0.0, wi = 0.0;   // sum_{k=i+1}^{p} N[i][k] T[k][p]
                for (int k = i + 1; k <= p; ++k) {
                    const int pos = b & 1 ? b2f_pos(k, i) : b2f_pos(i, k);
                    const double gr = S[pos], xr = Td[b][k][p][0];
                    if constexpr (CPLX) {
                        const double gi = S[256 + pos], xi = Td[b][k][p][NC - 1];
                        wr += gr * xr - gi * xi;
                        wi += gr * xi + gi * xr;
                    } else {
                        wr += gr * xr;
                    }
                }
                tr = -(u.re * wr - u.im * wi);
                ti = -(u.re * wi + u.im * wr);
            } else if (i > p) {
                tr = ti = 0.0;
            }
            Td[b][i][p][0] = tr;
            if constexpr (CPLX) Td[b][i][p][NC - 1] = ti;
        }
    }
    __syncthreads();
    if (!act) return;
    Tile<CPLX> t[PT];
#pragma unroll
    for (int c = 0; c < PT; ++c) {
        t[c] = tile0<CPLX>();
        if (c == b) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                t[c].re[e] = Td[b][g4 + 4 * e][i16][0];
                if constexpr (CPLX) t[c].im[e] = Td[b][g4 + 4 * e][i16][NC - 1];
            }
        }
    }
    auto chunk = [&](const double* S, int e) {
        Elt<CPLX> v{};
        v.re = S[e * 64 + lane];
        if constexpr (CPLX) v.im = S[256 + e * 64 + lane];
        return v;
    };
#pragma unroll
    for (int a = PT - 2; a >= 0; --a) {
        if (a >= b) continue;
        Tile<CPLX> s = tile0<CPLX>();
#pragma unroll
        for (int c = a + 1; c < PT; ++c) {
            if (c > b) continue;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                mma_add<CPLX>(chunk(N + b2f_tile(a, c) * TILE, e), t[c].re[e], imag(t[c], e), s);
        }
        Tile<CPLX> r = tile0<CPLX>();
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            Elt<CPLX> v{};
            v.re = Td[a][i16][4 * e + g4][0];
            if constexpr (CPLX) v.im = Td[a][i16][4 * e + g4][NC - 1];
            mma_sub<CPLX>(v, s.re[e], imag(s, e), r);
        }
        t[a] = r;
    }
    // every wave has its N in LDS, so T can go over G
#pragma unroll
    for (int a = 0; a < PT; ++a) {
        if (a > b) continue;
        double* tp = Tp + (int64_t)(a == b ? b2f_diag_tile(b) : b2f_tile(a, b)) * TILE;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = g4 + 4 * e, j = i16;
            if (a == b && i >= j) continue;
            const int pos = a == b && (b & 1) ? b2f_pos(j, i) : b2f_pos(i, j);
            tp[pos] = t[a].re[e];
            if constexpr (CPLX) tp[256 + pos] = t[a].im[e];
        }
    }
}

// --------------------------------------------------------------------------
// k_b2f_apply
// --------------------------------------------------------------------------
template <bool CPLX>
struct B2FLds {
    // the waves' partial W, in accumulator layout: [tile][element e][plane][lane];
    // summed over the waves into the first
    double W[B2F_NW][B2F<CPLX>::PT][4][B2F<CPLX>::NC][64];
    double Wp[B2F<CPLX>::PT][4][B2F<CPLX>::NC][64];   // W' = T W
};

// buffer resources with a scalar offset per load: no vector address arithmetic
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

__device__ inline d2 buf_d2(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff)
{
    return __builtin_bit_cast(d2, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
}

__device__ inline __amdgpu_buffer_rsrc_t b2f_rsrc(const double* p, int64_t bytes)
{
    const int64_t cap = (int64_t)1 << 31;   // offsets stay below (checked on the host)
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(p), 0,
                                             (int)(bytes < cap ? bytes : cap - 1), 0x00020000);
}

// The strip kernel.  For every panel p from P to 0 one pass over the rows of the
// strip: Z -= V_p W'_p (p < P, W'_p in LDS) and w = V_{p-1}^H Z (p > 0), in
// 16-row blocks dealt to the waves in turn; then the waves' w are summed and
// multiplied by T_{p-1}.
//
// Rows in registers as in k_b2f_gram: element e of lane group g is row r0+4g+e,
// so a lane reads and writes 32 contiguous bytes of its column of Z (64
// complex) and of the reflectors of the contraction; the update's A operand
// takes its rows in the same order (row i of the product is r0 + 4 (i%4) + i/4).
//
// The blocks inside the matrix run as a pipeline: each operand register is loaded
// again, half a block ahead, as soon as the matrix instruction that reads it has
// been issued, and on into the wave's next block (a whole block ahead, twice
// the registers, was slower: real 15.9 -> 18.1 ms, complex 199 -> 255 ms at the
// sizes below).  The blocks on the slope, where reflectors start (the first
// 2 PW rows of a pass), run in it with masks.
//
// FAST: two panels of reflectors fit a 32-bit byte range; otherwise every block
// goes the slow way of a ragged last one, with 64-bit addresses.
template <bool CPLX, bool FAST>
__global__ __launch_bounds__(64 * B2F_NW) void k_b2f_apply(
    int64_t n, int nbw, int64_t nev, const double* __restrict__ V, int64_t ldv,
    const double* __restrict__ tau, const double* __restrict__ Tw, double* __restrict__ Z,
    int64_t ldz, int* __restrict__ steps)
{
    using B = B2F<CPLX>;
    constexpr int PW = B::PW, PT = B::PT, NC = B::NC, SZ = 8 * NC;
    constexpr int NU = PW / 4, RU = NU / 2, RA = PT / 2;   // update chunks; operands in flight
    __shared__ B2FLds<CPLX> S;
    const int64_t J = b2f_reflectors(n, nbw);
    const int64_t P = b2f_panels<CPLX>(J);
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i16 = lane & 15, g4 = lane >> 4;
    const int64_t col = (int64_t)blockIdx.x * 16 + i16;
    const bool colok = col < nev;
    double* __restrict__ zc = Z + (colok ? col : nev - 1) * ldz * NC;
    const int iperm = 4 * (i16 & 3) + (i16 >> 2);
    const double* wl = &S.Wp[0][0][0][lane];
    auto wp = [&](int c, int pl) { return wl[(c * NC + pl) * 64]; };   // chunk c of W'

    Tile<CPLX> w[PT];   // this wave's partial W of the next panel
#pragma unroll
    for (int a = 0; a < PT; ++a) w[a] = tile0<CPLX>();
    Elt<CPLX> vu[RU], va[RA][4];
    Tile<CPLX> z;

    // Workgroups of one XCD (blockIdx mod 8) and one round of the chip keep in
    // step, panel by panel: they read the same reflectors at the same time, and
    // once they drift apart by more than its L2 holds beside their streams of Z
    // each fetches them again.  Only a matter of speed, so the wait is short
    // and is given up for good when it runs out.
    const int group = blockIdx.x / B2F_ROUND * 8 + blockIdx.x % 8;
    const int first = blockIdx.x / B2F_ROUND * B2F_ROUND + blockIdx.x % 8;
    const int peers = ((int)gridDim.x - first + 7) / 8 < B2F_ROUND / 8
                          ? ((int)gridDim.x - first + 7) / 8 : B2F_ROUND / 8;
    // Short passes drift too little to pay for it, nor do few strips.  Without and
    // with, nbw = 64, ms (n, nev): real (8192, 8192) 28.1 and 29.7, (12000, 8192)
    // 62.2 and 62.2, (16384, 4096) 55.1 and 57.2, (20480, 1000) 80.0 and 80.4,
    // (20480, 4096) 98.0 and 89.8, (24001, 2001) 148 and 126, (28000, 4096) 184 and
    // 164; complex (3000, 3000) 5.5 and 5.7, (5000, 5000) 30.9 and 30.7, (6144, 1500)
    // 20.1 and 20.6, (6144, 4096) 23.2 and 23.0, (8192, 4096) 41.6 and 39.9,
    // (10000, 8000) 134 and 121, (16384, 4096) 184 and 159.
    bool together = n >= (CPLX ? 6144 : 20480) && group < B2F_STEPS && peers > 1;
    auto keep_step = [&](int need) {   // one lane
        atomicAdd(&steps[group], 1);
        const uint64_t t0 = wall_clock64();
        while (__hip_atomic_load(&steps[group], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < need) {
            __builtin_amdgcn_s_sleep(2);
            if (wall_clock64() - t0 > B2F_STEP_TICKS) {
                together = false;
                break;
            }
        }
    };

    for (int64_t p = P; p >= 0; --p) {
        const bool upd = p < P, acc = p > 0;
        const int64_t jp = p * PW, jn = jp - PW;      // first reflectors of panels p, p-1
        const int64_t lo = (acc ? jn : jp) + nbw;     // first row of the pass
        int64_t r0 = (lo & ~(int64_t)15) + 16 * wv;   // this wave's first block
        const bool pipe = FAST && r0 + 16 <= n;

        // The reflectors through a buffer resource: a constant offset per lane, a
        // scalar one per load.  Those >= J (a short last panel) read J-1's; T has
        // zeros in their rows and columns.
        const int64_t jb = acc ? jn : jp, je = upd ? jp + PW : jp;
        const __amdgpu_buffer_rsrc_t rv =
            b2f_rsrc(V + jb * ldv * NC, (((je < J ? je : J) - 1 - jb) * ldv + n) * SZ);
        const uint32_t lb = (uint32_t)ldv * SZ;
        const uint32_t lastc = (uint32_t)(J - 1 - jb);
        const bool clip = FAST && je > J;
        const uint32_t ou = (uint32_t)((jp - jb + g4) * ldv + iperm) * SZ;
        const uint32_t oa = (uint32_t)((int64_t)i16 * ldv + 4 * g4) * SZ;
        // chunk k of the update, V[r0 + perm][jp + 4k + g], rows from byte rb
        auto ld_u = [&](int k, uint32_t rb) {
            uint32_t vo = ou, so = rb + (uint32_t)(4 * k) * lb;
            if (clip) {
                const uint32_t c = (uint32_t)(jp - jb) + 4 * k + g4;
                vo = (c < lastc ? c : lastc) * lb + iperm * SZ;
                so = rb;
            }
            if constexpr (CPLX) {
                const d2 v = buf_d2(rv, vo, so);
                vu[k % RU].re = v.x;
                vu[k % RU].im = v.y;
            } else {
                vu[k % RU].re = buffer_load_f64(rv, vo, so);
            }
        };
        // tile t of the contraction, V[r0 + 4g + e][jn + 16t + i]
        auto ld_a = [&](int t, uint32_t rb) {
            uint32_t vo = oa, so = rb + (uint32_t)(16 * t) * lb;
            if (clip) {
                const uint32_t c = 16 * t + i16;
                vo = (c < lastc ? c : lastc) * lb + 4 * g4 * SZ;
                so = rb;
            }
            if constexpr (CPLX) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const d2 v = buf_d2(rv, vo + 16 * e, so);
                    va[t % RA][e].re = v.x;
                    va[t % RA][e].im = v.y;
                }
            } else {
#pragma unroll
                for (int e = 0; e < 4; e += 2) {
                    const d2 v = buf_d2(rv, vo + 8 * e, so);
                    va[t % RA][e].re = v.x;
                    va[t % RA][e + 1].re = v.y;
                }
            }
        };
        auto ld_z = [&](int64_t r, Tile<CPLX>& x) {
            const double* q = zc + (r + 4 * g4) * NC;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                x.re[e] = q[e * NC];
                if constexpr (CPLX) x.im[e] = q[e * NC + 1];
            }
        };

        // ---- W'_p: sum the waves' partials of W_p in wave order (wave a the
        // tile a), then W'_p = T_p W_p; meanwhile the pass's first operands
        if (upd) {
#pragma unroll
            for (int a = 0; a < PT; ++a)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    S.W[wv][a][e][0][lane] = w[a].re[e];
                    if constexpr (CPLX) S.W[wv][a][e][NC - 1][lane] = w[a].im[e];
                }
        }
        if (pipe) {
            if (upd) {
#pragma unroll
                for (int k = 0; k < RU; ++k) ld_u(k, (uint32_t)r0 * SZ);
            }
            if (acc) {
#pragma unroll
                for (int t = 0; t < RA; ++t) ld_a(t, (uint32_t)r0 * SZ);
            }
        }
        __syncthreads();   // (and the strip's rows are as the pass before left them)
        if (pipe) ld_z(r0, z);
        if (upd) {
            if (threadIdx.x == 0 && together) keep_step(peers * (int)(P - p));
            if (wv < PT) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int c = 0; c < NC; ++c) {
                        double x = S.W[0][wv][e][c][lane];
#pragma unroll
                        for (int q = 1; q < B2F_NW; ++q) x += S.W[q][wv][e][c][lane];
                        S.W[0][wv][e][c][lane] = x;
                    }
            }
            __syncthreads();
            if (wv < PT) {
                // (a short last panel: T has only the first half of the tiles)
                const int nt = jp + 8 * PT >= J ? PT / 2 : PT;
                const double* __restrict__ Tp = Tw + p * B::TP;
                Tile<CPLX> y = tile0<CPLX>();
                if (wv < nt) {
                    const double* sd = Tp + b2f_diag_tile(wv) * B::TILE;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int j = 4 * e + g4;   // element [i16][j] of the diagonal tile
                        const int pos = wv & 1 ? b2f_pos(j, i16) : b2f_pos(i16, j);
                        const int64_t q = jp + 16 * wv + j;
                        const Elt<CPLX> td = ld_elt<CPLX>(tau, q < J ? q : J - 1);
                        Elt<CPLX> v{};
                        v.re = i16 < j ? sd[pos] : i16 == j && q < J ? td.re : 0.0;
                        if constexpr (CPLX)
                            v.im = i16 < j ? sd[256 + pos] : i16 == j && q < J ? td.im : 0.0;
                        mma_add<CPLX>(v, S.W[0][wv][e][0][lane],
                                      CPLX ? S.W[0][wv][e][NC - 1][lane] : 0.0, y);
                    }
                    for (int b = wv + 1; b < nt; ++b) {
                        const double* st = Tp + b2f_tile(wv, b) * B::TILE + lane;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            Elt<CPLX> v{};
                            v.re = st[e * 64];
                            if constexpr (CPLX) v.im = st[256 + e * 64];
                            mma_add<CPLX>(v, S.W[0][b][e][0][lane],
                                          CPLX ? S.W[0][b][e][NC - 1][lane] : 0.0, y);
                        }
                    }
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    S.Wp[wv][e][0][lane] = y.re[e];
                    if constexpr (CPLX) S.Wp[wv][e][NC - 1][lane] = y.im[e];
                }
            }
            __syncthreads();
#pragma unroll
            for (int a = 0; a < PT; ++a) w[a] = tile0<CPLX>();
        }

        // ---- the rows.  One block of the pipeline; EDGE: on the slope.
        auto block = [&](auto edge) {
            constexpr bool EDGE = decltype(edge)::value;
            const int64_t rn = r0 + 16 * B2F_NW;
            const bool more = rn + 16 <= n;
            const uint32_t rc = (uint32_t)r0 * SZ;                  // this block
            const uint32_t rb = (uint32_t)(more ? rn : r0) * SZ;    // the next (the last: its own again)
            Tile<CPLX> zn;
            ld_z(more ? rn : r0, zn);
            asm volatile("" ::: "memory");       // W' from LDS again in every block
            if (upd && (!EDGE || r0 + 16 > jp + nbw)) {
                const int du = (int)(jp + nbw - r0);   // entry of row r, reflector jp+x: r - r0 - x >= du
                Tile<CPLX> zu = z, z2 = tile0<CPLX>();
#pragma unroll
                for (int k = 0; k < NU; ++k) {
                    Elt<CPLX> v = vu[k % RU];
                    if (EDGE) {
                        const bool ok = iperm - g4 >= du + 4 * k;
                        v.re = ok ? v.re : 0.0;
                        if constexpr (CPLX) v.im = ok ? v.im : 0.0;
                    }
                    if (k + RU < NU) ld_u(k + RU, rc);
                    else ld_u(k + RU - NU, rb);
                    mma_sub<CPLX>(v, wp(k, 0), CPLX ? wp(k, NC - 1) : 0.0,
                                  (!CPLX && (k & 1)) ? z2 : zu);
                }
                if constexpr (!CPLX) zu.re += z2.re;
                double* q = zc + (r0 + 4 * g4) * NC;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (EDGE && 4 * g4 + e < du) continue;   // a row above the panel's
                    z.re[e] = zu.re[e];
                    if constexpr (CPLX) z.im[e] = zu.im[e];
                    if (colok) {
                        q[e * NC] = z.re[e];
                        if constexpr (CPLX) q[e * NC + 1] = z.im[e];
                    }
                }
            } else if (upd) {
#pragma unroll
                for (int k = 0; k < RU; ++k) ld_u(k, rb);
            }
            if (acc) {
                const int da = (int)(jn + nbw - r0);
                if (EDGE) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const bool ok = 4 * g4 + e >= da;
                        z.re[e] = ok ? z.re[e] : 0.0;
                        if constexpr (CPLX) z.im[e] = ok ? z.im[e] : 0.0;
                    }
                }
#pragma unroll
                for (int t = 0; t < PT; t += 2) {
                    Elt<CPLX> v[2][4];
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            v[h][e] = va[(t + h) % RA][e];
                            if (EDGE) {
                                const bool ok = 4 * g4 + e - i16 >= da + 16 * (t + h);
                                v[h][e].re = ok ? v[h][e].re : 0.0;
                                if constexpr (CPLX) v[h][e].im = ok ? v[h][e].im : 0.0;
                            }
                        }
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        if (t + h + RA < PT) ld_a(t + h + RA, rc);
                        else ld_a(t + h + RA - PT, rb);
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        mma_conj<CPLX>(v[0][e], z.re[e], imag(z, e), w[t]);
                        mma_conj<CPLX>(v[1][e], z.re[e], imag(z, e), w[t + 1]);
                    }
                }
            }
            z = zn;
            r0 = rn;
        };
        if constexpr (FAST) {
            const int64_t slope = (upd ? jp : jn) + PW - 1 + nbw;   // below: every reflector's rows
            while (r0 + 16 <= n && r0 < slope) block(std::true_type{});
            while (r0 + 16 <= n) block(std::false_type{});
        }
        // ---- a ragged last block: clamped loads, masked values
        for (; r0 < n; r0 += 16 * B2F_NW) {
            Tile<CPLX> x;
            int64_t r[4];
            bool rok[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                r[e] = r0 + 4 * g4 + e;
                rok[e] = r[e] < n && r[e] >= lo;
                const Elt<CPLX> v = ld_elt<CPLX>(zc, r[e] < n ? r[e] : n - 1);
                x.re[e] = rok[e] ? v.re : 0.0;
                if constexpr (CPLX) x.im[e] = rok[e] ? v.im : 0.0;
            }
            if (upd && r0 + 16 > jp + nbw) {
                Tile<CPLX> zu = x;
#pragma unroll
                for (int h = 0; h < NU; h += RU) {
#pragma unroll
                    for (int k = 0; k < RU; ++k)
                        vu[k] = v_sel<CPLX>(V, ldv, n, nbw, J, r0 + iperm, jp + 4 * (h + k) + g4);
#pragma unroll
                    for (int k = 0; k < RU; ++k)
                        mma_sub<CPLX>(vu[k], wp(h + k, 0), CPLX ? wp(h + k, NC - 1) : 0.0, zu);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (!rok[e] || r[e] < jp + nbw) continue;
                    x.re[e] = zu.re[e];
                    if constexpr (CPLX) x.im[e] = zu.im[e];
                    if (colok) st_elt<CPLX>(zc, r[e], zu.re[e], imag(zu, e));
                }
            }
            if (acc) {
#pragma unroll
                for (int h = 0; h < PT; h += RA) {
#pragma unroll
                    for (int t = 0; t < RA; ++t)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            va[t][e] = v_sel<CPLX>(V, ldv, n, nbw, J, r[e], jn + 16 * (h + t) + i16);
#pragma unroll
                    for (int t = 0; t < RA; ++t)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            mma_conj<CPLX>(va[t][e], x.re[e], imag(x, e), w[h + t]);
                }
            }
        }
    }
}

template <bool CPLX>
int b2f_validate(int64_t n, int nbw, int64_t nev, const void* V, int64_t ldv, const void* tau,
                 const void* Z, int64_t ldz, const void* work, size_t work_bytes)
{
    if (n < 0) return -1;
    if (nbw < 1) return -2;
    if (nev < 0 || nev > n) return -3;
    const int64_t J = b2f_reflectors(n, nbw);
    const bool active = J > 0 && nev > 0;
    if (active && !V) return -4;
    if (ldv < (n > 1 ? n : 1)) return -5;
    if (active && !tau) return -6;
    if (nev > 0 && n > 0 && !Z) return -7;
    if (ldz < (n > 1 ? n : 1)) return -8;
    if (work && ((uintptr_t)work % TRBT_WORK_ALIGN)) return -9;
    if (work_bytes && !work) return -9;
    return TRBT_SUCCESS;
}

size_t b2f_bytes(int64_t n, int nbw, bool cplx)
{
    const int64_t J = b2f_reflectors(n, nbw);
    if (J == 0) return 0;
    const size_t units = (size_t)(J + B2F_UNIT - 1) / B2F_UNIT;
    return B2F_HDR + units * B2F_UNIT * B2F_UNIT * (cplx ? 16 : 8);
}

template <bool CPLX>
int b2f_run(int64_t n, int nbw, int64_t nev, const double* V, int64_t ldv, const double* tau,
            double* Z, int64_t ldz, void* work, size_t work_bytes, void* stream_v)
{
    int rc = b2f_validate<CPLX>(n, nbw, nev, V, ldv, tau, Z, ldz, work, work_bytes);
    if (rc) return rc;
    const int64_t J = b2f_reflectors(n, nbw);
    if (J == 0 || nev == 0) return TRBT_SUCCESS;
    if (!work || work_bytes < b2f_bytes(n, nbw, CPLX)) return TRBT_ERR_WORKSPACE;
    rc = check_device();
    if (rc) return rc;
    hipStream_t st = (hipStream_t)stream_v;
    hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, st, (unsigned*)work, 64);
    double* Tw = (double*)((char*)work + B2F_HDR);
    int* steps = (int*)((char*)work + 32);
    using B = B2F<CPLX>;
    const unsigned P = (unsigned)b2f_panels<CPLX>(J), strips = (unsigned)((nev + 15) / 16);
    hipLaunchKernelGGL((k_b2f_gram<CPLX>), dim3(P, 4), dim3(64 * B2F_NW), 0, st, n, nbw, V, ldv, Tw);
    hipLaunchKernelGGL((k_b2f_tfac<CPLX>), dim3(P), dim3(64 * B::PT), 0, st, n, nbw, tau, Tw);
    // the pipeline addresses two panels of reflectors through a 32-bit range
    if ((2 * B::PW + 1) * ldv * 8 * B::NC < (int64_t)1 << 31)
        hipLaunchKernelGGL((k_b2f_apply<CPLX, true>), dim3(strips), dim3(64 * B2F_NW), 0, st, n, nbw,
                           nev, V, ldv, tau, (const double*)Tw, Z, ldz, steps);
    else
        hipLaunchKernelGGL((k_b2f_apply<CPLX, false>), dim3(strips), dim3(64 * B2F_NW), 0, st, n, nbw,
                           nev, V, ldv, tau, (const double*)Tw, Z, ldz, steps);
    return hipGetLastError() == hipSuccess ? TRBT_SUCCESS : TRBT_ERR_HIP;
}

// --------------------------------------------------------------------------
// Allocation-free variant (trans_ev_band_to_full_z_noalloc): the per-panel
// T factors go to a fixed array of device memory instead of a caller
// workspace.  Every device the library runs on holds its own copy of the
// array until the process ends; all calls on one device share it.  Host
// code never passes the array's name to a kernel (on the host it is only a
// stand-in for the symbol): it looks up the device address once per device
// and passes that.
// --------------------------------------------------------------------------
constexpr int B2F_MAX_DEVICES = 64;
std::mutex b2f_scratch_mu;
void* b2f_scratch_ptr[B2F_MAX_DEVICES];

}  // namespace

static_assert(TRBT_B2F_SCRATCH_BYTES % 256 == 0, "scratch size");
static __device__ __align__(256) unsigned char scratch[TRBT_B2F_SCRATCH_BYTES];

namespace {

// Device address of `scratch` on the current device (looked up on the first
// call on each device, with that device current).
int b2f_scratch(void** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return TRBT_ERR_HIP;
    if (dev < 0 || dev >= B2F_MAX_DEVICES) return TRBT_ERR_DEVICE;
    std::lock_guard<std::mutex> lock(b2f_scratch_mu);
    if (!b2f_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
            (void)hipGetLastError();
            return TRBT_ERR_HIP;
        }
        b2f_scratch_ptr[dev] = p;
    }
    *out = b2f_scratch_ptr[dev];
    return TRBT_SUCCESS;
}

}  // namespace

extern "C" {

int trbt_band_to_full_workspace_bytes(int64_t n, int nbw, int64_t nev, int is_complex,
                                      size_t* bytes)
{
    if (n < 0) return -1;
    if (nbw < 1) return -2;
    if (nev < 0 || nev > n) return -3;
    if (!bytes) return -4;
    *bytes = nev > 0 ? b2f_bytes(n, nbw, is_complex != 0) : 0;
    return TRBT_SUCCESS;
}

int trans_ev_band_to_full_d(int64_t n, int nbw, int64_t nev, const double* hh_v, int64_t ldv,
                            const double* hh_tau, double* Z, int64_t ldz, void* work,
                            size_t work_bytes, void* stream)
{
    return b2f_run<false>(n, nbw, nev, hh_v, ldv, hh_tau, Z, ldz, work, work_bytes, stream);
}

int trans_ev_band_to_full_z(int64_t n, int nbw, int64_t nev, const trbt_z* hh_v, int64_t ldv,
                            const trbt_z* hh_tau, trbt_z* Z, int64_t ldz, void* work,
                            size_t work_bytes, void* stream)
{
    return b2f_run<true>(n, nbw, nev, (const double*)hh_v, ldv, (const double*)hh_tau,
                         (double*)Z, ldz, work, work_bytes, stream);
}

int trans_ev_band_to_full_z_noalloc(int64_t n, int nbw, int64_t nev, const trbt_z* hh_v,
                                    int64_t ldv, const trbt_z* hh_tau, trbt_z* Z, int64_t ldz,
                                    void* stream)
{
    int rc = b2f_validate<true>(n, nbw, nev, hh_v, ldv, hh_tau, Z, ldz, nullptr, 0);
    if (rc) return rc;
    if (b2f_reflectors(n, nbw) == 0 || nev == 0) return TRBT_SUCCESS;
    if (b2f_bytes(n, nbw, true) > TRBT_B2F_SCRATCH_BYTES) return TRBT_ERR_SCRATCH;
    rc = check_device();
    if (rc) return rc;
    void* s = nullptr;
    rc = b2f_scratch(&s);
    if (rc) return rc;
    return b2f_run<true>(n, nbw, nev, (const double*)hh_v, ldv, (const double*)hh_tau,
                         (double*)Z, ldz, s, TRBT_B2F_SCRATCH_BYTES, stream);
}

}  // extern "C"
