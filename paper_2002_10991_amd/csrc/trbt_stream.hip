// trbt_stream.hip -- streaming form of the tridiagonal-to-banded eigenvector
// back-transformation on gfx950: one reflector at a time, any nbw, no
// workspace (the blocked form of trbt_device.h needs packed factors and a
// band width that is a multiple of 16).
//
// One workgroup per strip of 16 columns; its waves hold consecutive slots j
// (sweeps) and run them as a pipeline, wave w the slots j = w (mod NW).  Rows
// are cut into quads of 4 (rows 4Q .. 4Q+3).  Lane (c, g) = (lane % 16,
// lane / 16) holds row 4Q+g of column c of every quad in the slot's window, so
// a quad is one register per lane and a row keeps its lane while the window
// slides: in the four stages whose first row r0 = 4Q+d, d = 3 .. 0, lies in
// quad Q, register i of lane group g meets entry 4i+g-d of the reflector.
// After the four stages the bottom quad leaves and every register moves
// down by one (the last stage writes its update there), and the next
// quad enters on top.
//
// Order: reflector (s, j) needs (s+1, j) and (s+1, j-1).  Slot j walks its
// stages downwards, and a quad passes from slot j-1 to slot j only once slot
// j-1 has run every stage that touches any of its rows, so all of a row's
// earlier reflectors have been applied when slot j meets it.  Quads pass between
// waves through a ring in LDS, and from the last wave to the first (the
// next round of slots) through Z.
//
// Per four stages a wave loads the four reflectors (coalesced, one step ahead
// in registers) and lays them out in LDS with zeros around them, so the inner
// loops have no bounds.  A row outside the reflector takes no part, whatever
// it holds (an infinity or a NaN times a zero would spread): the first
// quad and those from LO on are masked; between them every row is inside,
// except in the slot's first stages, where the reflector is shorter (EDGE).
//
// What bounds it: instruction issue of the waves of one CU, and below that the
// chain of one slot's stages (a dot product, a sum over the four lane groups, an
// update).  A stage is about 125 instructions at complex nbw = 20, 48 of them
// the reflector's FMAs; a slot starts RL steps behind the one before it.
// Complex n = 1201, nbw = 20, nev = 401: 2.7 ms, 1280 steps in a row on each
// workgroup's first wave at 2.1 us with two waves per SIMD (one lane per column
// and a reflector's rows from memory, the form before: 265 ms); real n = 64,
// nbw = 8, nev = 16: 25 us a call (549 us).

#include <hip/hip_runtime.h>

#include <stdint.h>

#include "trbt_device.h"
#include "trbt_lanes.h"
#include "trbt_stream.h"

namespace {

constexpr int SR = 4;   // quads in a ring between two waves

template <int RL, int NW, bool CPLX>
struct StreamLds {
    static constexpr int E = CPLX ? 2 : 1;
    int written[NW], consumed[NW];
    int failed;
    double ring[NW > 1 ? NW - 1 : 1][SR][64 * E];
    double v[NW][4][4 * RL * E];   // the four reflectors of a step, entry x - d at x
    double tau[NW][4][E];
};

template <bool CPLX>
struct Val {
    double re;
};
template <>
struct Val<true> {
    double re, im;
};

template <bool CPLX>
__device__ inline Val<CPLX> val_zero()
{
    Val<CPLX> v;
    v.re = 0.0;
    if constexpr (CPLX) v.im = 0.0;
    return v;
}

template <bool CPLX>
__device__ inline Val<CPLX> val_ld(const double* p)
{
    Val<CPLX> v;
    v.re = p[0];
    if constexpr (CPLX) v.im = p[1];
    return v;
}

template <bool CPLX>
__device__ inline void val_st(double* p, Val<CPLX> v)
{
    p[0] = v.re;
    if constexpr (CPLX) p[1] = v.im;
}

// Global memory, said so to the compiler: the pointers come out of a table, and
// a generic (flat) load would count as an LDS operation too, so that
// every wait for LDS would wait for the loads made ahead.
typedef __attribute__((address_space(1))) double gdouble;

template <bool CPLX>
__device__ inline Val<CPLX> glb_ld(const double* p)
{
    const gdouble* q = (const gdouble*)p;
    Val<CPLX> v;
    v.re = q[0];
    if constexpr (CPLX) v.im = q[1];
    return v;
}

template <bool CPLX>
__device__ inline void glb_st(double* p, Val<CPLX> v)
{
    gdouble* q = (gdouble*)p;
    q[0] = v.re;
    if constexpr (CPLX) q[1] = v.im;
}

template <bool CPLX>
__device__ inline Val<CPLX> val_sel(bool c, Val<CPLX> a, Val<CPLX> b)
{
    Val<CPLX> v;
    v.re = c ? a.re : b.re;
    if constexpr (CPLX) v.im = c ? a.im : b.im;
    return v;
}

// Wait until ctr >= need (a counter in LDS that only grows; `seen` the last
// value read).  Bounded: false on the never-expected time-out.
__device__ inline bool stream_wait(int* ctr, int need, int& seen)
{
    wait_jitter(need, need);
    if (seen >= need) return true;
    int v;
#pragma unroll 1
    for (unsigned spins = 0;; ++spins) {
        v = __builtin_amdgcn_readfirstlane(
            __hip_atomic_load(ctr, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP));
        if (v >= need) break;
        if (spins > 16) __builtin_amdgcn_s_sleep(1);
        if (spins > (1u << 26)) return false;
    }
    seen = v;
    return true;
}

// One stage, r0 = 4q + d: reflector vl (LDS, entry e at position e + d), on
// the quads z[0 .. RL-1].  SHIFT: the update moves every quad down by one
// register, out takes the last (z[0] is then free).  The same operations in
// the same order in every form: a masked row adds a zero.
template <int LO, int RL, bool CPLX, bool SHIFT, bool EDGE>
__device__ inline void stream_stage(Val<CPLX> (&z)[RL], Val<CPLX>& out, const double* vl,
                                    const double* taul, int len, int gd)
{
    constexpr int E = CPLX ? 2 : 1;
    auto masked = [&](int i) { return EDGE || (i == 0 && !SHIFT) || i >= LO; };
    auto inside = [&](int i) { return (unsigned)(4 * i + gd) < (unsigned)len; };
    // the reflector stays in registers between its two uses where it fits
    constexpr bool KEEP = RL <= (CPLX ? 34 : 60);
    Val<CPLX> vk[KEEP ? RL : 1];
    if constexpr (KEEP) {
#pragma unroll
        for (int i = 0; i < RL; ++i) vk[i] = val_ld<CPLX>(vl + 4 * i * E);
    }
    auto vget = [&](int i) {
        if constexpr (KEEP) return vk[i];
        else return val_ld<CPLX>(vl + 4 * i * E);
    };
    const Val<CPLX> tau = val_ld<CPLX>(taul);
    Val<CPLX> s[2] = {val_zero<CPLX>(), val_zero<CPLX>()};
#pragma unroll
    for (int i = 0; i < RL; ++i) {
        const Val<CPLX> x = masked(i) ? val_sel(inside(i), z[i], val_zero<CPLX>()) : z[i];
        const Val<CPLX> v = vget(i);
        Val<CPLX>& a = s[i & 1];
        a.re = fma(v.re, x.re, a.re);
        if constexpr (CPLX) {   // conj(v) x
            a.re = fma(v.im, x.im, a.re);
            a.im = fma(v.re, x.im, a.im);
            a.im = fma(-v.im, x.re, a.im);
        }
    }
    if constexpr (!KEEP) asm volatile("" ::: "memory");
    Val<CPLX> a;
    const double dr = swap_add<32>(swap_add<16>(s[0].re + s[1].re));
    if constexpr (CPLX) {
        const double di = swap_add<32>(swap_add<16>(s[0].im + s[1].im));
        a.re = fma(tau.re, dr, -(tau.im * di));
        a.im = fma(tau.re, di, tau.im * dr);
    } else {
        a.re = tau.re * dr;
    }
#pragma unroll
    for (int i = RL - 1; i >= 0; --i) {
        const Val<CPLX> v = vget(i);
        Val<CPLX> x = z[i];
        x.re = fma(-a.re, v.re, x.re);
        if constexpr (CPLX) {
            x.re = fma(a.im, v.im, x.re);
            x.im = fma(-a.re, v.im, x.im);
            x.im = fma(-a.im, v.re, x.im);
        }
        if (masked(i)) x = val_sel(inside(i), x, z[i]);
        if constexpr (SHIFT) {
            if (i == RL - 1) out = x;
            else z[i + 1] = x;
        } else {
            z[i] = x;
        }
    }
}

template <int LO, int RL, int NW, bool CPLX, bool CKPT>
__device__ inline bool stream_strip(const StreamProb& P, int64_t strip, double* __restrict__ ckpt,
                                    StreamLds<RL, NW, CPLX>& S)
{
    constexpr int E = CPLX ? 2 : 1;
    constexpr int NV = (4 * RL + 15) / 16;   // loads per lane of a step's reflectors
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, g = lane >> 4;
    const int n = (int)P.n, b = (int)P.nbw;
    const int64_t col = strip * 16 + c;
    const bool colok = col < P.nev;
    double* __restrict__ zc = P.Z + (colok ? col : 0) * P.ldz * E;
    const int J = (int)sweeps_in_stage(n, b, 0);
    const int qmax = (n - 1) / 4;
    const int64_t ktot = ceil_sum(n - 2, b);
    int xput = 0, xget = 0, seen_in = 0, seen_out = 0;
    double* const vw = &S.v[w][0][0];
    double* const tw = &S.tau[w][0][0];

    auto z_load = [&](int q) {
        const int r = 4 * q + g;
        return glb_ld<CPLX>(zc + (int64_t)(r < n ? r : n - 1) * E);   // masked where it is used
    };
    auto z_store = [&](int q, Val<CPLX> v) {
        const int r = 4 * q + g;
        if (colok && r < n) glb_st<CPLX>(zc + (int64_t)r * E, v);
    };

    for (int j = w; j < J; j += NW) {
        const int rmin = 1 + j * b;             // first row of the slot's last stage
        const int qlast = rmin / 4;
        const int qhand = j + 1 < J ? (rmin + b) / 4 : qmax + 1;   // quads from here on go to slot j+1
        Val<CPLX> z[RL];
#pragma unroll
        for (int i = 0; i < RL; ++i) z[i] = val_zero<CPLX>();

        // Reflectors: lane group d = g loads the one of row r0 = 4q + d, stage
        // s = r0 - 1 - j b, index k = ktot - ceil_sum(M) + j with M = n-2-s (a
        // quotient mq and a remainder mr of b).  The next step's stage is 4
        // lower: M + 4, and k less the sweeps of the stages s-1 .. s-4,
        // sum of ceil((M+i)/b), i = 1 .. 4.
        int M = n - 1 - (4 * qmax + g) + j * b;
        int mq = 0, mr = 0;
        int64_t k = 0;
        auto locate = [&]() {
            if (M < 0) return;   // no stage of this lane's group yet
            mq = M / b;
            mr = M - mq * b;
            k = ktot - ((int64_t)b * mq * (mq + 1) / 2 + (int64_t)mr * (mq + 1)) + j;
        };
        locate();
        Val<CPLX> pv[NV], pt;
        auto v_load = [&](int q) {   // the reflectors of step q, into pv, pt
            const double* hk = P.hv + (k * b - g) * E;
            if (4 * q >= rmin && 4 * q + 3 + b <= n) {
                // whole reflectors: entries outside 0 .. b-1 are read from the
                // nearest inside and dropped where they go to LDS
                pt = glb_ld<CPLX>(P.ht + k * E);
#pragma unroll
                for (int t = 0; t < NV; ++t) {
                    const int x = c + 16 * t;
                    pv[t] = glb_ld<CPLX>(hk + (x < g ? g : x < g + b ? x : g + b - 1) * E);
                }
            } else {
                const int r0 = 4 * q + g;
                const bool ok = r0 >= rmin && r0 <= n - 2;
                const int len = n - r0 < b ? n - r0 : b;
                pt = ok ? glb_ld<CPLX>(P.ht + k * E) : val_zero<CPLX>();
#pragma unroll
                for (int t = 0; t < NV; ++t) {
                    const int x = c + 16 * t;
                    pv[t] = ok && x >= g && x < g + len ? glb_ld<CPLX>(hk + x * E)
                                                        : val_zero<CPLX>();
                }
            }
            // to the next step
            const int up = mr + 4;
            k -= 4 * mq + 4 + (up > b ? up - b : 0) + (up > 2 * b ? up - 2 * b : 0);
            M += 4;
            mr = up;
            while (mr >= b) {
                mr -= b;
                ++mq;
            }
            if (M < 4) locate();   // this lane group's first stage
        };
        // a quad that leaves the window
        auto put = [&](int q, Val<CPLX> v) -> bool {
            if (q > qmax) return true;
            if (q < qhand || w == NW - 1) {
                z_store(q, v);
                if (q < qhand) return true;
            } else {
                if (!stream_wait(&S.consumed[w], xput - SR + 1, seen_out)) return false;
                double* p = &S.ring[w][xput % SR][0];
                p[lane] = v.re;
                if constexpr (CPLX) p[64 + lane] = v.im;
            }
            ++xput;
            __hip_atomic_store(&S.written[w], xput, __ATOMIC_RELEASE,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
            return true;
        };

        // Wave 0 reads its quads from Z, one step ahead: slot 0 as they are,
        // later slots once the last wave has stored them.
        const bool fromz = w == 0;
        Val<CPLX> znext = val_zero<CPLX>();
        auto z_next = [&](int q) -> bool {
            if (j > 0 && !stream_wait(&S.written[NW - 1], ++xget, seen_in)) return false;
            znext = z_load(q);
            return true;
        };
        v_load(qmax);
        if (fromz && !z_next(qmax)) return false;
        for (int q = qmax; q >= qlast; --q) {
            // the step's reflectors to LDS (this wave's own area: its LDS
            // operations complete in order), the next step's from memory
#pragma unroll
            for (int t = 0; t < NV; ++t)
                if (16 * (t + 1) <= 4 * RL || c + 16 * t < 4 * RL)
                    val_st<CPLX>(vw + (g * 4 * RL + c + 16 * t) * E,
                                 val_sel((unsigned)(c + 16 * t - g) < (unsigned)b, pv[t],
                                         val_zero<CPLX>()));
            if (c == 0) val_st<CPLX>(tw + g * E, pt);
            z[0] = val_sel(colok && 4 * q + g < n, znext, val_zero<CPLX>());
            if (q > qlast) {
                v_load(q - 1);
                if (fromz && !z_next(q - 1)) return false;
            }
            if (!fromz) {   // the quad that enters, from the ring
                if (!stream_wait(&S.written[w - 1], xget + 1, seen_in)) return false;
                const double* p = &S.ring[w - 1][xget % SR][0];
                z[0].re = p[lane];
                if constexpr (CPLX) z[0].im = p[64 + lane];
                ++xget;
                __hip_atomic_store(&S.consumed[w - 1], xget, __ATOMIC_RELEASE,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            if constexpr (CKPT) {
                if (j == 0) {   // rows still as they came: row r opens block (n-2-r)/16
                    const int r = 4 * q + g;
                    const int64_t t = r < n - 1 ? (n - 2 - r) / 16 : 0;
                    const int64_t sbot = n - 18 - 16 * t > 0 ? n - 18 - 16 * t : 0;
                    if (colok && r >= 1 && r < n)
                        glb_st<CPLX>(ckpt + ((17 * t + 8 * t * (t - 1) + r - sbot - 1) * P.nev +
                                             col) * E, z[0]);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

            Val<CPLX> out = val_zero<CPLX>();
            // checkpoint: before stage n-3-16t, right after the one above it
            auto save = [&](int r0) {
                const int s = r0 - 1 - j * b, up = n - 3 - s;
                if (up % 16 != 15 || s < 1) return;
                const int64_t t = up / 16 + 1;
                const int64_t sbot = n - 18 - 16 * t > 0 ? n - 18 - 16 * t : 0;
                const int len = n - r0 < b ? n - r0 : b, d = r0 - 4 * q;
#pragma unroll
                for (int i = 0; i < RL; ++i) {
                    const int e = 4 * i + g - d;
                    if (colok && e >= 0 && e < len)
                        glb_st<CPLX>(ckpt + ((17 * t + 8 * t * (t - 1) + r0 + e - sbot - 1) *
                                                 P.nev + col) * E, z[i]);
                }
            };
            constexpr int VS = 4 * RL * E;
            if (!CKPT && 4 * q >= rmin && 4 * q + 3 + b <= n) {   // four whole stages
#pragma unroll 1
                for (int d = 3; d > 0; --d)
                    stream_stage<LO, RL, CPLX, false, false>(z, out, vw + d * VS + g * E,
                                                             tw + d * E, b, g - d);
                stream_stage<LO, RL, CPLX, true, false>(z, out, vw + g * E, tw, b, g);
            } else {
#pragma unroll 1
                for (int d = 3; d >= 0; --d) {
                    const int r0 = 4 * q + d;
                    if (r0 < rmin) break;
                    if (r0 <= n - 2)
                        stream_stage<LO, RL, CPLX, false, true>(z, out, vw + d * VS + g * E,
                                                                tw + d * E,
                                                                n - r0 < b ? n - r0 : b, g - d);
                    if constexpr (CKPT) {
                        if (r0 < n) save(r0);
                    }
                }
                out = z[RL - 1];
#pragma unroll
                for (int i = RL - 1; i > 0; --i) z[i] = z[i - 1];
            }
            if (!put(q + RL - 1, out)) return false;
        }
        // the window after the last stage: quad qlast + i in z[i+1]
#pragma unroll
        for (int i = RL - 2; i >= 0; --i)
            if (!put(qlast + i, z[i + 1])) return false;
    }
    return true;
}

template <int LO, int RL, int NW, bool CPLX, bool CKPT>
__global__ __launch_bounds__(64 * NW) void k_stream(StreamProb one,
                                                    const StreamProb* __restrict__ probs, int nprob,
                                                    double* __restrict__ ckpt,
                                                    unsigned* __restrict__ err)
{
    __shared__ StreamLds<RL, NW, CPLX> S;
    StreamProb P = one;
    int64_t strip = blockIdx.x;
    if (probs) {
        int lo = 0, hi = nprob;   // largest p with probs[p].first <= blockIdx.x
        while (hi - lo > 1) {
            const int mid = (lo + hi) / 2;
            if (probs[mid].first <= (int64_t)blockIdx.x) lo = mid;
            else hi = mid;
        }
        P = probs[lo];
        strip -= P.first;
    }
    if (threadIdx.x < NW) S.written[threadIdx.x] = S.consumed[threadIdx.x] = 0;
    if (threadIdx.x == 0) S.failed = 0;
    __syncthreads();
    if (!stream_strip<LO, RL, NW, CPLX, CKPT>(P, strip, ckpt, S)) S.failed = 1;
    __syncthreads();
    if (S.failed) {   // never expected
        if (err && threadIdx.x == 0) atomicOr(err, 1u);
        constexpr int E = CPLX ? 2 : 1;
        for (int64_t c = strip * 16; c < strip * 16 + 16 && c < P.nev; ++c)
            for (int64_t x = threadIdx.x; x < P.n * E; x += 64 * NW)
                P.Z[c * P.ldz * E + x] = __builtin_nan("");
    }
}

struct StreamArgs {
    StreamProb one;
    const StreamProb* probs;
    int nprob;
    int64_t grid;
    double* ckpt;
    unsigned* err;
    hipStream_t st;
};

// Waves per workgroup: as many as the registers of a lane allow (about 7 RL + 44
// real, 13 RL + 62 complex, the window and a reflector among them; a
// small spill, up to 250 bytes for complex nbw < 72, costs less than half the
// waves).
template <int LO, int RL, bool CPLX>
hipError_t stream_launch(const StreamArgs& a)
{
    constexpr int NW = RL <= (CPLX ? 5 : 12) ? 16 : RL <= (CPLX ? 19 : 30) ? 8 : 4;
    if constexpr (!CPLX) {
        if (a.ckpt) {
            hipLaunchKernelGGL((k_stream<LO, RL, NW, CPLX, true>), dim3((unsigned)a.grid),
                               dim3(64 * NW), 0, a.st, a.one, a.probs, a.nprob, a.ckpt, a.err);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((k_stream<LO, RL, NW, CPLX, false>), dim3((unsigned)a.grid), dim3(64 * NW), 0,
                       a.st, a.one, a.probs, a.nprob, a.ckpt, a.err);
    return hipGetLastError();
}

// Instances.  nbw < 40: one per nbw / 4 and per whether nbw % 4 needs one quad
// more (the window's quads, RL = (nbw + 2) / 4 + 1, are exact there: every
// quad more is a step's delay for each slot after it).  Beyond that one
// for every 8, then for every 32 and 64 of nbw, masked from the narrowest on.
template <bool CPLX>
hipError_t stream_dispatch(int cls, const StreamArgs& a)
{
    switch (cls) {
#define TRBT_STREAM(L)                                                                             \
    case 2 * L: return stream_launch<L, L + 1, CPLX>(a);                                           \
    case 2 * L + 1: return stream_launch<L, L + 2, CPLX>(a);
        case 1: return stream_launch<0, 2, CPLX>(a);
        TRBT_STREAM(1)
        TRBT_STREAM(2)
        TRBT_STREAM(3)
        TRBT_STREAM(4)
        TRBT_STREAM(5)
        TRBT_STREAM(6)
        TRBT_STREAM(7)
        TRBT_STREAM(8)
        TRBT_STREAM(9)
#undef TRBT_STREAM
        case 20: return stream_launch<10, 13, CPLX>(a);
        case 21: return stream_launch<12, 15, CPLX>(a);
        case 22: return stream_launch<14, 17, CPLX>(a);
        case 23: return stream_launch<16, 19, CPLX>(a);
        case 24: return stream_launch<18, 26, CPLX>(a);
        case 25: return stream_launch<25, 34, CPLX>(a);
        case 26: return stream_launch<33, 50, CPLX>(a);
        case 27: return stream_launch<49, 66, CPLX>(a);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

int stream_class(int64_t nbw)
{
    if (nbw < 40) return (int)(2 * (nbw / 4) + (nbw % 4 >= 2));
    if (nbw < 72) return (int)(20 + (nbw - 40) / 8);
    return nbw < 100 ? 24 : nbw < 132 ? 25 : nbw < 196 ? 26 : 27;
}

hipError_t stream_single(const StreamProb& p, bool cplx, double* ckpt, unsigned* err,
                         hipStream_t st)
{
    const StreamArgs a{p, nullptr, 0, stream_strips(p.nev), ckpt, err, st};
    return cplx ? stream_dispatch<true>(stream_class(p.nbw), a)
                : stream_dispatch<false>(stream_class(p.nbw), a);
}

hipError_t stream_batched(const StreamProb* probs, int nprob, int64_t grid, int cls, bool cplx,
                          unsigned* err, hipStream_t st)
{
    const StreamArgs a{StreamProb{}, probs, nprob, grid, nullptr, err, st};
    return cplx ? stream_dispatch<true>(cls, a) : stream_dispatch<false>(cls, a);
}
