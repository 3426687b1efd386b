// trbt_stream.h -- the streaming form of the back-transformation (any nbw, no
// workspace), shared by the single-problem call, the batched plans and the
// real adjoint's checkpointing forward.  Defined in trbt_stream.hip.
#pragma once

#include <hip/hip_runtime.h>

#include <stdint.h>

// One problem for the streaming kernel; complex data as interleaved doubles,
// ldz in elements.  first: the problem's first workgroup in a launch over
// several problems (one workgroup per strip of 16 columns).
struct StreamProb {
    int64_t n, nev, ldz;
    const double* hv;
    const double* ht;
    double* Z;
    int64_t first;
    int64_t nbw;
};

// The kernel instance a band width takes: 0 .. STREAM_CLASSES-1.  Problems of
// one class can share a launch.
constexpr int STREAM_CLASSES = 28;
__attribute__((visibility("hidden"))) int stream_class(int64_t nbw);

inline int64_t stream_strips(int64_t nev) { return (nev + 15) / 16; }

// Z <- Q^* Z for one problem (K > 0, nev > 0).  ckpt: null, or (real only) the
// adjoint's checkpoints, the state of rows [sbot_t + 1, n) before every
// 16-stage block t: ckpt[(cb_t + r - sbot_t - 1) * nev + c], cb_t the rows of
// the blocks before t.  err: null, or a word set if a wait between the waves
// of a workgroup gives up (never expected; those columns of Z are then NaN).
__attribute__((visibility("hidden"))) hipError_t stream_single(const StreamProb& p, bool cplx,
                                                               double* ckpt, unsigned* err,
                                                               hipStream_t st);

// The same for `nprob` problems of one class (descriptors in device memory,
// `grid` strips in all).
__attribute__((visibility("hidden"))) hipError_t stream_batched(const StreamProb* probs, int nprob,
                                                                int64_t grid, int cls, bool cplx,
                                                                unsigned* err, hipStream_t st);
