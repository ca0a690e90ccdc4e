// sqn_slice.hpp -- a workgroup's slice of 64 feature quads and the sums over a slice, shared by the
// split forms of Algorithms 3-4 (fw_sqn_split.hip, fw_sqn_split_run.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "sqn.hpp"
#include "sqn_device.hpp"
#include "sqn_split.hpp"

namespace fw {
namespace {

constexpr uint32_t kSliceWords = 8;                      // bitmap words of a slice's 256 features
constexpr uint32_t kPairPerWave = kSqnMaxM / kSplitWaves;      // stored pairs a thread holds (8)

struct Slice {
    uint32_t s, rep, tid, ql, wv;    // slice, replication, thread, quad within the slice, wavefront
    uint32_t q, qc;                  // the quad, and the quad clamped into range (for loads)
    bool own, owner;                 // q < nq; own and in the first wavefront (stores)
};

__device__ __forceinline__ Slice slice_of(const SqnSplit &P)
{
    Slice c;
    c.s = blockIdx.x;
    c.rep = blockIdx.y;
    c.tid = threadIdx.x;
    c.ql = c.tid % kSplitQuads;
    c.wv = __builtin_amdgcn_readfirstlane(c.tid / kSplitQuads);
    c.q = c.s * kSplitQuads + c.ql;
    c.own = c.q < P.A.nq;
    c.owner = c.own && c.wv == 0;
    c.qc = c.own ? c.q : P.A.nq - 1;
    return c;
}

// v's slice (zero past n) into sv[256], by the first wavefront
__device__ __forceinline__ void stage_slice(const Slice &c, const double (&v)[4], double *sv)
{
    if (c.wv == 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) sv[4 * c.ql + e] = c.own ? v[e] : 0.0;
    }
}

// The sum over the rows of coef[i] times the quad's four bits: each wavefront sums a contiguous
// quarter of the rows in order, then every thread adds the four quarters in order (part: LDS
// [kSplitWaves][64][4]). Every thread of the workgroup must call it; it synchronises.
__device__ __forceinline__ void slice_bit_sum(const Slice &c, const uint32_t *bits, const double *coef, uint32_t count,
                                              double (*part)[kSplitQuads][4], double (&out)[4])
{
    const uint32_t per = (count + kSplitWaves - 1) / kSplitWaves;
    const uint32_t i0 = min(count, c.wv * per), i1 = min(count, i0 + per);
    const uint32_t wq = c.ql >> 3, sh = 4 * (c.ql & 7);
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    if (i0 < i1) add_bits(bits + i0 * kSliceWords + wq, kSliceWords, sh, coef + i0, i1 - i0, a);
#pragma unroll
    for (int e = 0; e < 4; ++e) part[c.wv][c.ql][e] = a[e];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        double t = part[0][c.ql][e];
        for (uint32_t u = 1; u < kSplitWaves; ++u) t += part[u][c.ql][e];
        out[e] = t;
    }
}

__device__ __forceinline__ double dot4(const double (&a)[4], const double (&b)[4])
{
    double p = 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) p += a[e] * b[e];
    return p;
}

}  // namespace
}  // namespace fw
