// fw_paths_split.hpp -- Algorithm 1 with a replication's normals drawn by other wavefronts, for runs of
// few replications.
//
// fw_paths.hpp gives a replication one lane that draws and uses its normals; 64 replications are one
// wavefront, and a run of up to ~65,000 leaves most of the device's issue slots empty. Here a
// workgroup is 64 replications: one wavefront runs their paths as fw_paths.hpp does (a lane each), the
// other three (or seven) draw their normals, chunk by chunk, into the other of two LDS buffers. The draws
// are about four fifths of a replication's instructions, so they set the pace of three wavefronts about
// as the path does that of one; seven hide the latency of one another's chains where a SIMD has no other
// wavefront. Which wavefront runs the paths rotates with the workgroup, so that the SIMDs of a compute
// unit share them.
//
// What bounds it: the draws' issue and latency, then the path wavefront (its reads of the buffers are a
// tenth of its time). ms, a lane per replication -> split, 16,000 replications: d = N = 10, 1,000 iterations
// 4.7 -> 2.4; d = 16, N = 18, 500 5.7 -> 2.9; d = 20, N = 20, 400 6.6 -> 3.1; d = 27, N = 31, 200
// 7.7 -> 2.3 (seven drawing wavefronts from d = 7; three take 3.1). Binary64, 1,000 replications, 100
// iterations of d = N = 2: 0.15 -> 0.06.
//
// A chunk is a fixed number of units in stream order, across iterations. A unit is a group of samples
// that holds whole Philox blocks, or half of one where a group is long (D odd from 15 on: the block
// that straddles the halves is drawn for both). Sums, products and roundings are those of fw_paths.hpp: widths
// whose sums fuse with the Box-Muller product pass radius, cosine and sine instead of the product.
//
// The paths leave their outcome, hitting time and counts in memory; a second launch reduces them in
// the order of fw_paths.hpp's own reduction, so every result is the same bits.
#pragma once

#include "fw_paths.hpp"

namespace fw {

template <int D, int DRAW, typename Real>
struct SplitShape {
    static constexpr int kGroup = 4 / gcd_const(D, 4);                  // samples of whole blocks
    static constexpr int kGroupBlocks = kGroup * D / 4;
    static constexpr int kHalves = kGroup == 4 && kGroupBlocks > (sizeof(Real) == 8 ? 8 : 13) ? 2 : 1;
    static constexpr int kUnit = kGroup / kHalves;                      // samples of a unit
    static constexpr int first(int h) { return h * kUnit * D / 4; }     // its first block in the group
    static constexpr int blocks(int h) { return ((h + 1) * kUnit * D + 3) / 4 - first(h); }
    static constexpr int kBlocks = kHalves == 1 ? blocks(0) : (blocks(0) > blocks(1) ? blocks(0) : blocks(1));
    static constexpr bool kFused = kFuseSum<D>;
    static constexpr int kReals = kFused ? 6 : 4;                       // values of a block
    static constexpr int kTarget = sizeof(Real) == 8 ? 6 : DRAW > 3 ? 14 : kFused ? 10 : 12;   // blocks of a chunk, about
    static constexpr int kUnits = kBlocks > kTarget ? 1 : kTarget / kBlocks;   // units of a chunk
    static constexpr int kSlots = kUnits * kBlocks;
    static constexpr int kEach = (kSlots + DRAW - 1) / DRAW;            // slots of a drawing wavefront
    static constexpr int kBuffer = kSlots * kReals * 64;               // values of a chunk
};

// The path wavefront's side of the buffers. One barrier before each chunk.
template <int D, int DRAW, typename Real>
struct FedDraws {
    static constexpr bool kFed = true;
    static constexpr int kStride = 64;
    using Shape = SplitShape<D, DRAW, Real>;
    const Real *lane0;        // this lane's column of buffer 0
    int buf, pos;              // the current chunk's buffer and unit

    template <int H, class V>
    __device__ __forceinline__ void unit(uint32_t n, const V &v, V &s1, V &s2)
    {
        if (pos == Shape::kUnits) {
            __syncthreads();
            pos = 0;
            buf ^= 1;
        }
        const Real *u = lane0 + buf * Shape::kBuffer + pos * (Shape::kBlocks * Shape::kReals * 64);
        ++pos;
#pragma unroll
        for (int s = 0; s < Shape::kUnit; ++s) {
            if (s > 0 && static_cast<uint32_t>(s) >= n) break;
            Real z[D], rad[D], cs[D];
#pragma unroll
            for (int j = 0; j < D; ++j) {
                constexpr int kFirst = 4 * Shape::first(H);
                const int f = (H * Shape::kUnit + s) * D + j - kFirst, b = f / 4, c = f % 4;
                if constexpr (Shape::kFused) {
                    rad[j] = u[(b * 6 + c / 2 * 3) * 64];
                    cs[j] = u[(b * 6 + c / 2 * 3 + 1 + c % 2) * 64];
                    z[j] = rad[j] * cs[j];
                } else {
                    z[j] = u[(b * 4 + c) * 64];
                }
            }
            Real dot = Real(0);
#pragma unroll
            for (int j = 0; j < D; ++j) dot = fma(z[j], v[j], dot);
#pragma unroll
            for (int j = 0; j < D; ++j) {
#pragma clang fp contract(off)
                if (Shape::kFused && (kFuseRest<D> || n == static_cast<uint32_t>(Shape::kUnit))) s1[j] = fma(rad[j], cs[j], s1[j]);
                else s1[j] += z[j];
                s2[j] = fma(z[j], dot, s2[j]);
            }
        }
    }

    template <class V>
    __device__ __forceinline__ void samples(uint32_t N, const V &v, V &s1, V &s2)
    {
        for (uint32_t i = 0; i < N;) {
            unit<0>(min(N - i, static_cast<uint32_t>(Shape::kUnit)), v, s1, s2);
            i += Shape::kUnit;
            if constexpr (Shape::kHalves == 2) {
                if (i < N) unit<1>(min(N - i, static_cast<uint32_t>(Shape::kUnit)), v, s1, s2);
                i += Shape::kUnit;
            }
        }
    }
};

// Drawing wavefront w's side: its share of every chunk's slots, all their Philox chains side by side
// (w: a number, or an integral constant, which places the slots at compile time).
template <int D, int DRAW, typename Real, class Wave>
__device__ __forceinline__ void draw_chunks(const InstanceDesc *__restrict__ P, uint32_t r, Wave w, Real *lane0)
{
    using Shape = SplitShape<D, DRAW, Real>;
    constexpr int kEach = Shape::kEach;
    const uint32_t N = P->N, M = P->M, T = static_cast<uint32_t>(P->T);
    const uint32_t k0 = static_cast<uint32_t>(P->seed), k1 = static_cast<uint32_t>(P->seed >> 32);
    const uint32_t dom = P->instance & 0xFFFFFFu;
    const uint32_t units = (N + Shape::kUnit - 1) / Shape::kUnit;        // of an iteration
    const uint32_t n_last = N - (units - 1) * Shape::kUnit;             // samples of its last one
    const uint64_t chunks = (static_cast<uint64_t>(T) * units + Shape::kUnits - 1) / Shape::kUnits;
    uint32_t t0 = 0, u0 = 0;                                            // the chunk's first unit
    // this wavefront's slots: unit and block within it
    uint32_t in_unit[kEach], in_block[kEach];
    bool mine[kEach];
#pragma unroll
    for (int i = 0; i < kEach; ++i) {
        const uint32_t slot = w * kEach + i;
        mine[i] = slot < static_cast<uint32_t>(Shape::kSlots);
        in_unit[i] = mine[i] ? slot / Shape::kBlocks : i ? in_unit[i ? i - 1 : 0] : 0u;
        in_block[i] = slot % Shape::kBlocks;
    }
    Real *dst = lane0;
    for (uint64_t k = 0; k < chunks; ++k) {
        // each slot's block of the stream, its epoch, and whether a sample uses it
        uint32_t epoch[kEach], block[kEach];
        bool used[kEach], all = true;
        uint32_t t = t0, u = u0, at = 0;                // (t, u): the chunk's unit `at`
#pragma unroll
        for (int i = 0; i < kEach; ++i) {
            if (in_unit[i] != at) {
                u += in_unit[i] - at;
                at = in_unit[i];
                while (u >= units) {
                    u -= units;
                    ++t;
                }
            }
            const bool odd = Shape::kHalves == 2 && (u & 1u);
            const uint32_t first = odd ? Shape::first(Shape::kHalves - 1) : 0;
            uint32_t need = odd ? Shape::blocks(Shape::kHalves - 1) : Shape::blocks(0);
            if (u + 1 == units) need = (((odd ? Shape::kUnit : 0) + n_last) * D + 3) / 4 - first;
            epoch[i] = M == 1 ? t : t / M;
            block[i] = u / Shape::kHalves * Shape::kGroupBlocks + first + in_block[i];
            used[i] = mine[i] && t < T && in_block[i] < need;
            all = all && used[i];
        }
        PhiloxRow row[Shape::kUnits > 1 ? kEach : 1];
        Real q[kEach][6];
        auto draw = [&](int i) {
            const Words4 x = philox_block(row[Shape::kUnits > 1 ? i : 0], block[i], dom, k0, k1);
            const uint32_t xs[4] = {x.x0, x.x1, x.x2, x.x3};
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const float u1 = uniform_open01(xs[2 * e]), u2 = uniform_open01(xs[2 * e + 1]);
                if constexpr (sizeof(Real) == 8) {
                    q[i][3 * e] = sqrt(-2.0 * log(static_cast<double>(u1)));
                    sincospi(2.0 * static_cast<double>(u2), &q[i][3 * e + 2], &q[i][3 * e + 1]);
                } else {
                    q[i][3 * e] = __builtin_amdgcn_sqrtf(-__builtin_amdgcn_logf(u1));
                    q[i][3 * e + 1] = __builtin_amdgcn_cosf(u2);
                    q[i][3 * e + 2] = __builtin_amdgcn_sinf(u2);
                }
            }
        };
        auto put = [&](int i) {
            Real *o = dst + (w * kEach + i) * (Shape::kReals * 64);
            if constexpr (Shape::kFused) {
#pragma unroll
                for (int e = 0; e < 6; ++e) o[e * 64] = q[i][e];
            } else {
                o[0] = q[i][0] * q[i][1];
                o[64] = q[i][0] * q[i][2];
                o[128] = q[i][3] * q[i][4];
                o[192] = q[i][3] * q[i][5];
            }
        };
#pragma unroll
        for (int i = 0; i < kEach; ++i)
            if (Shape::kUnits > 1 || i == 0) row[Shape::kUnits > 1 ? i : 0] = philox_row(epoch[i], r, k0);
        if (all) {
#pragma unroll
            for (int i = 0; i < kEach; ++i) draw(i);
#pragma unroll
            for (int i = 0; i < kEach; ++i) put(i);
        } else {
#pragma unroll
            for (int i = 0; i < kEach; ++i)
                if (used[i]) {
                    draw(i);
                    put(i);
                }
        }
        u0 += Shape::kUnits;
        while (u0 >= units) {
            u0 -= units;
            ++t0;
        }
        dst = lane0 + (dst == lane0 ? Shape::kBuffer : 0);
        __syncthreads();
    }
}

// 64 replications per workgroup: a path wavefront and DRAW drawing ones.
template <int D, bool FEAT, int DRAW, typename Real>
__global__ __launch_bounds__(64 * (DRAW + 1)) void fw_paths_split_kernel(const InstanceDesc *__restrict__ P, RunBuffers B)
{
    constexpr bool kLds = !FEAT && D >= 7;
    using Shape = SplitShape<D, DRAW, Real>;
    __shared__ Real sm_z[2 * Shape::kBuffer];
    __shared__ uint64_t sm_feat[FEAT ? (D + 1) * 64 : 1];
    __shared__ uint32_t sm_sig[kLds ? (D + 1) * 64 : 1];
    __shared__ uint32_t sm_cnt[kLds ? (D + 1) * 64 : 1];
    const uint64_t R = P->R;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t role = __builtin_amdgcn_readfirstlane((threadIdx.x / 64 + blockIdx.x) & static_cast<uint32_t>(DRAW));
    const uint64_t r = static_cast<uint64_t>(blockIdx.x) * 64 + lane;
    const bool active = r < R;
    const uint32_t rc = static_cast<uint32_t>(active ? r : R - 1);
    if (role != 0) {
        if constexpr (DRAW == 3) {
            if (role == 1) draw_chunks<D, DRAW, Real>(P, rc, std::integral_constant<uint32_t, 0>{}, sm_z + lane);
            else if (role == 2) draw_chunks<D, DRAW, Real>(P, rc, std::integral_constant<uint32_t, 1>{}, sm_z + lane);
            else draw_chunks<D, DRAW, Real>(P, rc, std::integral_constant<uint32_t, 2>{}, sm_z + lane);
        } else {
            draw_chunks<D, DRAW, Real>(P, rc, role - 1, sm_z + lane);
        }
        return;
    }
    PathRec<D, uint32_t, kLds, 64> rec;
    if constexpr (kLds) {
        rec.s = sm_sig + lane;
        rec.c = sm_cnt + lane;
    }
    LaneResult res{0.0, kTauNone};
    run_path<D, true, Real, 0, uint32_t, FEAT, false>(P, B, rc, active, rec, res, sm_feat + lane,
                                                       FedDraws<D, DRAW, Real>{sm_z + lane, 1, Shape::kUnits});
    if (!active) return;
    B.rec_y[r] = res.y;
    B.rec_tau[r] = res.tau;
#pragma unroll
    for (int j = 0; j <= D; ++j) B.rec_cnt[static_cast<uint64_t>(j) * R + r] = rec.count(j);
    if (P->flags & 1u) {
#pragma unroll
        for (int j = 0; j < D; ++j) B.wsum[static_cast<uint64_t>(j) * R + r] = rec.sig(j);
    }
}

// The kernel of width d among LO .. HI.
template <int LO, int HI, bool FEAT, int DRAW, typename Real = float>
inline KernelFn choose_split(uint32_t d)
{
    if constexpr (LO > HI) {
        return nullptr;
    } else {
        if (d == static_cast<uint32_t>(LO)) return &fw_paths_split_kernel<LO, FEAT, DRAW, Real>;
        return choose_split<LO + 1, HI, FEAT, DRAW, Real>(d);
    }
}

// with 3 or 7 drawing wavefronts
KernelFn paths_split_narrow(uint32_t d, int draw);       // d <= 16
KernelFn paths_split_broad(uint32_t d, int draw);        // 17 <= d <= 32
KernelFn paths_split_features(uint32_t d);               // with features, d <= 32; 3
KernelFn paths_split_fp64(uint32_t d);                   // binary64, d <= 16; 3

}  // namespace fw
