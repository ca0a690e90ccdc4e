// fw_newsvendor_run.hip -- Algorithm 2 with one resource row, many iterations in one launch.
//
// The kernels of fw_newsvendor.hip take one launch per iteration: ~2.7 us of launch, then the loads
// of the quad, the previous step's reduction and the samples, 4.9 us in all up to 1e4 products. Here
// a cooperative launch runs iterations [t0, t1): a thread keeps its quad's coefficients and signature
// words in registers, the workgroups exchange their smallest ratio and its product in one tagged word
// (exchange.hpp), and the demand normals of the next epoch, which do not depend on the iterate, are
// drawn while the words travel. The parts of g'x only decide tau: they go to a log that one launch
// after the segment sums, an iteration per workgroup. The quads, their lanes, the workgroups and the
// order of every sum are those of the launch-per-iteration kernels, so the results are the same bits.
//
// What bounds an iteration is the exchange (1.6 us for 157 workgroups) and the chain of wavefront and
// workgroup reductions on either side of it, so those are kept short: the four counts of a quad travel
// over its lanes packed in one word, and the smallest ratio is an unsigned minimum of ordered keys (one
// instruction per step) followed by a ballot for its lane.
#include <hip/hip_runtime.h>

#include "device_rng.hpp"
#include "exchange.hpp"
#include "newsvendor.hpp"
#include "sim_types.hpp"
#include "wave_dpp.hpp"

namespace fw {

// NS: samples per lane held in registers, at least ceil(S / P)
template <int NS>
__global__ __launch_bounds__(kNvBlock) void nv_run_kernel(NvArgs A, NvRunArgs Q)
{
    __shared__ uint2 sm_key[kNvBlock / 64];             // (key, product) per wavefront: its products,
    __shared__ uint64_t st_key[kNvBlock / 64];          // and over the workgroups it polls
    __shared__ float sm_gx[kNvBlock / 64];
    // this workgroup's parts of g'x and, in workgroup 0, the vertices and their ratios, per iteration:
    // written out after the last one (a global store or atomic in the loop is waited for at its next
    // barrier: 1.6 us an iteration where workgroup 0 recorded as it went)
    __shared__ float log_gx[kRunSteps], log_best[kRunSteps];
    __shared__ uint32_t log_dec[kRunSteps];
    __shared__ uint32_t sm_fail;
    const uint32_t tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
    if (tid == 0) sm_fail = failure_get(Q.fail);
    __syncthreads();
    if (sm_fail) return;                                // an earlier launch of the run gave up
    const uint32_t r = blockIdx.y, g = blockIdx.x;
    const uint32_t P = A.P, sub = tid % P;
    const uint32_t q = g * (kNvBlock / P) + tid / P;
    const bool active = q < A.nq;
    const bool lead = sub == 0;                         // the lane that carries the quad after its counts are summed
    const uint32_t j0 = 4 * q;
    const uint32_t jc = 4 * (active ? q : A.nq - 1);    // a thread past the last quad loads the last and discards it

    const float4 mu4 = *reinterpret_cast<const float4 *>(A.mu_f + jc);
    const float4 isk4 = *reinterpret_cast<const float4 *>(A.isk_f + jc);
    const float4 a4 = *reinterpret_cast<const float4 *>(A.a_f + jc);
    const float4 b4 = *reinterpret_cast<const float4 *>(A.b_f + jc);
    const float4 ic4 = *reinterpret_cast<const float4 *>(A.ic_f + jc);
    const float4 xs4 = *reinterpret_cast<const float4 *>(A.xs_f + jc);
    uint64_t *sig = A.S_sig + static_cast<uint64_t>(r) * A.n + jc;
    const ulonglong2 s01 = reinterpret_cast<const ulonglong2 *>(sig)[0];
    const ulonglong2 s23 = reinterpret_cast<const ulonglong2 *>(sig)[1];
    uint64_t S4[4] = {s01.x, s01.y, s23.x, s23.y};
    float Sf[4];                                        // the signatures in binary32, by way of binary64
#pragma unroll
    for (int k = 0; k < 4; ++k) Sf[k] = static_cast<float>(static_cast<double>(S4[k]));
    const bool recorder = g == 0 && tid == 0;
    const float mu[4] = {mu4.x, mu4.y, mu4.z, mu4.w}, isk[4] = {isk4.x, isk4.y, isk4.z, isk4.w};
    const float ca[4] = {a4.x, a4.y, a4.z, a4.w}, cb[4] = {b4.x, b4.y, b4.z, b4.w};
    const float ic[4] = {ic4.x, ic4.y, ic4.z, ic4.w}, xs[4] = {xs4.x, xs4.y, xs4.z, xs4.w};

    // the quad's samples s = sub, sub + P, ... of an epoch; NaN past S counts nowhere
    float z[NS][4];
    auto draw = [&](uint32_t epoch) {
        const PhiloxRow row = philox_row(epoch, r, A.k0);
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            const uint32_t s = sub + i * P;
            Block4<float> b = normals_block_row(row, s * A.nq + q, A.dom, A.k0, A.k1);
#pragma unroll
            for (int k = 0; k < 4; ++k) z[i][k] = s < A.S ? b.z[k] : NAN;
        }
    };
    auto scale = [](uint64_t t) {
        return t == 0 ? 0.0f : static_cast<float>(2.0 / (static_cast<double>(t) * static_cast<double>(t + 1)));
    };
    uint32_t epoch = static_cast<uint32_t>(Q.t0 / Q.M), in_epoch = static_cast<uint32_t>(Q.t0 % Q.M);
    draw(epoch);
    float cw = scale(Q.t0);

    uint64_t *lines = Q.words + static_cast<size_t>(r) * A.nwg * kRunLine;    // this replication's slots

    for (uint64_t t = Q.t0; t < Q.t1; ++t) {
        float x[4], thr[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) x[k] = xs[k] * (Sf[k] * cw);
        if (t == 0 && Q.from_x0) {
            const float4 x04 = *reinterpret_cast<const float4 *>(A.x0_f + jc);
            x[0] = x04.x, x[1] = x04.y, x[2] = x04.z, x[3] = x04.w;
        }
        uint32_t packed = 0u;       // the four counts, eight bits each (at most S <= 255)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            // sigma_j = 0 stores an infinite scale: the threshold is then +-infinity, and +infinity
            // (every sample counted) where x_j equals the demand exactly
            thr[k] = (x[k] - mu[k]) * isk[k];
            if (thr[k] != thr[k]) thr[k] = INFINITY;
#pragma unroll
            for (int i = 0; i < NS; ++i) packed += (z[i][k] <= thr[k]) ? 1u << (8 * k) : 0u;
        }
        packed = dpp_sum_lanes(packed, P);
        float rmin = INFINITY, gx = 0.0f;
        uint32_t jmin = 0xFFFFFFFFu;
        if (active && lead) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float gj = ca[k] + cb[k] * static_cast<float>((packed >> (8 * k)) & 0xFFu);
                const float rj = gj * ic[k];
                if (rj < rmin) {
                    rmin = rj;
                    jmin = j0 + k;
                }
                gx = fmaf(gj, x[k], gx);
            }
        }
        uint32_t key = value_key(rmin);
        wave_min_key<true>(key, jmin);
        gx = dpp_sum64(gx);
        if (lane == 0) {
            sm_key[wave] = make_uint2(key, jmin);
            sm_gx[wave] = gx;
        }
        __syncthreads();
        if (tid == 0) {   // the wavefronts cover ascending product ranges: strict < keeps the lowest index
            uint2 m = sm_key[0];
            float gs = sm_gx[0];
#pragma unroll
            for (int w = 1; w < kNvBlock / 64; ++w) {
                if (sm_key[w].x < m.x) m = sm_key[w];
                gs += sm_gx[w];
            }
            vertex_put(lines, g, t, m.x, m.y);
            log_gx[t - Q.t0] = gs;
        }

        // while the words travel: the next iteration's normals and scale
        if (++in_epoch == Q.M) {
            in_epoch = 0;
            ++epoch;
            if (t + 1 < Q.t1) draw(epoch);
        }
        cw = scale(t + 1);

        // the vertex over the workgroups: the smallest ratio, the lowest product among equal ones
        const uint64_t m = vertex_get<kNvBlock>(lines, A.nwg, t, st_key, &sm_fail);
        if (sm_fail) {
            if (tid == 0) failure_raise(Q.fail);
            return;
        }
        const float best = key_value(static_cast<uint32_t>(m >> 32));
        const uint32_t a = (best < 0.0f) ? static_cast<uint32_t>(m) + 1u : 0u;
        if (recorder) {
            log_best[t - Q.t0] = best;
            log_dec[t - Q.t0] = a;
        }
        const uint32_t hit = a - 1u - j0;               // 0..3: the chosen product is in this quad
        if (hit < 4u) {
            const uint64_t add = t + 1;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                S4[k] += hit == static_cast<uint32_t>(k) ? add : 0;
                Sf[k] = static_cast<float>(static_cast<double>(S4[k]));
            }
        }
    }
    __syncthreads();
    for (uint32_t i = tid; i < Q.t1 - Q.t0; i += kNvBlock) {
        Q.gx_log[(i * A.R + r) * A.nwg + g] = log_gx[i];
        if (g == 0) {
            Q.best_log[i * A.R + r] = log_best[i];
            A.dec[static_cast<uint64_t>(r) * A.T + Q.t0 + i] = log_dec[i];
        }
    }
    if (active && lead) {
        reinterpret_cast<ulonglong2 *>(sig)[0] = make_ulonglong2(S4[0], S4[1]);
        reinterpret_cast<ulonglong2 *>(sig)[1] = make_ulonglong2(S4[2], S4[3]);
    }
}

namespace {

const void *nv_run_fn(uint32_t ns)
{
    if (ns <= 2) return reinterpret_cast<const void *>(&nv_run_kernel<2>);
    if (ns <= 4) return reinterpret_cast<const void *>(&nv_run_kernel<4>);
    if (ns <= 8) return reinterpret_cast<const void *>(&nv_run_kernel<8>);
    return reinterpret_cast<const void *>(&nv_run_kernel<kNvRunMaxNs>);
}

}  // namespace

bool nv_run_fits(uint32_t nwg, uint32_t R, uint32_t S, uint32_t P, int device)
{
    if ((S + P - 1) / P > kNvRunMaxNs || S > 255) return false;   // the counts travel in eight bits
    int cus = 0, coop = 0, per_cu = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess ||
        hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, device) != hipSuccess || !coop ||
        static_cast<uint64_t>(nwg) * R > 2ull * static_cast<uint64_t>(cus))
        return false;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, nv_run_fn((S + P - 1) / P), kNvBlock, 0) == hipSuccess &&
           per_cu >= 2;
}

int launch_nv_run(const NvArgs &A, const NvRunArgs &Q, hipStream_t s)
{
    NvArgs a = A;
    NvRunArgs q = Q;
    void *args[] = {&a, &q};
    if (int rc = launch_cooperative(nv_run_fn((A.S + A.P - 1) / A.P), dim3(A.nwg, A.R), kNvBlock, args, 0, s)) return rc;
    const RunLog L{Q.gx_log, Q.best_log, A.nwg, A.R, A.n, A.C, A.gap_eps, Q.t0, A.T, Q.fail, A.dec, A.tau, A.cnt};
    return launch_run_log(L, Q.t1 - Q.t0, s);
}

}  // namespace fw
