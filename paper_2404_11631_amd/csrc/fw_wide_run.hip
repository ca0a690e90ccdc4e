// fw_wide_run.hip -- Algorithm 1 at the paper's experimental shape, many iterations in one launch.
//
// The kernels of fw_wide.hip take three dependent launches per iteration, 11.8 us up to d = 5e4 with
// ~1 us of arithmetic in it. Here a cooperative launch runs iterations [t0, t1): the 256 threads of a
// unit keep its 128 assets' signature words, coefficients and normals in registers, and an iteration
// exchanges tagged words (exchange.hpp):
//   dots      each half wavefront publishes its samples' z_i'v over the unit's assets as soon as it has
//             them. Up to kWideDirectUnits units, every unit reads all units' words of the items it
//             needs (a half wavefront its own chunk's) and sums them itself: one exchange, but
//             (N + 1) units^2 words. Above that, a wavefront per item reads the units' words, sums them
//             and publishes the result, which every unit then reads: two exchanges, 2 (N + 1) units
//             words (an iteration at 79 units, N = 25: 5.8 us with one exchange, 4.3 us with two; 24 units: 4.1 us with one). Both sum in the
//             dot kernel's order;
//   vertex    the workgroups' smallest gradient entries, as in the newsvendor run. The next epoch's
//             normals, which do not depend on the iterate, are drawn while those words travel.
// A unit is a workgroup. The parts of g'w only decide tau: they go to a log summed after the launch.
// The assets, samples and the order of every sum are those of the launch-per-iteration kernels, so the
// results are the same bits.
#include <hip/hip_runtime.h>

#include "device_rng.hpp"
#include "exchange.hpp"
#include "sim_types.hpp"
#include "wave_dpp.hpp"
#include "wide.hpp"

namespace fw {

namespace {

// The dot kernel's sum over the units: its thread i has x_i = the values of units i, i + 256, ... in
// order, and its tree halves 256 of them down: 128 and 64 apart, then (here over lanes) 32, 16, 8, 4, 2
// and 1 apart. Each step leaves the partners equal, so a rotation within the 16 lanes of a row
// reaches the partner of the steps below 16. Every lane gets the sum.
__device__ __forceinline__ float dot_tree16(float s)
{
    const auto h = __builtin_amdgcn_permlane16_swap(__float_as_uint(s), __float_as_uint(s), false, false);
    s = __uint_as_float(h[0]) + __uint_as_float(h[1]);
    s += dpp_move<0x128>(s);
    s += dpp_move<0x124>(s);
    s += dpp_move<0x122>(s);
    s += dpp_move<0x121>(s);
    return s;
}

// lane l of the wavefront with x_l, x_{l+64}, x_{l+128}, x_{l+192}
__device__ __forceinline__ float dot_tree(const float (&x)[4])
{
    const float s = (x[0] + x[2]) + (x[1] + x[3]);
    const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
    return dot_tree16(__uint_as_float(h[0]) + __uint_as_float(h[1]));
}

__device__ __forceinline__ float word_value(uint64_t w) { return __uint_as_float(static_cast<uint32_t>(w >> 32)); }

}  // namespace

// NS: samples per chunk held in registers, at least ceil((N + 1) / kWideChunks); ROWS: units a lane of an
// item's wavefront reads, at least ceil(units / 64), or 0: one exchange for the dots (at most 32 units)
template <int NS, int ROWS>
__global__ __launch_bounds__(kWideBlock) void wide_run_kernel(WideArgs A, WideRunArgs Q)
{
    __shared__ float4 sm_s1[kWideBlock], sm_s2[kWideBlock];
    __shared__ uint64_t st_key[kWideBlock / 64];
    __shared__ float log_gw[kRunSteps], log_best[kRunSteps];
    __shared__ uint32_t log_dec[kRunSteps];
    __shared__ uint32_t sm_fail;
    __shared__ float sm_qn;
    const uint32_t tid = threadIdx.x, c = tid / kWideQuads, aq = tid % kWideQuads;
    if (tid == 0) sm_fail = failure_get(Q.fail);
    __syncthreads();
    if (sm_fail) return;                                // an earlier launch of the run gave up
    const uint32_t r = blockIdx.y, g = blockIdx.x;
    const uint32_t nu = A.nwg;
    const uint32_t q = g * kWideQuads + aq;
    const bool active = q < A.nq;
    const uint32_t j0 = 4 * q, jc = 4 * (active ? q : A.nq - 1);   // past the last quad: the last, discarded
    // Item i is z_i'v for i < N and s1'v for i = N; half wavefront i % 8 of each unit uses it, in slot
    // i / 8. ROWS = 0: a unit's words are [chunk][slot]; otherwise an item's words are [unit], and its sum
    // has a line of its own.
    constexpr uint32_t kItems = kWideChunks * NS;
    const float4 sz4 = *reinterpret_cast<const float4 *>(A.sz_f + jc);
    const float4 c14 = *reinterpret_cast<const float4 *>(A.c1_f + jc);
    const float4 c24 = *reinterpret_cast<const float4 *>(A.c2_f + jc);
    const float4 mu4 = *reinterpret_cast<const float4 *>(A.mu_f + jc);
    uint64_t *sig = A.S + static_cast<uint64_t>(r) * A.d + jc;
    const ulonglong2 s01 = reinterpret_cast<const ulonglong2 *>(sig)[0];
    const ulonglong2 s23 = reinterpret_cast<const ulonglong2 *>(sig)[1];
    uint64_t S[4] = {s01.x, s01.y, s23.x, s23.y};
    float Sf[4];                                        // the signatures in binary32, by way of binary64
#pragma unroll
    for (int k = 0; k < 4; ++k) Sf[k] = static_cast<float>(static_cast<double>(S[k]));
    const float sz[4] = {sz4.x, sz4.y, sz4.z, sz4.w}, c1[4] = {c14.x, c14.y, c14.z, c14.w};
    const float c2[4] = {c24.x, c24.y, c24.z, c24.w}, mu[4] = {mu4.x, mu4.y, mu4.z, mu4.w};
    uint64_t *lines = Q.words + static_cast<size_t>(r) * nu * kRunLine;
    uint64_t *parts = Q.words + static_cast<size_t>(A.R) * nu * kRunLine + static_cast<size_t>(r) * 2 * nu * kItems;
    uint64_t *sums = Q.words + static_cast<size_t>(A.R) * nu * (kRunLine + 2 * kItems) + static_cast<size_t>(r) * 2 * kItems * 8;
    const uint32_t items = A.N >= c ? (A.N - c) / kWideChunks + 1 : 0;   // items this half wavefront uses

    // the epoch's samples i = c, c + 8, ... of the quad, and their sum per asset into sm_s1 (the sum
    // fuses each term with the product that forms it, as in the sample kernel)
    float z[NS][4];
    auto draw = [&](uint32_t epoch) {
        const PhiloxRow row = philox_row(epoch, r, A.k0);
        float s1[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int m = 0; m < NS; ++m) {
            const uint32_t i = c + kWideChunks * m;
            const Words4 x = philox_block(row, i * A.nq + q, A.dom, A.k0, A.k1);
            const bool in = i < A.N;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float u1 = uniform_open01(h ? x.x2 : x.x0), u2 = uniform_open01(h ? x.x3 : x.x1);
                const float rad = in ? __builtin_amdgcn_sqrtf(-__builtin_amdgcn_logf(u1)) : 0.0f;
                const float cs = __builtin_amdgcn_cosf(u2), sn = __builtin_amdgcn_sinf(u2);
                s1[2 * h] = fmaf(rad, cs, s1[2 * h]);
                s1[2 * h + 1] = fmaf(rad, sn, s1[2 * h + 1]);
                z[m][2 * h] = rad * cs;
                z[m][2 * h + 1] = rad * sn;
            }
        }
        sm_s1[tid] = make_float4(s1[0], s1[1], s1[2], s1[3]);
    };
    // over the chunks, in chunk order (the first chunk's threads)
    auto chunk_sum = [&](const float4 *sm, float (&tot)[4]) {
        const float4 a = sm[aq];
        tot[0] = a.x, tot[1] = a.y, tot[2] = a.z, tot[3] = a.w;
#pragma unroll
        for (int cc = 1; cc < kWideChunks; ++cc) {
            const float4 b = sm[cc * kWideQuads + aq];
            tot[0] += b.x, tot[1] += b.y, tot[2] += b.z, tot[3] += b.w;
        }
    };
    auto scale = [](uint64_t t) {
        return t == 0 ? 0.0f : static_cast<float>(2.0 / (static_cast<double>(t) * static_cast<double>(t + 1)));
    };

    uint32_t epoch = static_cast<uint32_t>(Q.t0 / Q.M), in_epoch = static_cast<uint32_t>(Q.t0 % Q.M);
    draw(epoch);
    __syncthreads();
    float s1[4] = {0.0f, 0.0f, 0.0f, 0.0f};             // the first chunk's threads: sum_i z_i per asset
    bool fresh = true;                                  // the epoch's s1 is still to be summed
    float cw = scale(Q.t0);

    for (uint64_t t = Q.t0; t < Q.t1; ++t) {
        const uint32_t tag = static_cast<uint32_t>(t) + 1u;
        uint64_t *part = parts + static_cast<size_t>(t & 1) * nu * kItems;
        uint64_t *sum = sums + static_cast<size_t>(t & 1) * kItems * 8;
        float w[4], v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) w[k] = active ? Sf[k] * cw : 0.0f;
        if (t == 0 && Q.from_w0 && active) {
            const float4 w04 = *reinterpret_cast<const float4 *>(A.w0_f + jc);
            w[0] = w04.x, w[1] = w04.y, w[2] = w04.z, w[3] = w04.w;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = active ? sz[k] * w[k] : 0.0f;

        // the unit's part of z_i'v, lane m of the half wavefront publishing sample c + 8 m, then of s1'v
        auto part_put = [&](uint32_t item, float x) {
            uint64_t *slot = ROWS == 0 ? part + static_cast<size_t>(g) * kItems + (item % kWideChunks) * NS + item / kWideChunks
                                    : part + static_cast<size_t>(item) * nu + g;
            exchange_put(slot, __float_as_uint(x), tag);
        };
        {
            float mine = 0.0f;
#pragma unroll
            for (int m = 0; m < NS; ++m) {
                float p = 0.0f;
#pragma unroll
                for (int k = 0; k < 4; ++k) p = fmaf(z[m][k], v[k], p);
                p = dpp_sum32(p);
                mine = aq == static_cast<uint32_t>(m) ? p : mine;
            }
            if (aq < static_cast<uint32_t>(NS) && c + kWideChunks * aq < A.N) part_put(c + kWideChunks * aq, mine);
            if (c == 0) {
                if (fresh) chunk_sum(sm_s1, s1);
                float qp = 0.0f;
#pragma unroll
                for (int k = 0; k < 4; ++k) qp = fmaf(s1[k], v[k], qp);
                qp = dpp_sum32(qp);
                if (aq == 0) part_put(A.N, qp);
            }
            fresh = false;
        }
        cw = scale(t + 1);

        // A round's loads are all issued before the first is looked at; a lane past the last unit or a
        // slot past the last item repeats a valid one.
        bool seen = true;
        float dot[NS];
        if constexpr (ROWS == 0) {
            uint64_t word[NS];
            const uint64_t *src = part + static_cast<size_t>(aq < nu ? aq : nu - 1) * kItems + c * NS;
            seen = items == 0;
            for (uint32_t polls = 0; !seen && polls < kPollLimit; ++polls) {
#pragma unroll
                for (int s = 0; s < NS; ++s) word[s] = exchange_get(src + (static_cast<uint32_t>(s) < items ? s : 0));
                seen = true;
#pragma unroll
                for (int s = 0; s < NS; ++s) seen = seen && static_cast<uint32_t>(word[s]) == tag;
            }
#pragma unroll
            for (int s = 0; s < NS; ++s) dot[s] = dot_tree16(items && aq < nu ? word_value(word[s]) : 0.0f);
        } else {
            // the wavefront that owns item o: unit words, the sum
            const uint32_t lane = tid & 63u, o = g + nu * (tid / 64u);
            if (o <= A.N) {
                uint64_t word[ROWS];
                const uint64_t *src = part + static_cast<size_t>(o) * nu;
                bool all = false;
                for (uint32_t polls = 0; !all && polls < kPollLimit; ++polls) {
#pragma unroll
                    for (int k = 0; k < ROWS; ++k)
                        if (64u * k < nu) word[k] = exchange_get(src + (lane + 64u * k < nu ? lane + 64u * k : nu - 1));
                    all = true;
#pragma unroll
                    for (int k = 0; k < ROWS; ++k)
                        if (64u * k < nu) all = all && static_cast<uint32_t>(word[k]) == tag;
                }
                seen = all;
                float x[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int k = 0; k < ROWS; ++k)
                    if (64u * k < nu) x[k & 3] += lane + 64u * k < nu ? word_value(word[k]) : 0.0f;
                const float d = dot_tree(x);
                if (lane == 0) exchange_put(sum + 8 * static_cast<size_t>(o), __float_as_uint(d), tag);
            }
            uint64_t word[NS];
            bool all = items == 0;
            for (uint32_t polls = 0; !all && polls < kPollLimit; ++polls) {
#pragma unroll
                for (int s = 0; s < NS; ++s)
                    word[s] = exchange_get(sum + 8 * static_cast<size_t>(c + kWideChunks * (static_cast<uint32_t>(s) < items ? s : 0)));
                all = true;
#pragma unroll
                for (int s = 0; s < NS; ++s) all = all && static_cast<uint32_t>(word[s]) == tag;
            }
            seen = seen && all;
#pragma unroll
            for (int s = 0; s < NS; ++s) dot[s] = items ? word_value(word[s]) : 0.0f;
        }
        if (!seen) sm_fail = 1u;
#pragma unroll
        for (int s = 0; s < NS; ++s)
            if (aq == 0 && c + kWideChunks * s == A.N) sm_qn = dot[s];
        float s2[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int m = 0; m < NS; ++m) {
            if (c + kWideChunks * m < A.N) {
#pragma unroll
                for (int k = 0; k < 4; ++k) s2[k] = fmaf(z[m][k], dot[m], s2[k]);
            }
        }
        sm_s2[tid] = make_float4(s2[0], s2[1], s2[2], s2[3]);
        __syncthreads();
        if (sm_fail) {
            if (tid == 0) failure_raise(Q.fail);
            return;
        }
        if (c == 0) {
            float tot[4];
            chunk_sum(sm_s2, tot);
            const float qn = sm_qn * Q.inv_n;
            float gmin = INFINITY, gw = 0.0f;
            uint32_t jmin = 0xFFFFFFFFu;
            if (active) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float gj = fmaf(-s1[k], c1[k], fmaf(c2[k], fmaf(-s1[k], qn, tot[k]), -mu[k]));
                    if (gj < gmin) {
                        gmin = gj;
                        jmin = j0 + k;
                    }
                    gw = fmaf(gj, w[k], gw);
                }
            }
            // over the 32 lanes: the smallest key, then the lowest asset among the lanes that hold it
            const uint32_t key = value_key(gmin);
            const uint32_t m = dpp_min32(key);
            const uint32_t j = dpp_min32(key == m ? jmin : 0xFFFFFFFFu);
            if (aq == 0) vertex_put(lines, g, t, m, j);
            gw = dpp_sum32(gw);
            if (aq == 0) log_gw[t - Q.t0] = gw;
        }

        // while the vertex words travel: the next epoch's normals
        if (++in_epoch == Q.M) {
            in_epoch = 0;
            ++epoch;
            fresh = t + 1 < Q.t1;
            if (fresh) draw(epoch);
        }
        const uint64_t m = vertex_get<kWideBlock>(lines, nu, t, st_key, &sm_fail);
        if (sm_fail) {
            if (tid == 0) failure_raise(Q.fail);
            return;
        }
        const float best = key_value(static_cast<uint32_t>(m >> 32));
        const uint32_t a = (best < 0.0f) ? static_cast<uint32_t>(m) + 1u : 0u;
        if (g == 0 && tid == 0) {
            log_best[t - Q.t0] = best;
            log_dec[t - Q.t0] = a;
        }
        const uint32_t hit = a - 1u - j0;               // 0..3: the chosen asset is in this quad
        if (hit < 4u) {
            const uint64_t add = t + 1;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                S[k] += hit == static_cast<uint32_t>(k) ? add : 0;
                Sf[k] = static_cast<float>(static_cast<double>(S[k]));
            }
        }
    }
    __syncthreads();
    for (uint32_t i = tid; i < Q.t1 - Q.t0; i += kWideBlock) {
        Q.gw_log[(static_cast<uint64_t>(i) * A.R + r) * nu + g] = log_gw[i];
        if (g == 0) {
            Q.best_log[static_cast<uint64_t>(i) * A.R + r] = log_best[i];
            A.dec[static_cast<uint64_t>(r) * A.T + Q.t0 + i] = log_dec[i];
        }
    }
    if (active && c == 0) {
        reinterpret_cast<ulonglong2 *>(sig)[0] = make_ulonglong2(S[0], S[1]);
        reinterpret_cast<ulonglong2 *>(sig)[1] = make_ulonglong2(S[2], S[3]);
    }
}

namespace {

template <int NS>
const void *wide_run_form(uint32_t nwg)
{
    if (nwg <= kWideDirectUnits) return reinterpret_cast<const void *>(&wide_run_kernel<NS, 0>);
    if (nwg <= 192) return reinterpret_cast<const void *>(&wide_run_kernel<NS, 3>);
    return reinterpret_cast<const void *>(&wide_run_kernel<NS, kWideRunMaxUnits / 64>);
}

const void *wide_run_fn(uint32_t N, uint32_t nwg)
{
    const uint32_t ns = wide_run_ns(N);
    return ns == 2 ? wide_run_form<2>(nwg) : ns == 4 ? wide_run_form<4>(nwg) : wide_run_form<8>(nwg);
}

}  // namespace

bool wide_run_fits(uint32_t nwg, uint32_t R, uint32_t N, int device)
{
    // with more than kWideDirectUnits units there is a wavefront for every item (4 x 33 > N + 1)
    static_assert(4 * (kWideDirectUnits + 1) > kWideRunMaxN + 1, "an item without a wavefront would never be summed");
    if (N > kWideRunMaxN || nwg > kWideRunMaxUnits) return false;
    int cus = 0, coop = 0, per_cu = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess ||
        hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, device) != hipSuccess || !coop ||
        static_cast<uint64_t>(nwg) * R > 2ull * static_cast<uint64_t>(cus))
        return false;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, wide_run_fn(N, nwg), kWideBlock, 0) == hipSuccess && per_cu >= 2;
}

int launch_wide_run(const WideArgs &A, const WideRunArgs &Q, hipStream_t s)
{
    WideArgs a = A;
    WideRunArgs q = Q;
    void *args[] = {&a, &q};
    if (int rc = launch_cooperative(wide_run_fn(A.N, A.nwg), dim3(A.nwg, A.R), kWideBlock, args, 0, s)) return rc;
    const RunLog L{Q.gw_log, Q.best_log, A.nwg, A.R, A.d, 1.0f, A.gap_eps, Q.t0, A.T, Q.fail, A.dec, A.tau, A.cnt};
    return launch_run_log(L, Q.t1 - Q.t0, s);
}

}  // namespace fw
