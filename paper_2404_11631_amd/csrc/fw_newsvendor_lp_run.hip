// fw_newsvendor_lp_run.hip -- Algorithm 2 over X = {A x <= C, x >= 0}, many iterations in one launch.
//
// The kernels of fw_newsvendor.hip take two launches per iteration: the gradient (4.7 us) and the
// simplex on one workgroup (24.9 us at n = 1e3, M = 3: 4.8 pivots of six workgroup barriers, serial
// small-matrix steps and dependent reads). Here a cooperative launch runs iterations [t0, t1) with one
// simplex workgroup and the sample workgroups of the gradient kernel, which exchange tagged words
// (exchange.hpp):
//   samples   each sample lane group keeps its quad's x, coefficients and normals in registers, moves x
//             with the vertex it reads, counts, and publishes the quad's four counts in one word. The
//             next epoch's normals are drawn while the simplex runs.
//   simplex   reads the counts, forms g in LDS, and pivots with one barrier per pivot: every
//             wavefront keeps the basis inverse by rows and by columns (lane i its row and column i),
//             prices its columns of A, and repeats the small steps for itself; only the wavefronts'
//             best columns meet in LDS. The vertex goes out as M (column, value) pairs.
// Every operation on g, x, the basis and the reduced costs is rounded on its own and in the order of
// the launch-per-iteration kernels, so vertices, iterates and pivot counts are the same bits. The gap
// g'x - g's (binary64, for tau) is summed in another order, after the launch.
// What bounds it (cycles at n = 1,000, 3 rows, 5.7 pricings an iteration): the way of the vertex to the
// samples and of the counts back 7,800, and 2,980 a pricing's pass, a serial chain: y' = c_B' B^-1 280, the
// reduced costs 950, their minimum and the barrier 490, the choice 400, the ratio test 570, the update 320.
// At n = 10,000 a pricing's reduced costs are 10,600, one compute unit reading A through the L2.
#include <hip/hip_runtime.h>

#include "device_rng.hpp"
#include "exchange.hpp"
#include "newsvendor.hpp"
#include "newsvendor_device.hpp"
#include "sim_types.hpp"
#include "wave_dpp.hpp"

namespace fw {

namespace {

__device__ __forceinline__ double lane_double(double x, uint32_t lane)
{
    const uint64_t b = static_cast<uint64_t>(__double_as_longlong(x));
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(b), lane);
    const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(b >> 32), lane);
    return __longlong_as_double(static_cast<long long>((static_cast<uint64_t>(hi) << 32) | lo));
}

// the smallest of the wavefront's values, in every lane
__device__ __forceinline__ double wave_min(double x)
{
    x = fmin(x, dpp_move<0xB1>(x));
    x = fmin(x, dpp_move<0x4E>(x));
    x = fmin(x, dpp_move<0x141>(x));
    x = fmin(x, dpp_move<0x140>(x));
    double a, b;
    lane_swap<false>(x, a, b);
    x = fmin(a, b);
    lane_swap<true>(x, a, b);
    return fmin(a, b);
}

// the largest binary32 value <= x: z <= x in binary64 exactly when z <= floor32(x), for binary32 z
__device__ __forceinline__ float floor32(double x)
{
    const float f = static_cast<float>(x);
    if (!(static_cast<double>(f) > x)) return f;
    const uint32_t b = __float_as_uint(f);
    return __uint_as_float(f > 0.0f ? b - 1u : b == 0u ? 0x80000001u : b + 1u);
}

// The simplex workgroup's LDS besides g (and A), per launch.
template <int M>
struct LpLog {
    uint32_t basis[kLpRunSteps][M], pivots[kLpRunSteps];
    double value[kLpRunSteps][M], gs[kLpRunSteps];
};

}  // namespace

// The sample workgroups (blockIdx.x >= 1): quads, lanes and samples as in nv_lp_gradient_kernel.
template <int M>
__device__ void lp_sample_role(const NvLpArgs &A, const NvLpRunArgs &Q, uint64_t *counts, const uint64_t *vertex,
                               double *log_gx, double *sm, uint32_t *fail)
{
    const uint32_t r = blockIdx.y, tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, grp = blockIdx.x - 1;
    const uint32_t P = A.P, sub = tid % P;
    const uint32_t q = grp * (kNvBlock / P) + tid / P;
    const bool active = q < A.nq;
    const bool lead = sub == 0;
    const uint32_t qc = active ? q : A.nq - 1, j0 = 4 * qc;       // past the last quad: the last, discarded
    double xv[4], mu[4], isk[4], km[4], hv[4];
    double *x = A.x + static_cast<uint64_t>(r) * A.n;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        xv[k] = x[j0 + k];
        mu[k] = A.mu_d[j0 + k];
        isk[k] = A.isk_d[j0 + k];
        km[k] = A.km_d[j0 + k];
        hv[k] = A.hv_d[j0 + k];
    }
    float z[kLpRunMaxNs][4];                            // samples sub, sub + P, ...; NaN past S counts nowhere
    auto draw = [&](uint32_t epoch) {
        // opaque keys: the twenty round keys are added up here, not kept in scalar registers all along
        uint32_t k0 = A.k0, k1 = A.k1;
        FW_PIN_SGPR(k0);
        FW_PIN_SGPR(k1);
        const PhiloxRow row = philox_row(epoch, r, k0);
#pragma unroll
        for (int i = 0; i < static_cast<int>(kLpRunMaxNs); ++i) {
            if (i * P < A.S) {
                const uint32_t s = sub + i * P;
                const Block4<float> b = normals_block_row(row, s * A.nq + qc, A.dom, k0, k1);
#pragma unroll
                for (int k = 0; k < 4; ++k) z[i][k] = s < A.S ? b.z[k] : NAN;
            }
        }
    };
    uint32_t epoch = static_cast<uint32_t>(Q.t0 / Q.Mr), in_epoch = static_cast<uint32_t>(Q.t0 % Q.Mr);
    draw(epoch);
    for (uint64_t t = Q.t0; t < Q.t1; ++t) {
        const uint32_t tag = static_cast<uint32_t>(t) + 1u;
        uint32_t packed = 0u;       // the four counts, eight bits each (at most S <= 255)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            // sigma_j = 0 has an infinite scale: the threshold is +-infinity, and +infinity (every sample
            // counted) where x_j equals the demand exactly
            double thr = (xv[k] - mu[k]) * isk[k];
            if (thr != thr) thr = INFINITY;
            const float th = floor32(thr);
#pragma unroll
            for (int i = 0; i < static_cast<int>(kLpRunMaxNs); ++i)
                if (i * P < A.S) packed += (z[i][k] <= th) ? 1u << (8 * k) : 0u;
        }
        packed = dpp_sum_lanes(packed, P);
        if (active && lead) exchange_put(counts + static_cast<size_t>(t & 1) * A.nq + q, packed, tag);

        // while the simplex runs: this workgroup's part of g'x, the next epoch's normals
        double gx = 0.0;
        if (active && lead) {
#pragma unroll
            for (int k = 0; k < 4; ++k) gx += nv_lp_grad(km[k], hv[k], (packed >> (8 * k)) & 0xFFu, A.S) * xv[k];
        }
        gx = dpp_sum64(gx);
        if (lane == 0) sm[wave] = gx;
        if (++in_epoch == Q.Mr) {
            in_epoch = 0;
            ++epoch;
            if (t + 1 < Q.t1) draw(epoch);
        }
        // the vertex: M (column, value) pairs in three words each
        const uint64_t *src = vertex + static_cast<size_t>(t & 1) * kLpVertexWords;
        uint64_t word[3 * M];
        bool seen = false;
        for (uint32_t polls = 0; !seen && polls < kPollLimit; ++polls) {
#pragma unroll
            for (int i = 0; i < 3 * M; ++i) word[i] = exchange_get(src + i);
            seen = true;
#pragma unroll
            for (int i = 0; i < 3 * M; ++i) seen = seen && static_cast<uint32_t>(word[i]) == tag;
        }
        if (!seen) *fail = 1u;
        __syncthreads();
        if (*fail) {
            if (tid == 0) failure_raise(Q.fail);
            return;
        }
        if (tid == 0) log_gx[t - Q.t0] = (sm[0] + sm[1]) + (sm[2] + sm[3]);
        const double gamma = 2.0 / (static_cast<double>(t) + 2.0);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            double s = 0.0;
#pragma unroll
            for (int i = 0; i < M; ++i) {
                const uint64_t bits = (word[3 * i + 1] & 0xFFFFFFFF00000000ull) | (word[3 * i + 2] >> 32);
                if (static_cast<uint32_t>(word[3 * i] >> 32) == j0 + k) s = __longlong_as_double(static_cast<long long>(bits));
            }
            xv[k] = nv_lp_move(xv[k], s, gamma);
        }
        __syncthreads();            // sm is read above before the next iteration's sums are written
    }
    if (active && lead) {
#pragma unroll
        for (int k = 0; k < 4; ++k) x[j0 + k] = xv[k];
    }
    for (uint32_t i = tid; i < Q.t1 - Q.t0; i += kNvBlock)
        Q.gx_log[(static_cast<uint64_t>(i) * A.R + r) * A.nwg + grp] = log_gx[i];
}

// The simplex workgroup (blockIdx.x == 0). g: [n] in LDS; a: [M][n], in LDS or global memory.
template <int M>
__device__ void lp_simplex_role(const NvLpArgs &A, const NvLpRunArgs &Q, const uint64_t *counts, uint64_t *vertex, double *g,
                                const double *a, LpLog<M> &log, double *st_v, uint32_t *st_j, uint32_t *fail)
{
    constexpr int kWaves = kNvBlock / 64;
    const uint32_t r = blockIdx.y, tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t n = A.n;
    const uint32_t li = lane < M ? lane : 0;            // the row and column this lane keeps
    const double level = A.Cv[li];
    uint32_t origin = 0, buf = 0;

    for (uint64_t t = Q.t0; t < Q.t1; ++t) {
        const uint32_t tag = static_cast<uint32_t>(t) + 1u;
        // the counts of every quad, and g from them
        const uint64_t *src = counts + static_cast<size_t>(t & 1) * A.nq;
        bool seen = true;
        for (uint32_t q0 = tid; q0 < A.nq; q0 += 2 * kNvBlock) {
            const uint32_t q1 = q0 + kNvBlock;
            const bool two = q1 < A.nq;
            uint64_t w0 = 0, w1 = 0;
            bool all = false;
            for (uint32_t polls = 0; !all && polls < kPollLimit; ++polls) {
                w0 = exchange_get(src + q0);
                w1 = exchange_get(src + (two ? q1 : q0));
                all = static_cast<uint32_t>(w0) == tag && static_cast<uint32_t>(w1) == tag;
            }
            seen = seen && all;
            auto quad = [&](uint32_t q, uint32_t c) {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    g[4 * q + k] = nv_lp_grad(A.km_d[4 * q + k], A.hv_d[4 * q + k], (c >> (8 * k)) & 0xFFu, A.S);
            };
            quad(q0, static_cast<uint32_t>(w0 >> 32));
            if (two) quad(q1, static_cast<uint32_t>(w1 >> 32));
        }
        if (!seen) *fail = 1u;
        __syncthreads();
        if (*fail) {
            if (tid == 0) failure_raise(Q.fail);
            return;
        }

        // the slack basis: B = I, x_B = C; lane i holds row i and column i of B^-1, x_B,i, its basic
        // column and that column's cost
        double row[M], col[M];
#pragma unroll
        for (int k = 0; k < M; ++k) row[k] = col[k] = li == static_cast<uint32_t>(k) ? 1.0 : 0.0;
        double xb = level, cb = 0.0;
        uint32_t basis = n + li;
        uint32_t pivots = 0, degenerate = 0;
        bool solved = false;
        for (;;) {
            // y' = c_B' B^-1: lane k its y_k, then all of them in every lane
            double yk = 0.0;
#pragma unroll
            for (int i = 0; i < M; ++i) yk = __dadd_rn(yk, __dmul_rn(lane_double(cb, i), col[i]));
            double y[M];
#pragma unroll
            for (int k = 0; k < M; ++k) y[k] = lane_double(yk, k);
            // pricing: the most negative reduced cost (Dantzig), or after 2M + 2 degenerate pivots in a row
            // the lowest column with a negative one (Bland)
            const bool bland = degenerate > 2 * M + 2;
            // (a column counts when its reduced cost is below -eps_r; Bland's all carry the same value).
            // Four columns' loads at a time, and selects, not branches: a lane's columns ascend, so a
            // strictly smaller value keeps the lowest.
            double bv = -A.eps_r;
            uint32_t bj = 0xFFFFFFFFu;
            auto offer = [&](double rc, uint32_t j, bool in) {
                const bool take = in && rc < bv;
                bv = take ? (bland ? -INFINITY : rc) : bv;
                bj = take ? j : bj;
            };
            for (uint32_t jb = tid; jb < n; jb += 4 * kNvBlock) {
                double rc[4], c[4][M];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t j = jb + i * kNvBlock < n ? jb + i * kNvBlock : jb;
                    rc[i] = g[j];
#pragma unroll
                    for (int k = 0; k < M; ++k) c[i][k] = a[k * n + j];
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
#pragma unroll
                    for (int k = 0; k < M; ++k) rc[i] = __dsub_rn(rc[i], __dmul_rn(y[k], c[i][k]));
                    offer(rc[i], jb + i * kNvBlock, jb + i * kNvBlock < n);
                }
            }
            offer(-yk, n + lane, wave == kWaves - 1 && lane < M);         // the slacks, the highest columns
            const double wv = wave_min(bv);
            const uint32_t wj = dpp_min64(bv == wv ? bj : 0xFFFFFFFFu);
            if (lane == 0) {
                st_v[kWaves * buf + wave] = wv;
                st_j[kWaves * buf + wave] = wj;
            }
            __syncthreads();
            // over the wavefronts: every group of four lanes reads the four candidates
            static_assert(kWaves == 4, "a quad of lanes holds the wavefronts' candidates");
            double v = st_v[kWaves * buf + (lane & 3u)];
            uint32_t q = st_j[kWaves * buf + (lane & 3u)];
            argmin_take(v, q, dpp_move<0xB1>(v), dpp_move<0xB1>(q));
            argmin_take(v, q, dpp_move<0x4E>(v), dpp_move<0x4E>(q));
            q = __builtin_amdgcn_readfirstlane(q);
            buf ^= 1u;                                  // the next pivot's candidates go to the other half
            if (q == 0xFFFFFFFFu) {                     // no negative reduced cost: optimal
                solved = true;
                break;
            }
            if (pivots == A.max_pivots) break;
            // d = B^-1 A_q (lane i its d_i), then the ratio test: the smallest x_B,i / d_i over d_i > eps_d
            // (lowest i among equal ratios)
            const double aq = q < n ? a[li * n + q] : (q - n == li ? 1.0 : 0.0);
            double d = 0.0;
#pragma unroll
            for (int k = 0; k < M; ++k) d = __dadd_rn(d, __dmul_rn(row[k], lane_double(aq, k)));
            const double ratio = lane < M && d > A.eps_d ? __ddiv_rn(xb, d) : INFINITY;
            double theta = INFINITY;
            uint32_t lv = 0xFFFFFFFFu;
#pragma unroll
            for (int i = 0; i < M; ++i) {
                const double x = lane_double(ratio, i);
                if (x < theta) {
                    theta = x;
                    lv = i;
                }
            }
            if (lv == 0xFFFFFFFFu) break;   // unbounded direction: impossible when every column has a positive entry
            // the pivot: row lv divided by d_lv, the others reduced by it; x_B and the basis likewise
            double mine = col[0];
#pragma unroll
            for (int i = 1; i < M; ++i) mine = lv == static_cast<uint32_t>(i) ? col[i] : mine;
            const double prow = __ddiv_rn(mine, lane_double(d, lv));      // lane k: entry k of the pivot row
            const double dm = d;
#pragma unroll
            for (int k = 0; k < M; ++k) {
                const double pk = lane_double(prow, k), di = lane_double(dm, k);
                row[k] = li == lv ? pk : __dsub_rn(row[k], __dmul_rn(dm, pk));
                col[k] = static_cast<uint32_t>(k) == lv ? prow : __dsub_rn(col[k], __dmul_rn(di, prow));
            }
            const double nx = li == lv ? theta : __dsub_rn(xb, __dmul_rn(dm, theta));
            xb = nx > 0.0 ? nx : 0.0;
            if (li == lv) {
                basis = q;
                cb = q < n ? g[q] : 0.0;
            }
            degenerate = theta == 0.0 ? degenerate + 1 : 0;
            ++pivots;
        }

        // the vertex to the sample workgroups, the records, g's
        if (wave == 0 && lane < M) {
            uint64_t *out = vertex + static_cast<size_t>(t & 1) * kLpVertexWords + 3 * lane;
            const uint64_t bits = static_cast<uint64_t>(__double_as_longlong(xb));
            exchange_put(out, basis, tag);
            exchange_put(out + 1, static_cast<uint32_t>(bits >> 32), tag);
            exchange_put(out + 2, static_cast<uint32_t>(bits), tag);
            log.basis[t - Q.t0][lane] = basis;
            log.value[t - Q.t0][lane] = xb;
        }
        double gs = 0.0;
        bool at_origin = true;
#pragma unroll
        for (int i = 0; i < M; ++i) {
            const double xi = lane_double(xb, i);
            if (__builtin_amdgcn_readlane(basis, i) < n && xi > 0.0) {
                gs = __dadd_rn(gs, __dmul_rn(lane_double(cb, i), xi));
                at_origin = false;
            }
        }
        origin += at_origin ? 1u : 0u;
        if (tid == 0) {
            log.gs[t - Q.t0] = gs;
            log.pivots[t - Q.t0] = solved ? pivots : A.max_pivots + 1;
        }
    }
    __syncthreads();
    for (uint32_t i = tid; i < Q.t1 - Q.t0; i += kNvBlock) {
        const uint64_t o = static_cast<uint64_t>(r) * A.T + Q.t0 + i;
#pragma unroll
        for (int k = 0; k < M; ++k) {
            A.rec_basis[o * M + k] = log.basis[i][k];
            A.rec_value[o * M + k] = log.value[i][k];
        }
        A.rec_piv[o] = log.pivots[i];
        Q.gs_log[static_cast<uint64_t>(i) * A.R + r] = log.gs[i];
    }
    if (tid == 0) A.origin[r] += origin;
}

// ALDS: the technology matrix is copied into LDS; otherwise it is read from global memory (L2).
template <int M, bool ALDS>
__global__ __launch_bounds__(kNvBlock) void nv_lp_run_kernel(NvLpArgs A, NvLpRunArgs Q)
{
    HIP_DYNAMIC_SHARED(double, lds)                     // g [n], A [M][n] (ALDS); the sample workgroups use none
    __shared__ LpLog<M> log;
    __shared__ double st_v[2 * kNvBlock / 64];
    __shared__ uint32_t st_j[2 * kNvBlock / 64];
    __shared__ uint32_t sm_fail;
    const uint32_t tid = threadIdx.x, r = blockIdx.y;
    if (tid == 0) sm_fail = failure_get(Q.fail);
    __syncthreads();
    if (sm_fail) return;                                // an earlier launch of the run gave up
    uint64_t *counts = Q.words + static_cast<size_t>(r) * 2 * A.nq;
    uint64_t *vertex = Q.words + static_cast<size_t>(A.R) * 2 * A.nq + static_cast<size_t>(r) * 2 * kLpVertexWords;
    if (blockIdx.x > 0) {
        lp_sample_role<M>(A, Q, counts, vertex, log.gs, st_v, &sm_fail);
        return;
    }
    const double *a = A.Am;
    if constexpr (ALDS) {
        for (uint32_t i = tid; i < M * A.n; i += kNvBlock) lds[A.n + i] = A.Am[i];
        a = lds + A.n;
    }
    __syncthreads();
    lp_simplex_role<M>(A, Q, counts, vertex, lds, a, log, st_v, st_j, &sm_fail);
}

// The gap and tau of iteration t0 + blockIdx.x from the logs: g'x over the sample workgroups, less g's.
__global__ __launch_bounds__(64) void nv_lp_log_kernel(NvLpArgs A, NvLpRunArgs Q)
{
    const uint32_t r = blockIdx.y;
    if (*Q.fail) return;                                // a run that gave up left no log
    const uint64_t row = static_cast<uint64_t>(blockIdx.x) * A.R + r;
    double gx = 0.0;
    for (uint32_t i = threadIdx.x; i < A.nwg; i += 64) gx += Q.gx_log[row * A.nwg + i];
    gx = dpp_sum64(gx);
    if (threadIdx.x == 0 && gx - Q.gs_log[row] <= A.gap_eps)
        atomicMin(A.tau + r, static_cast<uint32_t>(Q.t0 + blockIdx.x));
}

namespace {

template <int M>
const void *lp_run_fn(uint32_t m, bool alds)
{
    if constexpr (M > static_cast<int>(kNvLpMaxM)) {
        return nullptr;
    } else {
        if (m != static_cast<uint32_t>(M)) return lp_run_fn<M + 1>(m, alds);
        return alds ? reinterpret_cast<const void *>(&nv_lp_run_kernel<M, true>)
                    : reinterpret_cast<const void *>(&nv_lp_run_kernel<M, false>);
    }
}

// dynamic LDS of the form: g, and A where both fit beside the logs
size_t lp_run_lds(uint32_t n, uint32_t M, bool &alds)
{
    alds = static_cast<size_t>(n) * (M + 1) * sizeof(double) <= kLpRunLds;
    return static_cast<size_t>(n) * (alds ? M + 1 : 1) * sizeof(double);
}

}  // namespace

static_assert(kLpRunMaxNs * kNvMaxLanes <= 255, "counts travel in bytes");
bool nv_lp_run_fits(const NvLpArgs &A, int device)
{
    if (static_cast<size_t>(A.n) * sizeof(double) > kLpRunLds || (A.S + A.P - 1) / A.P > kLpRunMaxNs) return false;
    int cus = 0, coop = 0, per_cu = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess ||
        hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, device) != hipSuccess || !coop ||
        static_cast<uint64_t>(A.nwg + 1) * A.R > static_cast<uint64_t>(cus))
        return false;
    bool alds;
    const size_t lds = lp_run_lds(A.n, A.M, alds);
    const void *fn = lp_run_fn<1>(A.M, alds);
    // the form's largest size, not this run's: the attribute is the function's, for every context and thread
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(kLpRunLds)) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, kNvBlock, lds) == hipSuccess && per_cu >= 1;
}

int launch_nv_lp_run(const NvLpArgs &A, const NvLpRunArgs &Q, hipStream_t s)
{
    NvLpArgs a = A;
    NvLpRunArgs q = Q;
    void *args[] = {&a, &q};
    bool alds;
    const size_t lds = lp_run_lds(A.n, A.M, alds);
    if (int rc = launch_cooperative(lp_run_fn<1>(A.M, alds), dim3(A.nwg + 1, A.R), kNvBlock, args, lds, s)) return rc;
    hipLaunchKernelGGL(nv_lp_log_kernel, dim3(static_cast<uint32_t>(Q.t1 - Q.t0), A.R), dim3(64), 0, s, A, Q);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace fw
