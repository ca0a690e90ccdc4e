// fw_paths.hpp -- one lane per replication of Algorithm 1 (Section 3.1), fused with the FP64
// cross-path reduction (last workgroup finalises).
//
// Per iteration t of replication r (epoch k = t div M):
//   w_t       = w_0 at t = 0, else 2 S_j / (t (t+1)) from the integer signature S_j = sum of
//               (s+1) over the steps s < t that chose e_j (the step rule 2/(t+2) gives this
//               closed form of the recurrence w + gamma (s - w));
//   sampling  N samples R_i = mu + sigma .* z_i (Gaussian) or mu + sigma .* a_i z_i (elliptical t),
//             reduced in one pass to s1 = sum_i z_i and s2 = sum_i z_i (z_i' v), v = sigma .* w, so
//             Rbar = mu + sigma .* s1 / N                                        (Eq. (5))
//             (N-1) Sigma_hat w = sigma .* (s2 - s1 (s1' v) / N)                 (Eq. (4));
//   gradient  g = 2 lambda Sigma_hat w - Rbar;
//   decision  e_j for the lowest index attaining min_j g_j when that minimum is negative, else the
//             origin (the vertices of W);
//   gap       g'(w - s) and its first passage below eps (tau);
//   update    S_j += t+1 for the chosen e_j; checkpoint f(w_{t+1}) in FP64 from S.
// The outcome is Y = f(w_T) in FP64 from the exact signature.
//
// State: s1, s2, v in registers (binary32 or binary64); the signature S (u32 while T(T+1)/2 < 2^32,
// else u64) and the decision counts in a per-thread LDS column for the u32 runs from 7 assets on, in
// registers otherwise. No HBM traffic per step except the optional decision log.
//
// The kernels are templates over the asset count; each translation unit that includes this header
// instantiates one family (the selector functions at the end), so they compile side by side.
#pragma once

#include <hip/hip_runtime.h>

#include "device_reduce.hpp"
#include "device_rng.hpp"
#include "sim_types.hpp"

#include <type_traits>

namespace fw {

// ---------------------------------------------------------------------------------------------
// per-precision coefficient access
// ---------------------------------------------------------------------------------------------
template <typename Real>
struct Coef;

template <>
struct Coef<float> {
    const InstanceDesc *P;
    __device__ float mu(int j) const { return P->mu_f[j]; }
    __device__ float sz(int j) const { return P->sz_f[j]; }
    __device__ float c1(int j) const { return P->c1_f[j]; }
    __device__ float c2(int j) const { return P->c2_f[j]; }
    __device__ float w0(int j) const { return P->w0_f[j]; }
    __device__ float inv_n() const { return P->inv_n_f; }
    __device__ float tscale() const { return P->tscale_f; }
    __device__ static float rsqrt(float x) { return __builtin_amdgcn_rsqf(x); }
};

template <>
struct Coef<double> {
    const InstanceDesc *P;
    __device__ double mu(int j) const { return P->mu_d[j]; }
    __device__ double sz(int j) const { return P->sig_d[j]; }
    __device__ double c1(int j) const { return P->c1_d[j]; }
    __device__ double c2(int j) const { return P->c2_d[j]; }
    __device__ double w0(int j) const { return P->w0_d[j]; }
    __device__ double inv_n() const { return P->inv_n_d; }
    __device__ double tscale() const { return P->tscale_d; }
    __device__ static double rsqrt(double x) { return 1.0 / sqrt(x); }
};

// Block `block` of the noise stream (epoch, r): binary32 starts from the stream's Philox row,
// binary64 runs the whole generator.
template <typename Real>
__device__ __forceinline__ Block4<Real> block_of_row(const PhiloxRow &row, uint32_t block, uint32_t epoch,
                                                     uint32_t r, uint32_t dom, uint32_t k0, uint32_t k1)
{
    if constexpr (std::is_same<Real, float>::value)
        return normals_block_row(row, block, dom, k0, k1);
    else
        return normals_block<Real>(block, epoch, r, dom, k0, k1);
}

constexpr int gcd_const(int a, int b) { return b == 0 ? a : gcd_const(b, a % b); }

// The widths of the named workloads, and the small ones.
template <int D>
constexpr bool kWorkloadWidth = D <= 6 || D == 8 || D == 10 || D == 12 || D == 16;

// Whether a sample's term of s1 fuses with the product that forms it (radius times cosine or sine). It
// does in the whole groups of the named workloads' widths, at 1, 2, 6 and 10 assets in the
// samples of a last, partial group too, and under t noise with the product by the scale; elsewhere the
// product is rounded first, as the generic kernels' cursor does. A width thus keeps its decisions,
// whichever kernel runs it (a rounding more or less in s1 decides a near tie the other way: of 1e6
// replications of d = 10, N = 5, 600 iterations, the variance moved by 4e-7 of itself).
template <int D>
constexpr bool kFuseSum = kWorkloadWidth<D>;
template <int D>
constexpr bool kFuseRest = kFuseSum<D> && (D == 1 || 4 / gcd_const(D, 4) == 2);

// How an exact-width Gaussian kernel runs its samples. One table for all widths costs some of them up to
// 15 %, by registers (wavefronts per SIMD) and, with a wavefront per SIMD, by where the sample loop's code
// lies: its instructions are 8 bytes for the most part, a few of 4, and the loop is 3 to 10 % slower where
// the 8-byte ones straddle 8-byte boundaries. ms at 65,000 replications, N = 60, with the code before the
// loop padded to 0 | 4 bytes past a multiple of 8: binary32 d = 2 3.78 | 4.08, d = 8 3.53 | 3.83, d = 16
// 3.83 | 3.48; binary64 d = 5 2.75 | 2.71; 64-bit signature, d = 4, N = 12, 1,000 replications 220 | 207.
// Drawn at once, a group holds more normals and has its Philox chains side by side: binary64 d = 10,
// N = 9, 65,000 replications 2.76 against 2.93 ms; binary32 d = 3, N = 9, 5.02 against 4.84.
struct PathForm {
    bool at_once;    // a group's blocks are drawn before its first sample (or each as the samples reach it)
    bool several;    // binary32: several short groups at a time
    int start;       // the code before the sample loop is padded to this many bytes past a multiple of 8, or -1
};

template <int D, typename Real, typename WS, int NOISE, bool FEAT>
constexpr PathForm path_form()
{
    if (NOISE != 0) return {false, !FEAT, -1};
    if (FEAT) return {false, false, D <= 2 ? 0 : -1};
    if (sizeof(Real) == 8 && sizeof(WS) == 8) return {false, false, -1};
    if (sizeof(Real) == 8)
        return {D == 2 || D == 3 || D == 5 || D >= 10, false, D == 3 || D == 5 || D == 6 || D == 8 ? 4 : 0};
    if (sizeof(WS) == 8) return {D == 10, D == 8, D == 4 || D == 5 || D == 10 || D == 16 ? 4 : 0};
    if (!kWorkloadWidth<D>) return {false, true, -1};
    return {D == 1 || D == 6, D == 4 || D == 8, D == 10 || D == 16 ? 4 : 0};
}

template <int START>
__device__ __forceinline__ void code_start()
{
    if constexpr (START == 0) asm volatile(".p2align 3");
    if constexpr (START == 4) asm volatile(".p2align 3\n\ts_nop 0");
}

// The per-replication records a run accumulates: signature S_j and decision counts. With a 32-bit
// signature and 7 assets or more they live in LDS, [category][thread], each thread its own column (category 0 the origin,
// whose signature row only absorbs the additions of steps that choose it): a step is then two LDS
// additions at a dynamic index, where registers need a compare, a select and an add per asset for
// each of S and the counts -- 50 of the 250 VALU instructions an iteration spends outside its
// samples at d = 10, and 2 d + 1 registers. Feature runs (whose LDS holds the category sums) and 64-bit
// signatures keep registers.
template <int D, typename WS, bool LDS, int STRIDE = kBlock>
struct PathRec;

template <int D, typename WS, int STRIDE>
struct PathRec<D, WS, true, STRIDE> {
    WS *s;             // this thread's signature column
    uint32_t *c;       // and its count column
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int j = 0; j <= D; ++j) {
            s[j * STRIDE] = 0;
            c[j * STRIDE] = 0;
        }
    }
    __device__ __forceinline__ WS sig(int j) const { return s[(j + 1) * STRIDE]; }
    __device__ __forceinline__ uint32_t count(int j) const { return c[j * STRIDE]; }
    __device__ __forceinline__ void step(int a, WS tp1)
    {
        __hip_atomic_fetch_add(s + a * STRIDE, tp1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_fetch_add(c + a * STRIDE, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
};

template <int D, typename WS, int STRIDE>
struct PathRec<D, WS, false, STRIDE> {
    WS s[D];
    uint32_t c[D + 1];
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int j = 0; j < D; ++j) s[j] = 0;
#pragma unroll
        for (int j = 0; j <= D; ++j) c[j] = 0;
    }
    __device__ __forceinline__ WS sig(int j) const { return s[j]; }
    __device__ __forceinline__ uint32_t count(int j) const
    {
        uint32_t x = 0;
#pragma unroll
        for (int k = 0; k <= D; ++k)
            if (k == j) x = c[k];
        return x;
    }
    __device__ __forceinline__ void step(int a, WS tp1)
    {
        c[0] += (a == 0) ? 1u : 0u;
#pragma unroll
        for (int j = 0; j < D; ++j) {
            const bool hit = (a == j + 1);
            s[j] += hit ? tp1 : WS(0);
            c[j + 1] += hit ? 1u : 0u;
        }
    }
};

// f(w) = lambda sum_j sigma_j^2 w_j^2 - mu' w at w = c S (Eq. (3), diagonal Sigma), in FP64
template <int D, bool EXACT, class Rec>
__device__ __forceinline__ double objective_from_signature(const InstanceDesc *__restrict__ P, const Rec &rec, double c)
{
    const int d = EXACT ? D : static_cast<int>(P->d);
    double quad = 0.0, lin = 0.0;
#pragma unroll
    for (int j = 0; j < D; ++j) {
        if (j < d) {
            const double w = static_cast<double>(rec.sig(j)) * c;
            const double sw = P->sig_d[j] * w;
            quad = fma(sw, sw, quad);
            lin = fma(P->mu_d[j], w, lin);
        }
    }
    return fma(P->lambda, quad, -lin);
}

struct LaneResult {
    double y;
    uint32_t tau;
};

__device__ __forceinline__ float lane_value(float x, uint32_t lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}

__device__ __forceinline__ double lane_value(double x, uint32_t lane)
{
    const uint64_t b = static_cast<uint64_t>(__double_as_longlong(x));
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(b), lane);
    const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(b >> 32), lane);
    return __longlong_as_double(static_cast<long long>((static_cast<uint64_t>(hi) << 32) | lo));
}

// The source of a replication's normals: its own lane draws them (fw_paths_split.hpp has another).
struct OwnDraws {
    static constexpr bool kFed = false;
    static constexpr int kStride = kBlock;             // lanes of an LDS record row
};

// One replication of Algorithm 1; returns Y and tau, leaves signature and counts in rec. Every lane of
// the wavefront takes part (lanes past R repeat the last replication and store nothing).
template <int D, bool EXACT, typename Real, int NOISE, typename WS, bool FEAT, bool SCHED, class Rec, class Feed = OwnDraws>
__device__ __forceinline__ void run_path(const InstanceDesc *__restrict__ P, const RunBuffers &B,
                                         uint32_t r, bool active, Rec &rec, LaneResult &res, uint64_t *feat_cnt, Feed feed = Feed{})
{
    const Coef<Real> C{P};
    const int d = EXACT ? D : static_cast<int>(P->d);
    uint32_t N = P->N;
    const uint32_t M = P->M;
    // per-epoch sample sizes: N_k, 1/N_k and the coefficient rows of the current epoch
    const Real *c1s = nullptr;
    const Real *c2s = nullptr;
    Real inv_ns = Real(0);
    auto set_epoch = [&](uint32_t e) {
        if constexpr (SCHED) {
            N = B.sched_n[e];
            if constexpr (std::is_same<Real, float>::value) {
                inv_ns = B.sched_inv_f[e];
                c1s = B.sched_c_f + static_cast<uint64_t>(e) * 2 * d;
            } else {
                inv_ns = B.sched_inv_d[e];
                c1s = B.sched_c_d + static_cast<uint64_t>(e) * 2 * d;
            }
            c2s = c1s + d;
        }
    };
    set_epoch(0);
    // the 32-bit signature bounds T, so its runs count iterations in one scalar register
    using Step = std::conditional_t<sizeof(WS) == 4, uint32_t, uint64_t>;
    const Step T = static_cast<Step>(P->T);
    const uint32_t k0 = static_cast<uint32_t>(P->seed), k1 = static_cast<uint32_t>(P->seed >> 32);
    const uint32_t dom = P->instance & 0xFFFFFFu;   // domain 0: path noise
    const uint64_t R = P->R;
    const bool logged = active && (P->flags & 2u) && (static_cast<uint64_t>(r) - P->log_begin) < P->log_count;
    const uint32_t n_ckpt = P->n_ckpt;

    rec.clear();
    uint32_t tau = kTauNone;
    uint32_t ck = 0;
    Step next_ckpt = n_ckpt ? static_cast<Step>(P->ckpt[0]) : 0;
    uint32_t epoch = 0, m_in_epoch = 0;   // t = epoch * M + m_in_epoch
    // control-variate summaries: per category (0 origin, j+1 vertex e_j) the integer sum of (t+1)^2
    // over iterations whose epoch's reference decision is that category, in this thread's column
    // of LDS (feat_cnt[c * Feed::kStride]); the (t+1)-weighted count of the most probable category
    uint64_t fcnt1 = 0;
    const uint32_t ftop = FEAT ? P->cv_top : 0u;
    if constexpr (FEAT) {
#pragma unroll
        for (int c = 0; c <= D; ++c) feat_cnt[c * Feed::kStride] = 0;
    }

    Real cw_lane = Real(0);
    for (Step t = 0; t < T; ++t) {
        // the scale 2/(t (t+1)) of the signature: lane l divides for iteration t + l once every 64
        // iterations, and each iteration reads its lane (an FP64 division is ~17 double-rate
        // instructions, 2% of an iteration at d = N = 10)
        const uint32_t tl = static_cast<uint32_t>(t) & 63u;
        if (tl == 0u) {
            const double tt = static_cast<double>(t) + static_cast<double>(threadIdx.x & 63u);
            cw_lane = static_cast<Real>(tt == 0.0 ? 0.0 : 2.0 / (tt * (tt + 1.0)));
        }
        const Real cwr = lane_value(cw_lane, tl);
        // iterate w_t and v = sigma .* w_t
        Real v[D], s1[D], s2[D];
        Real g1[D];          // FEAT with t noise: sum of the Gaussian numerators
        // w_t = cw S except at t = 0 with a given start point (S = 0 and cw = 0 there, so the
        // origin needs no special case); one uniform branch instead of a select per asset
        const bool from_w0 = (t == 0) && P->has_w0;
#pragma unroll
        for (int j = 0; j < D; ++j) {
            v[j] = (j < d) ? C.sz(j) * (static_cast<Real>(rec.sig(j)) * cwr) : Real(0);
            s1[j] = Real(0);
            s2[j] = Real(0);
            g1[j] = Real(0);
        }
        if (from_w0) {
#pragma unroll
            for (int j = 0; j < D; ++j) v[j] = (j < d) ? C.sz(j) * C.w0(j) : Real(0);
        }
        const bool feat_epoch = FEAT && m_in_epoch == 0;   // draws repeat within an epoch

        // one sample's part of the sums, in the order every kernel here uses
        auto add_sample = [&](const Real *z, auto fuse) {
            Real dot = Real(0);
#pragma unroll
            for (int j = 0; j < D; ++j) dot = fma(z[j], v[j], dot);
#pragma unroll
            for (int j = 0; j < D; ++j) {
                if constexpr (decltype(fuse)::value) {
                    s1[j] += z[j];
                } else {
#pragma clang fp contract(off)
                    s1[j] += z[j];
                }
                s2[j] = fma(z[j], dot, s2[j]);
            }
        };
        // t noise: the scale of the next sample, from nu normals of the stream's second part
        NormalCursor<Real> ext;
        if constexpr (NOISE == 1) ext.seek(N * static_cast<uint32_t>(d), epoch, r, dom, k0, k1);
        auto t_scale = [&]() {
            Real ss = Real(0);
            for (uint32_t k = 0; k < P->nu; ++k) {
                const Real e = ext.next(epoch, r, dom, k0, k1);
                ss = fma(e, e, ss);
            }
            return C.tscale() * Coef<Real>::rsqrt(ss);
        };

        if constexpr (Feed::kFed) {
            feed.samples(N, v, s1, s2);
        } else if constexpr (EXACT) {
            // groups of G samples hold a whole number of Philox blocks: static packing. Drawn as the
            // samples reach them, blocks leave a wide instance to hold one sample and a part. Several
            // groups at a time have enough independent Philox chains (4 to 6 blocks) to cover a
            // chain's latency at few wavefronts per SIMD.
            constexpr int G = 4 / gcd_const(D, 4);
            constexpr int NB = G * D / 4;
            constexpr PathForm F = path_form<D, Real, WS, NOISE, FEAT>();
            constexpr int MUL = F.several && sizeof(Real) == 4 ? (NB == 1 ? 4 : NB <= 3 ? 2 : 1) : 1;
            PhiloxRow row{};
            if constexpr (std::is_same<Real, float>::value) row = philox_row(epoch, r, k0);
            // the next samples from block b0 on: all GS of them, or with GS = 0 the first n of a group
            auto group = [&](uint32_t b0, uint32_t n, auto size) {
                constexpr int GS = decltype(size)::value ? decltype(size)::value : G;
                Real z[GS * D];
                auto block = [&](int b) {
                    const Block4<Real> q = block_of_row<Real>(row, b0 + b, epoch, r, dom, k0, k1);
                    z[4 * b + 0] = q.z[0];
                    z[4 * b + 1] = q.z[1];
                    z[4 * b + 2] = q.z[2];
                    z[4 * b + 3] = q.z[3];
                };
                if constexpr (F.at_once) {
#pragma unroll
                    for (int b = 0; b < GS * D / 4; ++b) {
                        if (decltype(size)::value || static_cast<uint32_t>(b) < (n * D + 3) / 4) block(b);
                        else z[4 * b + 0] = z[4 * b + 1] = z[4 * b + 2] = z[4 * b + 3] = Real(0);
                    }
                }
#pragma unroll
                for (int s = 0; s < GS; ++s) {
                    if (decltype(size)::value || static_cast<uint32_t>(s) < n) {
                        if constexpr (!F.at_once) {
#pragma unroll
                            for (int b = (s * D + 3) / 4; b < ((s + 1) * D + 3) / 4; ++b) block(b);
                        }
                        if constexpr (FEAT && NOISE == 1) {
#pragma unroll
                            for (int j = 0; j < D; ++j) g1[j] += z[s * D + j];
                        }
                        if constexpr (NOISE == 1) {
                            const Real a = t_scale();
                            Real y[D];
#pragma unroll
                            for (int j = 0; j < D; ++j) y[j] = z[s * D + j] * a;
                            add_sample(y, std::true_type{});
                        } else {
                            add_sample(z + s * D, std::integral_constant<bool, decltype(size)::value != 0 ? kFuseSum<D> : kFuseRest<D>>{});
                        }
                    }
                }
            };
            const uint32_t full = N / G, rem = N % G;
            uint32_t gi = 0;
            if constexpr (MUL > 1) {
                code_start<F.start>();
                for (; gi + MUL <= full; gi += MUL) group(gi * NB, 0, std::integral_constant<int, MUL * G>{});
            }
            code_start<F.start>();
            for (; gi < full; ++gi) group(gi * NB, 0, std::integral_constant<int, G>{});
            if (rem) group(full * NB, rem, std::integral_constant<int, 0>{});
        } else {
            NormalCursor<Real> cur;
            cur.seek(0u, epoch, r, dom, k0, k1);
            for (uint32_t i = 0; i < N; ++i) {
                Real z[D];
#pragma unroll
                for (int j = 0; j < D; ++j) z[j] = (j < d) ? cur.next(epoch, r, dom, k0, k1) : Real(0);
                if constexpr (FEAT && NOISE == 1) {
#pragma unroll
                    for (int j = 0; j < D; ++j) g1[j] += z[j];
                }
                if constexpr (NOISE == 1) {
                    const Real a = t_scale();
#pragma unroll
                    for (int j = 0; j < D; ++j) z[j] *= a;
                }
                add_sample(z, std::integral_constant<bool, NOISE == 1>{});
            }
        }

        if constexpr (FEAT) {
            if (feat_epoch) {
                // the reference decision for b - sigma .* zbar (lowest index among equal minima,
                // the origin when the minimum is >= 0), weighted by the epoch's sums of (t+1)^2
                // and (t+1) over [t, min(t + M, T))
                const uint64_t t0 = t, t1 = (t0 + M < T) ? t0 + M : T;
                const uint64_t w2 = (M == 1) ? (t0 + 1) * (t0 + 1)
                                             : t1 * (t1 + 1) * (2 * t1 + 1) / 6 - t0 * (t0 + 1) * (2 * t0 + 1) / 6;
                const uint64_t w1 = (M == 1) ? t0 + 1 : t1 * (t1 + 1) / 2 - t0 * (t0 + 1) / 2;
                float vmin = 0.0f;
                uint32_t pick = 0;
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    if (j < d) {
                        const float u = static_cast<float>((NOISE == 1) ? g1[j] : s1[j]);
                        const float v = fmaf(-P->cv_s[j], u, P->cv_b[j]);
                        if (v < vmin) {
                            vmin = v;
                            pick = static_cast<uint32_t>(j + 1);
                        }
                    }
                }
                feat_cnt[pick * Feed::kStride] += w2;
                fcnt1 += (pick == ftop) ? w1 : 0u;
            }
        }

        // gradient, linear subproblem over the vertices of W, Frank-Wolfe gap
        Real dot1 = Real(0);
#pragma unroll
        for (int j = 0; j < D; ++j) dot1 = fma(s1[j], v[j], dot1);
        const Real qn = dot1 * (SCHED ? inv_ns : C.inv_n());
        Real gmin = Real(0);
        int jmin = -1;
        Real gw = Real(0);
        Real gv[D];
#pragma unroll
        for (int j = 0; j < D; ++j) {
            gv[j] = Real(0);
            if (j < d) {
                // c2 (s2 - s1 qn) - mu - c1 s1 with every product fused explicitly, so that each
                // kernel instantiation rounds it the same way
                const Real c1j = SCHED ? c1s[j] : C.c1(j), c2j = SCHED ? c2s[j] : C.c2(j);
                const Real g = fma(-c1j, s1[j], fma(c2j, fma(-s1[j], qn, s2[j]), -C.mu(j)));
                if (jmin < 0 || g < gmin) {
                    gmin = g;
                    jmin = j;
                }
                gv[j] = g;
                gw = fma(g, static_cast<Real>(rec.sig(j)) * cwr, gw);
            }
        }
        if (from_w0) {
            gw = Real(0);
#pragma unroll
            for (int j = 0; j < D; ++j)
                if (j < d) gw = fma(gv[j], C.w0(j), gw);
        }
        const int a = (gmin < Real(0)) ? jmin + 1 : 0;
        const Real gap = gw - (gmin < Real(0) ? gmin : Real(0));
        if (tau == kTauNone && gap <= static_cast<Real>(P->gap_eps)) tau = static_cast<uint32_t>(t);
        if (logged) B.dlog[static_cast<uint64_t>(t) * P->log_count + (r - P->log_begin)] = static_cast<uint8_t>(a);

        // step 2/(t+2): the signature absorbs the update
        rec.step(a, static_cast<WS>(t + 1));
        if (t + 1 == next_ckpt) {
            const double c = 2.0 / (static_cast<double>(t + 1) * static_cast<double>(t + 2));
            const double f = objective_from_signature<D, EXACT>(P, rec, c);
            if (active) B.fck[static_cast<uint64_t>(ck) * R + r] = f;
            ++ck;
            next_ckpt = ck < n_ckpt ? static_cast<Step>(P->ckpt[ck]) : 0;
        }
        if (++m_in_epoch == M) {
            m_in_epoch = 0;
            ++epoch;
            if (t + 1 < T) set_epoch(epoch);
        }
    }
    res.y = objective_from_signature<D, EXACT>(
        P, rec, 2.0 / (static_cast<double>(T) * static_cast<double>(T + 1)));
    res.tau = tau;
    if constexpr (FEAT) {
        // x_j for vertex e_j (category j+1), x_d for the origin, x_{d+1} the (t+1)-weighted count of
        // the most probable category; the integer counts are exact in FP64 (< 2^53)
        if (active) {
#pragma unroll
            for (int c = 0; c <= D; ++c) {
                if (c <= d) {
                    const uint64_t row = (c == 0) ? static_cast<uint64_t>(d) : static_cast<uint64_t>(c - 1);
                    B.feat[row * R + r] =
                        static_cast<float>((static_cast<double>(feat_cnt[c * Feed::kStride]) - P->cv_mean[c]) * P->cv_inv[c]);
                }
            }
            B.feat[static_cast<uint64_t>(d + 1) * R + r] =
                static_cast<float>((static_cast<double>(fcnt1) - P->cv_mean1) * P->cv_inv1);
        }
    }
}

// The workgroup's partials and, in the last workgroup to finish, the run's statistics, from replication
// r's outcome, hitting time and decision counts (256 threads, LDS sm_f [2 kBlock / 64], sm_i
// [kBlock / 64], sm_last).
template <class Count>
__device__ __forceinline__ void reduce_paths(const InstanceDesc *__restrict__ P, const RunBuffers &B, uint64_t r, bool active, int d,
                                             double y, uint32_t tau, Count count, double *sm_f, uint64_t *sm_i, uint32_t *sm_last)
{
    const uint64_t R = P->R;
    // per-workgroup partials: streams Y, f(w_c), RSE_c
    const uint32_t nb = B.nblocks;
    const uint32_t n_ckpt = P->n_ckpt;
    const uint32_t n_streams = 1 + 2 * n_ckpt;
    for (uint32_t s = 0; s < n_streams; ++s) {
        double x = 0.0;
        bool valid = active;
        if (active) {
            if (s == 0) {
                x = y;
            } else if (s <= n_ckpt) {
                x = B.fck[static_cast<uint64_t>(s - 1) * R + r];
            } else {
                const double f = B.fck[static_cast<uint64_t>(s - 1 - n_ckpt) * R + r];
                valid = (f != 0.0);
                const double e = valid ? (f - y) / f : 0.0;
                x = e * e;
            }
        }
        if (!valid) x = 0.0;
        double h = x, l = 0.0;
        block_sum_dd(h, l, sm_f);
        double qh = x * x, ql = fma(x, x, -(x * x));
        block_sum_dd(qh, ql, sm_f);
        double ch = valid ? 1.0 : 0.0, cl = 0.0;
        block_sum_dd(ch, cl, sm_f);
        if (threadIdx.x == 0) {
            double *base = B.part_f + static_cast<uint64_t>(s) * kStreamFields * nb + blockIdx.x;
            store_agent(base + 0 * nb, h);
            store_agent(base + 1 * nb, l);
            store_agent(base + 2 * nb, qh);
            store_agent(base + 3 * nb, ql);
            store_agent(base + 4 * nb, ch);
        }
    }
    {
        const double ymin = block_extreme<false>(active ? y : INFINITY, sm_f);
        const double ymax = block_extreme<true>(active ? y : -INFINITY, sm_f);
        if (threadIdx.x == 0) {
            double *base = B.part_f + static_cast<uint64_t>(n_streams) * kStreamFields * nb + blockIdx.x;
            store_agent(base, ymin);
            store_agent(base + nb, ymax);
        }
    }
    for (int j = 0; j <= d; ++j) {
        const uint32_t cj = active ? count(j) : 0u;
        const uint64_t tot = block_sum_u64(cj, sm_i);
        if (threadIdx.x == 0) store_agent(B.part_i + static_cast<uint64_t>(j) * nb + blockIdx.x, tot);
    }
    {
        const bool hit = active && tau != kTauNone;
        const uint64_t tc = block_sum_u64(hit ? 1u : 0u, sm_i);
        const uint64_t ts = block_sum_u64(hit ? tau : 0u, sm_i);
        if (threadIdx.x == 0) {
            store_agent(B.part_i + static_cast<uint64_t>(d + 1) * nb + blockIdx.x, tc);
            store_agent(B.part_i + static_cast<uint64_t>(d + 2) * nb + blockIdx.x, ts);
        }
    }

    // the last workgroup to finish reduces every partial in a fixed order
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t prev = __hip_atomic_fetch_add(B.done, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        *sm_last = (prev == nb - 1) ? 1u : 0u;
    }
    __syncthreads();
    if (!*sm_last) return;
    __threadfence();

    for (uint32_t s = 0; s < n_streams; ++s) {
        const double *base = B.part_f + static_cast<uint64_t>(s) * kStreamFields * nb;
        double h = 0.0, l = 0.0, qh = 0.0, ql = 0.0, ch = 0.0, cl = 0.0;
        for (uint32_t b = threadIdx.x; b < nb; b += kBlock) {
            dd_add(h, l, load_agent(base + 0 * nb + b), load_agent(base + 1 * nb + b));
            dd_add(qh, ql, load_agent(base + 2 * nb + b), load_agent(base + 3 * nb + b));
            dd_add(ch, cl, load_agent(base + 4 * nb + b), 0.0);
        }
        block_sum_dd(h, l, sm_f);
        block_sum_dd(qh, ql, sm_f);
        block_sum_dd(ch, cl, sm_f);
        if (threadIdx.x == 0) {
            double *o = B.final_f + static_cast<uint64_t>(s) * kStreamFields;
            o[0] = h;
            o[1] = l;
            o[2] = qh;
            o[3] = ql;
            o[4] = ch + cl;
        }
    }
    {
        const double *base = B.part_f + static_cast<uint64_t>(n_streams) * kStreamFields * nb;
        double mn = INFINITY, mx = -INFINITY;
        for (uint32_t b = threadIdx.x; b < nb; b += kBlock) {
            mn = fmin(mn, load_agent(base + b));
            mx = fmax(mx, load_agent(base + nb + b));
        }
        mn = block_extreme<false>(mn, sm_f);
        mx = block_extreme<true>(mx, sm_f);
        if (threadIdx.x == 0) {
            B.final_f[n_streams * kStreamFields] = mn;
            B.final_f[n_streams * kStreamFields + 1] = mx;
        }
    }
    for (int j = 0; j < d + 3; ++j) {
        uint64_t x = 0;
        for (uint32_t b = threadIdx.x; b < nb; b += kBlock) x += load_agent(B.part_i + static_cast<uint64_t>(j) * nb + b);
        x = block_sum_u64(x, sm_i);
        if (threadIdx.x == 0) B.final_i[j] = x;
    }
    if (threadIdx.x == 0) __hip_atomic_store(B.done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------------------------------------
// kernel: paths + per-workgroup partials + last-workgroup finalisation
// ---------------------------------------------------------------------------------------------
template <int D, bool EXACT, typename Real, int NOISE, typename WS, bool FEAT, bool SCHED>
__global__ __launch_bounds__(kBlock) void fw_paths_kernel(const InstanceDesc *__restrict__ P,
                                                          RunBuffers B)
{
    __shared__ double sm_f[2 * (kBlock / 64)];
    __shared__ uint64_t sm_i[kBlock / 64];
    __shared__ uint32_t sm_last;
    // control-variate counts, [category][thread]: each thread owns its column
    __shared__ uint64_t sm_feat[FEAT ? (D + 1) * kBlock : 1];

    constexpr bool kLds = !FEAT && sizeof(WS) == 4 && D >= 7;
    __shared__ WS sm_sig[kLds ? (D + 1) * kBlock : 1];
    __shared__ uint32_t sm_cnt[kLds ? (D + 1) * kBlock : 1];

    const uint64_t R = P->R;
    const uint64_t r = static_cast<uint64_t>(blockIdx.x) * kBlock + threadIdx.x;
    const bool active = r < R;
    const int d = EXACT ? D : static_cast<int>(P->d);

    PathRec<D, WS, kLds> rec;
    if constexpr (kLds) {
        rec.s = sm_sig + threadIdx.x;
        rec.c = sm_cnt + threadIdx.x;
    }
    LaneResult res{0.0, kTauNone};
    // a wavefront with any replication runs whole; one with none only joins the reductions
    const bool wave_active = r - (threadIdx.x & 63u) < R;
    if (wave_active) {
        run_path<D, EXACT, Real, NOISE, WS, FEAT, SCHED>(P, B, static_cast<uint32_t>(active ? r : R - 1), active, rec, res,
                                                         sm_feat + threadIdx.x);
    } else {
        rec.clear();
    }
    if (active) {
        if ((P->flags & 8u) && !(P->flags & 1u)) B.y[r] = res.y;   // outcomes only
        if (P->flags & 1u) {
            B.y[r] = res.y;
            B.tau[r] = res.tau;
#pragma unroll
            for (int j = 0; j <= D; ++j)
                if (j <= d) B.cnt[static_cast<uint64_t>(j) * R + r] = rec.count(j);
#pragma unroll
            for (int j = 0; j < D; ++j)
                if (j < d) B.wsum[static_cast<uint64_t>(j) * R + r] = static_cast<uint64_t>(rec.sig(j));
        }
    }

    reduce_paths(P, B, r, active, d, res.y, res.tau, [&](int j) { return rec.count(j); }, sm_f, sm_i, &sm_last);
}

// ---------------------------------------------------------------------------------------------
// host dispatch over the instantiated shapes
// ---------------------------------------------------------------------------------------------
using KernelFn = void (*)(const InstanceDesc *, RunBuffers);

struct KernelChoice {
    KernelFn fn;
    int D;
    bool exact;
};

// The kernel of width d among those of exactly LO .. HI assets.
template <int LO, int HI, typename Real, int NOISE, typename WS, bool FEAT>
inline KernelChoice choose_exact(uint32_t d)
{
    if constexpr (LO > HI) {
        return {nullptr, 0, false};
    } else {
        if (d == static_cast<uint32_t>(LO)) return {&fw_paths_kernel<LO, true, Real, NOISE, WS, FEAT, false>, LO, true};
        return choose_exact<LO + 1, HI, Real, NOISE, WS, FEAT>(d);
    }
}

// The smallest generic kernel of at least d assets.
template <typename Real, int NOISE, typename WS, bool FEAT, bool SCHED>
inline KernelChoice choose_generic(uint32_t d)
{
    if constexpr (NOISE == 1)
        if (d <= 8) return {&fw_paths_kernel<8, false, Real, NOISE, WS, FEAT, SCHED>, 8, false};
    if (d <= 16) return {&fw_paths_kernel<16, false, Real, NOISE, WS, FEAT, SCHED>, 16, false};
    if constexpr (sizeof(Real) == 4)
        if (d <= 32) return {&fw_paths_kernel<32, false, Real, NOISE, WS, FEAT, SCHED>, 32, false};
    return {nullptr, 0, false};
}

// One selector per translation unit (fw_paths_*.hip). Exact-width kernels pack each group of samples
// into whole Philox blocks at compile time; the generic ones read the stream through a cursor, one
// normal at a time, and take d <= D at run time, which costs four times as much per normal at d = 27
// (45.1 ms against 10.8 ms of issue time for 2.2e10 normals). Binary32 runs with a 32-bit signature have an exact kernel
// for every d, features too under Gaussian noise. Elsewhere the widths that the named workloads use are
// exact. Runs with per-epoch sample sizes (SCHED) use the generic kernels, whose per-sample arithmetic
// and order are the exact-width kernels' but for the rounding that kFuseSum names: a constant schedule makes the
// plain run's decisions, at the widths that fuse except in near ties.
KernelChoice paths_gauss_narrow(uint32_t d);                            // binary32, u32, d <= 16
KernelChoice paths_gauss_broad(uint32_t d);                             // binary32, u32, 17 <= d <= 32
KernelChoice paths_t_narrow(uint32_t d);                                // binary32, u32, t noise, d <= 16
KernelChoice paths_t_broad(uint32_t d);                                 // binary32, u32, t noise, 17 <= d <= 32
KernelChoice paths_features(uint32_t d, uint32_t noise);                // binary32, u32, features
KernelChoice paths_long(uint32_t d, uint32_t noise);                    // binary32, u64
KernelChoice paths_fp64(uint32_t d, uint32_t noise, bool wide);         // binary64
KernelChoice paths_sched(uint32_t d, uint32_t noise, bool fp64, bool wide);   // per-epoch sample sizes

}  // namespace fw
