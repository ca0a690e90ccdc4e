// fw_batch.hip -- instances of uneven size and horizon, as wavefront tiles.
//
// Algorithm 1 (Section 3.1) as in fw_paths.hpp, reorganised for a batch of instances with d up to
// 32 in one kernel:
//   * one wavefront per tile; every tile of the batch is in one launch, longest first, so the
//     hardware dispatcher hands the heaviest tiles out first and fills in with the lighter ones;
//   * a tile holds 64/P replications of one instance with P = Pa x Ps lanes per replication:
//     Pa lanes split the assets (a lane holds at most 8 of them: their iterate, sample sums,
//     signature and decision counts stay in registers), Ps lanes split the N samples into
//     contiguous chunks;
//   * the Pa lanes of a sample chunk draw its normals together: per round of G = 4/gcd(d,4)
//     samples (a whole number of Philox blocks) each lane draws every Pa-th block into LDS, and
//     each lane then reads its own assets' normals back; the sample's dot product with the
//     iterate is summed over the Pa lanes with an xor butterfly;
//   * after the samples the Ps partial sums are combined by an xor butterfly over the lanes that
//     hold the same assets; the gradient's dot product, the minimum of the linear subproblem
//     (lowest index among equal values), the gap and the objective at checkpoints are reduced over
//     the Pa lanes the same way. Butterflies give every lane of a replication the same bits, so all
//     of them take the same decision;
//   * each tile writes its partial sums to a slot fixed by (instance, replication block), and a
//     second kernel reduces every instance's slots in order, so the statistics do not depend on
//     the order in which tiles ran.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_reduce.hpp"
#include "device_rng.hpp"
#include "sim_types.hpp"
#include "wave_dpp.hpp"

namespace fw {

constexpr int kWave = 64;
constexpr int kBatchMaxD = 32;
// Workgroups up to which the one-wavefront form has three drawing wavefronts: two of four wavefronts per compute
// unit. us per iteration with one and with three: at 512 d = 10, N = 60 1.92, 1.83, N = 200 4.60, 4.36; at 1,024
// 1.95, 2.01 and 4.67, 4.76.
constexpr uint32_t kWaveManyDrawers = 512;
constexpr uint32_t kWaveMaxThreads = 256;      // up to three drawing wavefronts
constexpr int kLaneAssets = 8;                 // assets held by one lane
// LDS staging of one wavefront: a sub-group of Pa lanes draws G d <= 4 d <= 32 Pa normals per
// round, and a wavefront has 64 / Pa sub-groups. Sub-group areas are 32 Pa + 1 floats apart (131 at
// Pa = 4): with areas 32 Pa floats apart every lane of a write or read instruction would fall in
// the same few of the 64 banks (16- to 32-way conflicts); the padded stride leaves at most two
// lanes per bank for every pattern the kernel issues (checked over all d, rounds and offsets).
constexpr int kStageFloats = kBatchStageFloats;   // max over Pa of (64 / Pa) x stride
// rows of a tile's coefficient table in LDS (binary32, indexed by asset, zero past d)
constexpr int kCoefSz = 0, kCoefC1 = 1, kCoefC2 = 2, kCoefMu = 3, kCoefW0 = 4, kCoefRows = 5;
__device__ __forceinline__ uint32_t stage_stride(uint32_t Pa) { return 32u * Pa + (Pa == 4u ? 3u : 1u); }
// A lane reads kLaneAssets floats of a sample also where it has fewer assets: up to 14 past its
// sub-group's area (the neighbour's, or this pad), finite values that meet a zero coefficient.
constexpr int kStagePad = 16;

// x of this lane and of lane ^ M, added, by DPP moves and lane swaps
template <int M>
__device__ __forceinline__ float xor_sum(float x)
{
    if constexpr (M == 1) return x + dpp_move<0xB1>(x);
    if constexpr (M == 2) return x + dpp_move<0x4E>(x);
    if constexpr (M == 4) return x + dpp_move<0x1B>(dpp_move<0x141>(x));   // 7 - i, then 3 - i within the quad
    if constexpr (M == 8) return x + dpp_move<0x128>(x);                   // a 16-lane row rotated by 8
    if constexpr (M == 16) {
        const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        return __uint_as_float(p[0]) + __uint_as_float(p[1]);
    }
    if constexpr (M == 32) {
        const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        return __uint_as_float(p[0]) + __uint_as_float(p[1]);
    }
}

__device__ __forceinline__ double bfly_sum(double x, uint32_t lo, uint32_t hi)
{
    for (uint32_t m = lo; m < hi; m <<= 1) x += __shfl_xor(x, m, kWave);
    return x;
}

// Sum over the Pa <= 4 lanes of a quad-aligned group by DPP quad permutes (lane xor 1, then xor 2),
// without the LDS crossbar a shuffle goes through. Addition is commutative, so every lane of the
// group ends with the same bits. Every lane of the wavefront executes it.
__device__ __forceinline__ float quad_group_sum(float x, uint32_t Pa)
{
    if (Pa >= 2) x += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0xB1, 0xF, 0xF, true));
    if (Pa >= 4) x += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x4E, 0xF, 0xF, true));
    return x;
}

// The staging area belongs to this wavefront alone (one wavefront per workgroup), and the LDS
// instructions of a wavefront complete in issue order, so draws written by some lanes are seen by
// the reads other lanes issue after them. Only the compiler must not move LDS accesses across this
// point; no workgroup barrier (and none of its waits on outstanding global loads) is needed.
__device__ __forceinline__ void wave_lds_order()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
}

// f(w) at w = c S over this lane's assets, FP64 (Eq. (3), diagonal Sigma), summed over the Pa lanes
template <int K>
__device__ __forceinline__ double tile_objective(const InstanceDesc *__restrict__ P, const uint32_t (&S)[K],
                                                 uint32_t hibits, uint32_t a0, uint32_t acnt, uint32_t Pa, double c)
{
    double quad = 0.0, lin = 0.0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (static_cast<uint32_t>(k) < acnt) {
            const double sj = static_cast<double>(S[k]) + ((hibits >> k) & 1u ? 4294967296.0 : 0.0);
            const double w = sj * c;
            const double sw = P->sig_d[a0 + k] * w;
            quad = fma(sw, sw, quad);
            lin = fma(P->mu_d[a0 + k], w, lin);
        }
    }
    quad = bfly_sum(quad, 1u, Pa);
    lin = bfly_sum(lin, 1u, Pa);
    return fma(P->lambda, quad, -lin);
}

// PA asset lanes; a lane holds up to K assets (kLaneAssets with several lanes). What bounds it is the
// vector instructions issued (2.5e10 for 5.7e10 normals, of which the draws are about two thirds), and
// for the longest tiles an iteration's serial chain. Hence K for narrow instances, no draw past the last
// sample of a round, reads without a guard per asset, two samples side by side, the sums over lanes by
// lane moves instead of the LDS crossbar, and the step scales 64 iterations at a time. 64 instances of
// d 2..32, N 2..50, T to 10,000, 1,024 replications each: 61.5 -> 56.4 ms; a tile alone, us per
// iteration: d = 13, N = 43 over 32 lanes 4.0 -> 3.2, d = 30, N = 39 over 16 lanes 8.4 -> 6.1, d = 7,
// N = 39 on one lane 21.3 -> 14.9. Four wavefronts per SIMD instead of three (128 registers, 36 bytes
// spilled) and wave priorities by length changed nothing; tiles ordered to even out the SIMDs' loads
// gained 6 % here and lost 8 % elsewhere.
template <int PA, int K>
__device__ __forceinline__ void run_tile(const BatchBuffers &B, const Tile tile, float *stage, float (*coef)[kBatchMaxD])
{
    const InstanceDesc *P = B.inst + tile.inst;
    const uint32_t lane = threadIdx.x;
    constexpr uint32_t Pa = PA;
    const uint32_t Pl = tile.P;
    const uint32_t g = lane / Pl;                  // replication within the tile
    const uint32_t ps = (lane % Pl) / Pa;          // sample chunk
    const uint32_t pa = lane % Pa;                 // asset slice
    const bool active = g < tile.nrep;
    const bool owner = active && ps == 0;          // writes this lane's assets of the path record
    const bool leader = owner && pa == 0;
    const uint32_t r = tile.rep0 + g;
    const uint32_t d = P->d;
    const uint32_t a0 = pa * kLaneAssets;
    const uint32_t acnt = a0 < d ? (d - a0 < K ? d - a0 : K) : 0u;
    const uint32_t N = P->N, M = P->M;
    const uint64_t T = P->T;
    const uint32_t k0 = static_cast<uint32_t>(P->seed), k1 = static_cast<uint32_t>(P->seed >> 32);
    const uint32_t dom = P->instance & 0xFFFFFFu;
    const uint32_t n_ckpt = P->n_ckpt;
    const bool tnoise = P->noise != 0;
    const uint32_t nu = P->nu;
    const bool logged = leader && (P->flags & 2u) && (static_cast<uint64_t>(r) - P->log_begin) < P->log_count;
    const uint64_t log_count = P->log_count, log_at = P->dlog_base + (static_cast<uint64_t>(r) - P->log_begin);
    const bool has_w0 = P->has_w0 != 0;
    const float inv_n = P->inv_n_f, gap_eps = static_cast<float>(P->gap_eps), tscale = P->tscale_f;

    // The instance's binary32 coefficients, copied once into this wavefront's LDS and zero past d,
    // so the iteration reads them unconditionally (a0 + k < 4 x 8 = kBatchMaxD) and its reads issue
    // together: read from the descriptor under per-asset guards, each would wait for the one before.
    if (lane < static_cast<uint32_t>(kBatchMaxD)) {
        const bool in = lane < d;
        coef[kCoefSz][lane] = in ? P->sz_f[lane] : 0.0f;
        coef[kCoefC1][lane] = in ? P->c1_f[lane] : 0.0f;
        coef[kCoefC2][lane] = in ? P->c2_f[lane] : 0.0f;
        coef[kCoefMu][lane] = in ? P->mu_f[lane] : 0.0f;
        coef[kCoefW0][lane] = (in && has_w0) ? P->w0_f[lane] : 0.0f;
    }
    for (uint32_t i = lane; i < kStageFloats + kStagePad; i += kWave) stage[i] = 0.0f;
    wave_lds_order();

    // G = 4/gcd(d,4) samples hold a whole number of Philox blocks; lane chunks start on such a
    // group. A round is the largest multiple of G samples whose normals fit the sub-group's 32 Pa
    // floats of staging: the blocks a round does not divide evenly among the Pa lanes (drawn and
    // discarded) are then a small share of its draws.
    const uint32_t G = (d & 3u) == 0 ? 1u : ((d & 1u) == 0 ? 2u : 4u);
    const uint32_t align = tnoise ? 4u : G;
    const uint32_t Ps = Pl / Pa;
    uint32_t chunk = (N + Ps - 1) / Ps;
    chunk = (chunk + align - 1) / align * align;
    const uint32_t i0 = ps * chunk;
    const uint32_t i_end = (i0 + chunk < N) ? i0 + chunk : N;   // this lane's samples: [i0, i_end)
    uint32_t Gr = (32u * Pa) / d / G * G;
    Gr = Gr < G ? G : Gr;
    Gr = Gr > chunk ? chunk : Gr;                  // chunk is a multiple of G
    // the samples of the longest chunk, and whether some lanes have fewer than it or none
    const uint32_t longest = chunk < N ? chunk : N;
    const bool ragged = Ps * chunk != N;
    const uint32_t rounds = (longest + Gr - 1) / Gr;
    float *sub = stage + (lane / Pa) * stage_stride(Pa);   // this sub-group's staging area

    uint32_t S[K], cnt[K];
#pragma unroll
    for (int k = 0; k < K; ++k) S[k] = cnt[k] = 0u;
    uint32_t cnt0 = 0u, hibits = 0u;
    uint32_t tau = kTauNone;
    uint32_t ck = 0;
    uint64_t next_ckpt = n_ckpt ? P->ckpt[0] : 0;
    uint32_t epoch = 0, m_in_epoch = 0;
    const bool narrow = T <= kMaxNarrowT;          // S stays below 2^32
    float cw_lane = 0.0f;                          // lane i: the scale 2 / (t (t + 1)) of t = 64 floor(t / 64) + i

    for (uint64_t t = 0; t < T; ++t) {
        const uint32_t tl = static_cast<uint32_t>(t) % kWave;
        if (tl == 0) {
            const uint64_t u = t + lane;
            cw_lane = u == 0 ? 0.0f : static_cast<float>(2.0 / (static_cast<double>(u) * static_cast<double>(u + 1)));
        }
        const float cw = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cw_lane), tl));
        // past this lane's assets S = 0 and the coefficients are 0: w = v = 0 there, as required
        float w[K], v[K], s1[K], s2[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const float wk = (t == 0) ? coef[kCoefW0][a0 + k]
                                      : narrow ? static_cast<float>(S[k]) * cw
                                               : (static_cast<float>(S[k]) + ((hibits >> k) & 1u ? 4294967296.0f : 0.0f)) * cw;
            w[k] = wk;
            v[k] = coef[kCoefSz][a0 + k] * wk;
            s1[k] = 0.0f;
            s2[k] = 0.0f;
        }

        const PhiloxRow row = philox_row(epoch, r, k0);
        for (uint32_t rd = 0; rd < rounds; ++rd) {
            const uint32_t ib = i0 + rd * Gr;                // first sample of the round
            const uint32_t blk0 = ib * d / 4;                // its first Philox block
            const uint32_t left = longest - rd * Gr, ns = left < Gr ? left : Gr;   // samples some chunk has here
            const uint32_t nb = (ns * d + 3) / 4;            // their blocks
            const uint32_t mb = (nb + Pa - 1) / Pa;          // a lane's
            // draw: blocks pa, pa + Pa, ... of the round, two at a time
            auto put = [&](uint32_t b, const Block4<float> &q) {
                if (Pa == 1 || b < nb) {
                    sub[4 * b + 0] = q.z[0];
                    sub[4 * b + 1] = q.z[1];
                    sub[4 * b + 2] = q.z[2];
                    sub[4 * b + 3] = q.z[3];
                }
            };
            uint32_t m = 0;
            for (; m + 2 <= mb; m += 2) {
                const uint32_t b0 = pa + m * Pa, b1 = b0 + Pa;
                const Block4<float> q0 = normals_block_row(row, blk0 + b0, dom, k0, k1);
                const Block4<float> q1 = normals_block_row(row, blk0 + b1, dom, k0, k1);
                put(b0, q0);
                put(b1, q1);
            }
            if (m < mb) {
                const uint32_t b0 = pa + m * Pa;
                put(b0, normals_block_row(row, blk0 + b0, dom, k0, k1));
            }
            wave_lds_order();
            // NS samples from sidx on, their reads and dot products side by side
            auto take = [&](auto n_samples, uint32_t sidx) {
                constexpr int NS = decltype(n_samples)::value;
                float z[NS][K], dot[NS];
#pragma unroll
                for (int e = 0; e < NS; ++e) {
                    const float *src = sub + (sidx + e) * d + a0;
#pragma unroll
                    for (int k = 0; k < K; ++k) z[e][k] = src[k];
                }
                if (tnoise) {
#pragma unroll
                    for (int e = 0; e < NS; ++e) {
                        NormalCursor<float> ext;
                        ext.seek(N * d + nu * (ib + sidx + e), epoch, r, dom, k0, k1);
                        float ss = 0.0f;
#pragma unroll 1
                        for (uint32_t q = 0; q < nu; ++q) {
                            const float x = ext.next(epoch, r, dom, k0, k1);
                            ss = fmaf(x, x, ss);
                        }
                        const float a = tscale * __builtin_amdgcn_rsqf(ss);
#pragma unroll
                        for (int k = 0; k < K; ++k) z[e][k] *= a;
                    }
                }
#pragma unroll
                for (int e = 0; e < NS; ++e) {
                    dot[e] = 0.0f;
#pragma unroll
                    for (int k = 0; k < K; ++k) dot[e] = fmaf(z[e][k], v[k], dot[e]);
                }
#pragma unroll
                for (int e = 0; e < NS; ++e) dot[e] = quad_group_sum(dot[e], Pa);
#pragma unroll
                for (int e = 0; e < NS; ++e) {
                    if (!ragged || ib + sidx + e < i_end) {
#pragma unroll
                        for (int k = 0; k < K; ++k) {
                            s1[k] += z[e][k];
                            s2[k] = fmaf(z[e][k], dot[e], s2[k]);
                        }
                    }
                }
            };
            uint32_t sidx = 0;
            for (; sidx + 2 <= ns; sidx += 2) take(std::integral_constant<int, 2>{}, sidx);
            if (sidx < ns) take(std::integral_constant<int, 1>{}, sidx);
            wave_lds_order();
        }
        // combine the Ps sample chunks (lanes holding the same assets)
        auto combine = [&](auto lanes) {
            constexpr int M = decltype(lanes)::value;
            if (M >= PA && static_cast<uint32_t>(M) < Pl) {
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    s1[k] = xor_sum<M>(s1[k]);
                    s2[k] = xor_sum<M>(s2[k]);
                }
            }
        };
        combine(std::integral_constant<int, 1>{});
        combine(std::integral_constant<int, 2>{});
        combine(std::integral_constant<int, 4>{});
        combine(std::integral_constant<int, 8>{});
        combine(std::integral_constant<int, 16>{});
        combine(std::integral_constant<int, 32>{});

        // gradient, linear subproblem over the vertices of W, Frank-Wolfe gap
        float dot1 = 0.0f;
#pragma unroll
        for (int k = 0; k < K; ++k) dot1 = fmaf(s1[k], v[k], dot1);
        dot1 = quad_group_sum(dot1, Pa);
        const float qn = dot1 * inv_n;
        float c1[K], c2[K], mu[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            c1[k] = coef[kCoefC1][a0 + k];
            c2[k] = coef[kCoefC2][a0 + k];
            mu[k] = coef[kCoefMu][a0 + k];
        }
        float gmin = INFINITY, gw = 0.0f;
        uint32_t jmin = 0xFFFFFFFFu;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (static_cast<uint32_t>(k) < acnt) {
                const uint32_t j = a0 + k;
                const float gj = fmaf(-c1[k], s1[k], fmaf(c2[k], fmaf(-s1[k], qn, s2[k]), -mu[k]));
                if (jmin == 0xFFFFFFFFu || gj < gmin) {
                    gmin = gj;
                    jmin = j;
                }
                gw = fmaf(gj, w[k], gw);
            }
        }
        auto smaller = [&](float og, uint32_t oj) {
            if (og < gmin || (og == gmin && oj < jmin)) {
                gmin = og;
                jmin = oj;
            }
        };
        if (Pa >= 2) smaller(dpp_move<0xB1>(gmin), dpp_move<0xB1>(jmin));
        if (Pa >= 4) smaller(dpp_move<0x4E>(gmin), dpp_move<0x4E>(jmin));
        gw = quad_group_sum(gw, Pa);
        const uint32_t a = (gmin < 0.0f) ? jmin + 1 : 0u;
        const float gap = gw - (gmin < 0.0f ? gmin : 0.0f);
        if (tau == kTauNone && gap <= gap_eps) tau = static_cast<uint32_t>(t);
        if (logged) B.dlog[log_at + t * log_count] = static_cast<uint8_t>(a);

        // step 2/(t+2): the signature absorbs the update
        cnt0 += (a == 0u) ? 1u : 0u;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (a == a0 + k + 1) {
                const uint32_t now = S[k] + static_cast<uint32_t>(t + 1);
                if (!narrow && now < S[k]) hibits |= 1u << k;
                S[k] = now;
                cnt[k] += 1u;
            }
        }
        if (t + 1 == next_ckpt) {
            const double c = 2.0 / (static_cast<double>(t + 1) * static_cast<double>(t + 2));
            const double f = tile_objective(P, S, hibits, a0, acnt, Pa, c);
            if (leader) B.fck[static_cast<uint64_t>(ck) * B.total_R + P->path_base + r] = f;
            ++ck;
            next_ckpt = ck < n_ckpt ? P->ckpt[ck] : 0;
        }
        if (++m_in_epoch == M) {
            m_in_epoch = 0;
            ++epoch;
        }
    }
    const double y = tile_objective(P, S, hibits, a0, acnt, Pa, 2.0 / (static_cast<double>(T) * static_cast<double>(T + 1)));

    if (owner && B.y) {
        const uint64_t R = P->R;
        if (pa == 0) {
            B.y[P->path_base + r] = y;
            B.tau[P->path_base + r] = tau;
            B.cnt[P->cnt_base + r] = cnt0;
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (static_cast<uint32_t>(k) < acnt) {
                const uint64_t j = a0 + k;
                B.cnt[P->cnt_base + (j + 1) * R + r] = cnt[k];
                B.wsum[P->wsum_base + j * R + r] =
                    static_cast<uint64_t>(S[k]) | (static_cast<uint64_t>((hibits >> k) & 1u) << 32);
            }
        }
    }

    // tile partials (leaders only)
    TilePartial &out = B.partials[tile.slot];
    for (uint32_t s = 0; s < kTileStreams; ++s) {
        if (s >= 1 + 2 * n_ckpt) {
            if (lane == 0)
                for (int f = 0; f < kStreamFields; ++f) out.f[s * kStreamFields + f] = 0.0;
            continue;
        }
        double x = 0.0;
        bool valid = leader;
        if (leader) {
            if (s == 0) {
                x = y;
            } else if (s <= n_ckpt) {
                x = B.fck[static_cast<uint64_t>(s - 1) * B.total_R + P->path_base + r];
            } else {
                const double f = B.fck[static_cast<uint64_t>(s - 1 - n_ckpt) * B.total_R + P->path_base + r];
                valid = (f != 0.0);
                const double e = valid ? (f - y) / f : 0.0;
                x = e * e;
            }
        }
        if (!valid) x = 0.0;
        double h = x, l = 0.0, qh = x * x, ql = fma(x, x, -(x * x)), ch = valid ? 1.0 : 0.0, cl = 0.0;
        wave_sum_dd(h, l);
        wave_sum_dd(qh, ql);
        wave_sum_dd(ch, cl);
        if (lane == 0) {
            double *o = out.f + s * kStreamFields;
            o[0] = h;
            o[1] = l;
            o[2] = qh;
            o[3] = ql;
            o[4] = ch + cl;
        }
    }
    const double mn = wave_extreme<false>(leader ? y : INFINITY);
    const double mx = wave_extreme<true>(leader ? y : -INFINITY);
    if (lane == 0) {
        out.ymin = mn;
        out.ymax = mx;
    }
    {
        const uint64_t tot = wave_sum_u64(leader ? cnt0 : 0u);
        if (lane == 0) out.dec[0] = tot;
    }
    for (uint32_t j = 0; j < static_cast<uint32_t>(kBatchMaxD); ++j) {
        uint32_t c = 0u;
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (a0 + k == j) c = cnt[k];
        const uint64_t tot = wave_sum_u64((owner && j < d) ? c : 0u);
        if (lane == 0) out.dec[j + 1] = tot;
    }
    const bool hit = leader && tau != kTauNone;
    const uint64_t tc = wave_sum_u64(hit ? 1u : 0u);
    const uint64_t ts = wave_sum_u64(hit ? tau : 0u);
    if (lane == 0) {
        out.tau_count = tc;
        out.tau_sum = ts;
    }
}

// Sums and (value, index) minima over the 32 lanes of each half wavefront on DPP and the 16-lane row
// swap (wave_dpp.hpp); the FP64 sum keeps the shuffle butterfly (checkpoints only).
__device__ __forceinline__ float half_sum32(float x) { return dpp_sum32(x); }

// The smallest of the first half wavefront's values and its lane, lowest among equal ones. Ordered as
// keys, so -0.0 comes before 0.0; a decision only takes a negative minimum.
__device__ __forceinline__ void first_argmin32(float &g, uint32_t &j)
{
    const uint32_t key = value_key(g), m = __builtin_amdgcn_readfirstlane(dpp_min32(key));
    j = static_cast<uint32_t>(__builtin_ctzll(__builtin_amdgcn_ballot_w64(key == m) | (1ull << 32)));
    g = key_value(m);
}

__device__ __forceinline__ double half_sum32(double x)
{
#pragma unroll
    for (int m = 1; m < 32; m <<= 1) x += __shfl_xor(x, m, 32);
    return x;
}

// One replication per wavefront (every tile of P = 64 lanes, Gaussian noise, N d + 3 <= the
// staging area): lane j < d holds asset j (d <= 32, so the assets sit in the first half wavefront).
// Lane i forms sample i's dot product with v = sz .* w, lane j the sums over the samples of z_ij
// and z_ij (z_i'v); the gradient, its minimum (lowest index among equal values) and g'w are reduced
// over the first half wavefront. Same formulas as the tile kernel, summed in a different order.
// The workgroup's other wavefronts draw the next epochs' normals into LDS (a Philox block per lane at a time);
// one workgroup barrier per epoch hands a buffer over. The normals do not depend on the iterate, so the draw
// leaves the iteration's dependent chain.
//
// The chain is what bounds it (1,024 replications are a wavefront per SIMD). In registers (wave_in_registers) a
// lane takes its sample's row (up to DR assets) and its asset's column (up to NC samples) while the previous
// iteration's reductions run, from one of three buffers drawn two epochs ahead, and v_j and the dot products
// reach the other lanes as scalars: no LDS round trip is left in the chain. DR = 0: rows and columns are read
// from LDS in the iteration, as are v and the dot products; two buffers, one epoch ahead.
// Registers are set out for DR and NC, so more instructions and fewer resident wavefronts: past one or two
// wavefronts per SIMD they lose. us per iteration in registers and from LDS, at 1,024, 2,048 and 3,000
// replications: d = 10, N = 5 0.89, 1.06; 1.15, 1.21; 1.85, 1.45. d = N = 10 0.97, 1.05; 1.32, 1.22; 2.11, 1.49.
// d = 17, N = 8 0.94, 0.98; 1.23, 1.16; 1.99, 1.41. d = 24, N = 12 1.19, 1.22; 1.68, 1.51; 2.59, 1.91. With
// N = 17 to 32 in registers d = 24, N = 24 takes 1.66 at 1,024 and 2.28 at 1,500, from LDS 1.47 and 1.89.
template <int DR, int NC>
__device__ __forceinline__ void run_wave(const BatchBuffers &B, const Tile tile, float *lds)
{
    const InstanceDesc *P = B.inst + tile.inst;
    constexpr bool kAhead = DR > 0;                    // normals drawn two epochs ahead, else one
    const uint32_t lane = threadIdx.x % kWave;
    // the other wavefronts; as a scalar branch in the form from LDS
    const bool drawer = DR ? threadIdx.x >= kWave : __builtin_amdgcn_readfirstlane(threadIdx.x / kWave) != 0;
    const uint32_t r = tile.rep0;
    const uint32_t d = P->d, N = P->N, M = P->M, nd = N * d, nb = (nd + 3) / 4;
    const uint32_t T = static_cast<uint32_t>(P->T);    // at most kMaxBatchT
    const uint32_t k0 = static_cast<uint32_t>(P->seed), k1 = static_cast<uint32_t>(P->seed >> 32);
    const uint32_t dom = P->instance & 0xFFFFFFu;
    const uint32_t n_ckpt = P->n_ckpt;
    const bool logged = lane == 0 && (P->flags & 2u) && (static_cast<uint64_t>(r) - P->log_begin) < P->log_count;
    const uint64_t log_count = P->log_count, log_at = P->dlog_base + (static_cast<uint64_t>(r) - P->log_begin);
    const bool in = lane < d;
    const uint32_t jc = in ? lane : 0u;
    const float sz = in ? P->sz_f[jc] : 0.0f, c1 = P->c1_f[jc], c2 = P->c2_f[jc], mu = P->mu_f[jc];
    const float w0 = (in && P->has_w0) ? P->w0_f[jc] : 0.0f;
    const double sig_d = in ? P->sig_d[jc] : 0.0, mu_d = in ? P->mu_d[jc] : 0.0, lambda = P->lambda;
    const float inv_n = P->inv_n_f, gap_eps = static_cast<float>(P->gap_eps);

    uint32_t S = 0u, cnt = 0u, cnt0 = 0u, hib = 0u;
    uint32_t tau = kTauNone, ck = 0, epoch = 0, m_in_epoch = 0;
    uint32_t next_ckpt = n_ckpt ? static_cast<uint32_t>(P->ckpt[0]) : 0;
    const bool narrow = T <= kMaxNarrowT;              // S stays below 2^32
    float cw_lane = 0.0f;                              // lane i: the scale of w_t = cw S at t = 64 floor(t / 64) + i
    // f(w) at w = c S, FP64 (Eq. (3), diagonal Sigma), summed over the assets' lanes
    auto objective = [&](double c) {
        const double w = (static_cast<double>(S) + (hib ? 4294967296.0 : 0.0)) * c;
        const double sw = sig_d * w;
        const double quad = half_sum32(in ? sw * sw : 0.0);
        const double lin = half_sum32(in ? mu_d * w : 0.0);
        return fma(lambda, quad, -lin);
    };

    // the normals of epoch e into its buffer (e mod 3, or 2), blocks b = first, first + stride, ...
    const uint32_t stage = 4 * nb;
    float *const vs = lds, *const dots = lds + 32, *const zs = DR ? lds : lds + 32 + (N + 3) / 4 * 4;
    float *const buf[3] = {zs, zs + stage, zs + (kAhead ? 2 * stage : 0)};
    auto draw = [&](uint32_t e, float *dst, uint32_t first, uint32_t stride) {
        const PhiloxRow row = philox_row(e, r, k0);
        for (uint32_t b = first; b < nb; b += stride) {
            const Block4<float> q = normals_block_row(row, b, dom, k0, k1);
            dst[4 * b + 0] = q.z[0];
            dst[4 * b + 1] = q.z[1];
            dst[4 * b + 2] = q.z[2];
            dst[4 * b + 3] = q.z[3];
        }
    };
    float *z_now = buf[0], *z_next = buf[1], *z_draw = buf[2];      // epoch, epoch + 1 and, of three, epoch + 2
    draw(0u, z_now, threadIdx.x, blockDim.x);
    if (kAhead && M < T) draw(1u, z_next, threadIdx.x, blockDim.x);
    __syncthreads();

    // sample min(lane, N - 1)'s row, which past d meets zeros of v, and this asset's column, zero past N;
    // what is read past the sample or the buffer is finite (the kernel clears the LDS)
    float row[DR ? DR : 1], col[NC ? NC : 1];
    auto take = [&](const float *zc) {
        const float *zr = zc + min(lane, N - 1) * d, *za = zc + jc;
#pragma unroll
        for (int j = 0; j < DR; ++j) row[j] = zr[j];
#pragma unroll
        for (int i = 0; i < NC; ++i) col[i] = za[i * d];
#pragma unroll
        for (int i = 0; i < NC; ++i) col[i] = static_cast<uint32_t>(i) < N ? col[i] : 0.0f;
    };
    auto scalar = [](float x, int from) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), from)); };
    if (!drawer) take(z_now);

    for (uint32_t t = 0; t < T; ++t) {
        const bool ends = m_in_epoch + 1 == M;          // the epoch's last iteration
        if (drawer) {
            // the buffer drawn into was last read before the previous barrier
            constexpr uint32_t kNext = kAhead ? 2 : 1;
            if (ends && (static_cast<uint64_t>(epoch) + kNext) * M < T)
                draw(epoch + kNext, kAhead ? z_draw : z_next, threadIdx.x - kWave, blockDim.x - kWave);
        } else {
            // the scale 2/(t (t+1)): an FP64 division every 64 iterations instead of one in each one's chain
            const uint32_t tl = t % kWave;
            if (tl == 0) {
                const uint32_t u = t + lane;
                cw_lane = u == 0 ? 0.0f : static_cast<float>(2.0 / (static_cast<double>(u) * (static_cast<double>(u) + 1.0)));
            }
            const float cw = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cw_lane), tl));
            const float w = (t == 0) ? w0
                            : narrow ? static_cast<float>(S) * cw
                                     : (static_cast<float>(S) + (hib ? 4294967296.0f : 0.0f)) * cw;
            const float v = sz * w;
            float s1 = 0.0f, s2 = 0.0f;
            if constexpr (DR > 0) {
                float dot = 0.0f;
#pragma unroll
                for (int j = 0; j < DR; j += 8)
                    if (j == 0 || static_cast<uint32_t>(j) < d) {
#pragma unroll
                        for (int e = 0; e < 8; ++e) dot = fmaf(row[j + e], scalar(v, j + e), dot);
                    }
#pragma unroll
                for (int i = 0; i < NC; i += 8)
                    if (i == 0 || static_cast<uint32_t>(i) < N) {
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            s1 += col[i + e];
                            s2 = fmaf(col[i + e], scalar(dot, i + e), s2);
                        }
                    }
                if (!in) s1 = s2 = 0.0f;
                if (ends && t + 1 < T) take(z_next);
            } else {
                if (lane < 32) vs[lane] = v;
                wave_lds_order();
                for (uint32_t i = lane; i < N; i += kWave) {
                    float dot = 0.0f;
#pragma unroll 8
                    for (uint32_t j = 0; j < d; ++j) dot = fmaf(z_now[i * d + j], vs[j], dot);
                    dots[i] = dot;
                }
                wave_lds_order();
                if (in) {
#pragma unroll 8
                    for (uint32_t i = 0; i < N; ++i) {
                        const float z = z_now[i * d + lane];
                        s1 += z;
                        s2 = fmaf(z, dots[i], s2);
                    }
                }
                wave_lds_order();                           // vs and dots are rewritten next iteration
            }
            const float qn = half_sum32(s1 * v) * inv_n;
            float g = INFINITY;
            uint32_t jg = 0xFFFFFFFFu;
            if (in) g = fmaf(-c1, s1, fmaf(c2, fmaf(-s1, qn, s2), -mu));
            const float g_lane = in ? g * w : 0.0f;
            first_argmin32(g, jg);
            const uint32_t a = (g < 0.0f) ? jg + 1 : 0u;
            if (__builtin_amdgcn_readfirstlane(tau) == kTauNone) {
                const float gap = half_sum32(g_lane) - (g < 0.0f ? g : 0.0f);
                if (gap <= gap_eps) tau = t;
            }
            if (logged) B.dlog[log_at + static_cast<uint64_t>(t) * log_count] = static_cast<uint8_t>(a);
            // step 2/(t+2): the signature absorbs the update
            cnt0 += (a == 0u) ? 1u : 0u;
            if (a == lane + 1) {
                const uint32_t now = S + t + 1;
                if (!narrow && now < S) hib = 1u;
                S = now;
                cnt += 1u;
            }
            if (t + 1 == next_ckpt) {
                const double f = objective(2.0 / (static_cast<double>(t + 1) * static_cast<double>(t + 2)));
                if (lane == 0) B.fck[static_cast<uint64_t>(ck) * B.total_R + P->path_base + r] = f;
                ++ck;
                next_ckpt = ck < n_ckpt ? static_cast<uint32_t>(P->ckpt[ck]) : 0;
            }
        }
        ++m_in_epoch;
        if (ends) {
            __syncthreads();   // all wavefronts: the drawn buffer is complete and the oldest is free
            float *const z = z_now;
            z_now = z_next;
            z_next = kAhead ? z_draw : z;
            z_draw = z;
            m_in_epoch = 0;
            ++epoch;
        }
    }
    if (drawer) return;
    const double y = objective(2.0 / (static_cast<double>(T) * static_cast<double>(T + 1)));

    if (B.y) {
        const uint64_t R = P->R;
        if (lane == 0) {
            B.y[P->path_base + r] = y;
            B.tau[P->path_base + r] = tau;
            B.cnt[P->cnt_base + r] = cnt0;
        }
        if (in) {
            B.cnt[P->cnt_base + (static_cast<uint64_t>(lane) + 1) * R + r] = cnt;
            B.wsum[P->wsum_base + static_cast<uint64_t>(lane) * R + r] =
                static_cast<uint64_t>(S) | (static_cast<uint64_t>(hib) << 32);
        }
    }

    // the tile's partial record (one replication): its streams, extremes, decision totals and tau
    TilePartial &out = B.partials[tile.slot];
    if (lane == 0) {
        for (uint32_t s = 0; s < kTileStreams; ++s) {
            double *o = out.f + s * kStreamFields;
            if (s >= 1 + 2 * n_ckpt) {
                for (int f = 0; f < kStreamFields; ++f) o[f] = 0.0;
                continue;
            }
            double x;
            bool valid = true;
            if (s == 0) {
                x = y;
            } else if (s <= n_ckpt) {
                x = B.fck[static_cast<uint64_t>(s - 1) * B.total_R + P->path_base + r];
            } else {
                const double f = B.fck[static_cast<uint64_t>(s - 1 - n_ckpt) * B.total_R + P->path_base + r];
                valid = (f != 0.0);
                const double e = valid ? (f - y) / f : 0.0;
                x = e * e;
            }
            if (!valid) x = 0.0;
            o[0] = x;
            o[1] = 0.0;
            o[2] = x * x;
            o[3] = fma(x, x, -(x * x));
            o[4] = valid ? 1.0 : 0.0;
        }
        out.ymin = y;
        out.ymax = y;
        out.dec[0] = cnt0;
        out.tau_count = tau != kTauNone ? 1u : 0u;
        out.tau_sum = tau != kTauNone ? tau : 0u;
    }
    if (lane < static_cast<uint32_t>(kBatchMaxD)) out.dec[lane + 1] = in ? cnt : 0u;
}

// One wavefront per tile, every tile of the batch, longest first.
__global__ __launch_bounds__(kWave) void fw_tile_kernel(BatchBuffers B)
{
    __shared__ float stage[kStageFloats + kStagePad];
    __shared__ float coef[kCoefRows][kBatchMaxD];
    const Tile tile = B.tiles[blockIdx.x];
    const uint32_t d = B.inst[tile.inst].d;
    if (tile.Pa == 4) run_tile<4, kLaneAssets>(B, tile, stage, coef);
    else if (tile.Pa == 2) run_tile<2, kLaneAssets>(B, tile, stage, coef);
    else if (d > 6) run_tile<1, 8>(B, tile, stage, coef);
    else if (d > 4) run_tile<1, 6>(B, tile, stage, coef);
    else if (d > 2) run_tile<1, 4>(B, tile, stage, coef);
    else run_tile<1, 2>(B, tile, stage, coef);
}

// One replication per workgroup (a wavefront for the iteration, the others for the next epochs'
// normals), every tile of a batch that qualifies (BatchBuffers.wave_mode). A kernel for each mode: in one,
// the form that reads from LDS has the registers of the other and runs up to 6 % slower. The forms' order in
// the second decides how the compiler lays out the chain: d = N = 10 0.96 us per iteration, others 0.95 to 1.01.
template <class Run>
__device__ __forceinline__ void wave_run(const BatchBuffers &B, float4 *lds4, Run run)
{
    float *const lds = reinterpret_cast<float *>(lds4);
    for (uint32_t i = threadIdx.x; i < B.wave_lds; i += blockDim.x) lds[i] = 0.0f;
    __syncthreads();
    const Tile tile = B.tiles[blockIdx.x];
    run(tile, lds, B.inst[tile.inst].d, B.inst[tile.inst].N);
}

__global__ __launch_bounds__(kWaveMaxThreads) void fw_wave_kernel(BatchBuffers B)
{
    HIP_DYNAMIC_SHARED(float4, lds4)                   // v, dot products, buffers (wave_lds), 16-byte aligned
    wave_run(B, lds4, [&](const Tile &tile, float *lds, uint32_t, uint32_t) { run_wave<0, 0>(B, tile, lds); });
}

__global__ __launch_bounds__(kWaveMaxThreads) void fw_wave_registers_kernel(BatchBuffers B)
{
    HIP_DYNAMIC_SHARED(float4, lds4)
    wave_run(B, lds4, [&](const Tile &tile, float *lds, uint32_t d, uint32_t N) {
        if (d <= 16 && N > 8) run_wave<16, 16>(B, tile, lds);
        else if (d <= 16) run_wave<16, 8>(B, tile, lds);
        else if (N > 8) run_wave<32, 16>(B, tile, lds);
        else run_wave<32, 8>(B, tile, lds);
    });
}

// One workgroup per instance: its tile slots in order.
__global__ __launch_bounds__(kBlock) void fw_batch_reduce(BatchBuffers B)
{
    __shared__ double sm_f[2 * (kBlock / 64)];
    __shared__ uint64_t sm_i[kBlock / 64];
    const uint32_t i = blockIdx.x;
    const uint32_t b0 = B.slot_begin[i], b1 = B.slot_begin[i + 1];
    TilePartial &o = B.final_stats[i];
    for (int s = 0; s < kTileStreams; ++s) {
        double h = 0.0, l = 0.0, qh = 0.0, ql = 0.0, ch = 0.0, cl = 0.0;
        for (uint32_t b = b0 + threadIdx.x; b < b1; b += kBlock) {
            const double *f = B.partials[b].f + s * kStreamFields;
            dd_add(h, l, f[0], f[1]);
            dd_add(qh, ql, f[2], f[3]);
            dd_add(ch, cl, f[4], 0.0);
        }
        block_sum_dd(h, l, sm_f);
        block_sum_dd(qh, ql, sm_f);
        block_sum_dd(ch, cl, sm_f);
        if (threadIdx.x == 0) {
            double *f = o.f + s * kStreamFields;
            f[0] = h;
            f[1] = l;
            f[2] = qh;
            f[3] = ql;
            f[4] = ch + cl;
        }
    }
    double mn = INFINITY, mx = -INFINITY;
    for (uint32_t b = b0 + threadIdx.x; b < b1; b += kBlock) {
        mn = fmin(mn, B.partials[b].ymin);
        mx = fmax(mx, B.partials[b].ymax);
    }
    mn = block_extreme<false>(mn, sm_f);
    mx = block_extreme<true>(mx, sm_f);
    if (threadIdx.x == 0) {
        o.ymin = mn;
        o.ymax = mx;
    }
    for (int j = 0; j < 33 + 2; ++j) {
        uint64_t x = 0;
        for (uint32_t b = b0 + threadIdx.x; b < b1; b += kBlock)
            x += j < 33 ? B.partials[b].dec[j] : (j == 33 ? B.partials[b].tau_count : B.partials[b].tau_sum);
        x = block_sum_u64(x, sm_i);
        if (threadIdx.x == 0) {
            if (j < 33) o.dec[j] = x;
            else if (j == 33) o.tau_count = x;
            else o.tau_sum = x;
        }
    }
}

// A drawing wavefront draws 256 normals a pass: more of them from the second pass on, where the device
// still holds every workgroup at once.
inline uint32_t wave_threads(const BatchBuffers &B)
{
    return B.wave_stage > 256 && B.n_tiles <= kWaveManyDrawers ? kWaveMaxThreads : 2 * kWave;
}

// the tile kernel over every tile, then the per-instance reduction, in stream order
int launch_fw_batch(const BatchBuffers &B, hipStream_t stream)
{
    if (B.n_tiles) {
        if (B.wave_mode) {
            const auto kernel = B.wave_mode == kWaveRegisters ? fw_wave_registers_kernel : fw_wave_kernel;
            hipLaunchKernelGGL(kernel, dim3(B.n_tiles), dim3(wave_threads(B)), sizeof(float) * B.wave_lds, stream, B);
        }
        else hipLaunchKernelGGL(fw_tile_kernel, dim3(B.n_tiles), dim3(kWave), 0, stream, B);
    }
    hipLaunchKernelGGL(fw_batch_reduce, dim3(B.n_inst), dim3(kBlock), 0, stream, B);
    return hipGetLastError() == hipSuccess ? 0 : -3;
}

}  // namespace fw
