// exchange.hpp -- values passed between the workgroups of one cooperative launch.
//
// A chain of dependent launches costs ~2.7 us per launch on gfx950 before any work; the iterations
// of the single-replication paths are such chains. Inside one launch a workgroup publishes a value
// as one 64-bit word, the value in the high half and the iteration's tag in the low one, stored and
// loaded with relaxed agent-scope atomics: a reader that sees the tag has the value of the same
// store, so no fence is needed (a release fence writes back the whole L2 of an XCD, which made a
// counter-based form five times slower than the launches it replaced), and the reader's poll is the
// only wait. A slot may be overwritten once every reader is known to be done with it. Where a workgroup
// publishes iteration t + 1 only after it has read every value of iteration t, two buffers by the iteration's
// parity do: the vertex words (each workgroup's on a 64-byte line of its own), the wide run's dots, the
// constraint run's counts and vertex (which share lines) and the SQN run's row sums. The SQN run's other
// blocks are single; why that is enough stands at SqnSplitSlots.
//
// Every wait is bounded: a poll that does not see its tag within kPollLimit rounds (about a second,
// where a value arrives within microseconds) gives up, the workgroup raises the run's failure word and
// leaves, and the others follow by their own limits; the host reports the failure or runs the
// launch-by-launch form. The launches are cooperative, so all workgroups are resident together.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "run_shape.hpp"
#include "wave_dpp.hpp"

namespace fw {

// A cooperative launch of kernel fn: 0, or kRunRefused. The occupancy that the fit rules ask for is the
// whole device's; the stream may hold less of it.
static inline int launch_cooperative(const void *fn, dim3 grid, int threads, void **args, size_t lds, hipStream_t s)
{
    if (hipLaunchCooperativeKernel(fn, grid, dim3(threads), args, static_cast<unsigned>(lds), s) == hipSuccess) return 0;
    (void)hipGetLastError();                            // or the next launch's check would report it
    return kRunRefused;
}

#ifndef FW_POLL_LIMIT
#define FW_POLL_LIMIT (1u << 20)
#endif
constexpr uint32_t kPollLimit = FW_POLL_LIMIT;

__device__ __forceinline__ void exchange_put(uint64_t *slot, uint32_t value, uint32_t tag)
{
    __hip_atomic_store(slot, (static_cast<uint64_t>(value) << 32) | tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint64_t exchange_get(const uint64_t *slot)
{
    return __hip_atomic_load(const_cast<uint64_t *>(slot), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint32_t failure_get(const uint32_t *fail)
{
    return __hip_atomic_load(const_cast<uint32_t *>(fail), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void failure_raise(uint32_t *fail)
{
    __hip_atomic_store(fail, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The smallest key over the wavefront and the lowest index among the lanes that hold it; with SORTED
// the lanes' indices ascend and the first such lane has it.
template <bool SORTED>
__device__ __forceinline__ void wave_min_key(uint32_t &key, uint32_t &j)
{
    const uint32_t m = dpp_min64(key);
    if constexpr (SORTED)
        j = __builtin_amdgcn_readlane(j, __builtin_ctzll(__builtin_amdgcn_ballot_w64(key == m)));
    else
        j = dpp_min64(key == m ? j : 0xFFFFFFFFu);
    key = m;
}

// A workgroup's smallest value, its index (24 bits) and 8 bits of the tag in one word.
__device__ __forceinline__ void vertex_put(uint64_t *lines, uint32_t g, uint64_t t, uint32_t key, uint32_t j)
{
    exchange_put(lines + static_cast<size_t>(g) * kRunLine + 8 * (t & 1), key, (j << 8) | ((static_cast<uint32_t>(t) + 1u) & 0xFFu));
}

// The smallest (key, index) over the nwg workgroups' words of iteration t, by a workgroup of BLOCK threads
// with one barrier; st holds a word per wavefront. `fail` (LDS) is set when a word did not come, before
// the barrier. All threads get the result: key in the high half, index (0xFFFFFF: none) in the low.
template <int BLOCK>
__device__ __forceinline__ uint64_t vertex_get(const uint64_t *lines, uint32_t nwg, uint64_t t, uint64_t *st, uint32_t *fail)
{
    const uint32_t tag = static_cast<uint32_t>(t) + 1u;
    uint32_t key = 0xFFFFFFFFu, j = 0xFFFFFFFFu;
    bool seen = true;
    for (uint32_t i = threadIdx.x; i < nwg; i += BLOCK) {
        const uint64_t *slot = lines + static_cast<size_t>(i) * kRunLine + 8 * (t & 1);
        uint64_t w = exchange_get(slot);
        for (uint32_t polls = 0; ((static_cast<uint32_t>(w) ^ tag) & 0xFFu) != 0u; w = exchange_get(slot))
            if (++polls == kPollLimit) {
                seen = false;
                break;
            }
        const uint32_t xk = static_cast<uint32_t>(w >> 32), xj = static_cast<uint32_t>(w) >> 8;
        if (xk < key || (xk == key && xj < j)) {
            key = xk;
            j = xj;
        }
    }
    if (!seen) *fail = 1u;
    wave_min_key<false>(key, j);
    if ((threadIdx.x & 63u) == 0u) st[threadIdx.x / 64] = (static_cast<uint64_t>(key) << 32) | j;
    __syncthreads();
    uint64_t m = st[0];
#pragma unroll
    for (int w = 1; w < BLOCK / 64; ++w) m = min(m, st[w]);
    return m;
}

// What a cooperative launch leaves for the gap, tau and the decision counts, and the launch that takes
// them from it, an iteration per workgroup.
struct RunLog {
    const float *gx;            // [steps][R][nwg] the workgroups' parts of g'x
    const float *best;          // [steps][R] smallest value of the linear subproblem
    uint32_t nwg, R, n;
    float scale, gap_eps;       // gap = g'x - min(0, scale best)
    uint64_t t0, T;
    const uint32_t *fail;       // the run's failure word: a run that gave up left no log
    const uint32_t *dec;        // [R][T]
    uint32_t *tau;              // [R]
    uint32_t *cnt;              // [R][n + 1]
};

// 256 threads, the sum in the order of the launch-per-iteration kernels: strided over the threads,
// the wavefront's butterfly, the wavefronts in order.
static __global__ __launch_bounds__(256) void run_log_kernel(RunLog L)
{
    __shared__ float sm[4];
    const uint32_t tid = threadIdx.x, r = blockIdx.y;
    if (*L.fail) return;
    const uint64_t row = static_cast<uint64_t>(blockIdx.x) * L.R + r;
    float gs = 0.0f;
    for (uint32_t i = tid; i < L.nwg; i += 256) gs += L.gx[row * L.nwg + i];
    gs = dpp_sum64(gs);
    if (tid % 64 == 0) sm[tid / 64] = gs;
    __syncthreads();
    if (tid == 0) {
        float gsum = sm[0];
        for (int w = 1; w < 4; ++w) gsum += sm[w];
        const float best = L.best[row];
        const float gap = gsum - (best < 0.0f ? L.scale * best : 0.0f);
        const uint64_t t = L.t0 + blockIdx.x;
        // kTauNone is the largest value: the minimum is the first iteration at or below the threshold
        if (gap <= L.gap_eps) atomicMin(L.tau + r, static_cast<uint32_t>(t));
        const uint32_t a = L.dec[static_cast<uint64_t>(r) * L.T + t];
        if (a <= L.n) atomicAdd(L.cnt + static_cast<uint64_t>(r) * (L.n + 1) + a, 1u);
    }
}

static inline int launch_run_log(const RunLog &L, uint64_t steps, hipStream_t s)
{
    hipLaunchKernelGGL(run_log_kernel, dim3(static_cast<uint32_t>(steps), L.R), dim3(256), 0, s, L);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace fw
