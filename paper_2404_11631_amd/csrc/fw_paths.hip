// fw_paths.hip -- the launch of the one-lane-per-replication kernels (fw_paths.hpp).
#include "fw_paths_split.hpp"

namespace fw {

// The statistics of a run whose paths left records (fw_paths_split.hpp).
__global__ __launch_bounds__(kBlock) void fw_paths_reduce_kernel(const InstanceDesc *__restrict__ P, RunBuffers B)
{
    __shared__ double sm_f[2 * (kBlock / 64)];
    __shared__ uint64_t sm_i[kBlock / 64];
    __shared__ uint32_t sm_last;
    const uint64_t R = P->R, r = static_cast<uint64_t>(blockIdx.x) * kBlock + threadIdx.x;
    const bool active = r < R;
    reduce_paths(P, B, r, active, static_cast<int>(P->d), active ? B.rec_y[r] : 0.0, active ? B.rec_tau[r] : kTauNone,
                 [&](int j) { return B.rec_cnt[static_cast<uint64_t>(j) * R + r]; }, sm_f, sm_i, &sm_last);
}

// drawing wavefronts of a workgroup
static int split_draw(const InstanceDesc &desc, bool fp64)
{
    return !fp64 && !(desc.flags & 4u) && desc.d >= kSplitSevenFrom && desc.R <= kSplitRepsSeven ? 7 : 3;
}

static KernelFn split_kernel(const InstanceDesc &desc, bool fp64)
{
    if (fp64) return paths_split_fp64(desc.d);
    const int draw = split_draw(desc, false);
    return desc.flags & 4u ? paths_split_features(desc.d)
           : desc.d <= 16  ? paths_split_narrow(desc.d, draw)
                           : paths_split_broad(desc.d, draw);
}

static uint32_t split_grid(const InstanceDesc &desc) { return static_cast<uint32_t>((desc.R + 63) / 64); }

bool paths_split_applies(const InstanceDesc &desc, bool fp64, bool sched, int device)
{
    if (sched || desc.noise != 0 || desc.d > (fp64 ? 16u : 32u) || desc.T > kMaxNarrowT) return false;
    const bool own_kernel = desc.d <= 6 || desc.d == 8 || desc.d == 10 || desc.d == 12 || desc.d == 16;    // in binary64
    const bool odd = desc.d == 5 || (desc.d == 3 && desc.N > 4);
    const uint64_t most = fp64 ? (!own_kernel ? kSplitReps64Generic : desc.d <= 8 && !odd ? kSplitReps64 : kSplitReps64Wide)
                               : (desc.d == 2 ? kSplitRepsTwo : kSplitReps);
    if (desc.R > most || (fp64 ? (desc.flags & 4u) != 0 : desc.d < 2)) return false;
    int cus = 0, per_cu = 0;
    return hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) == hipSuccess &&
           hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void *>(split_kernel(desc, fp64)),
                                                        64 * (split_draw(desc, fp64) + 1), 0) ==
               hipSuccess &&
           static_cast<uint64_t>(cus) * static_cast<uint64_t>(per_cu) >= split_grid(desc);
}

// Returns 0 and launches, or a negative code: -5 unsupported shape, -3 launch failure.
// Feature-writing kernels exist for binary32 state and the 32-bit signature (T <= 92681).
int launch_fw_paths(const InstanceDesc &host_desc, const InstanceDesc *dev_desc, const RunBuffers &B,
                    bool fp64, hipStream_t stream, int *kernel_width)
{
    const bool wide = host_desc.T > kMaxNarrowT;
    const bool feat = (host_desc.flags & 4u) != 0;
    const uint32_t d = host_desc.d, noise = host_desc.noise;
    KernelChoice kc{nullptr, 0, false};
    if (B.rec_y) {
        if (kernel_width) *kernel_width = static_cast<int>(d);
        hipLaunchKernelGGL(split_kernel(host_desc, fp64), dim3(split_grid(host_desc)), dim3(64 * (split_draw(host_desc, fp64) + 1)), 0, stream, dev_desc, B);
        hipLaunchKernelGGL(fw_paths_reduce_kernel, dim3(B.nblocks), dim3(kBlock), 0, stream, dev_desc, B);
        return hipGetLastError() == hipSuccess ? 0 : -3;
    }
    if (feat) {
        if (fp64 || wide || B.sched_n) return -5;
        kc = paths_features(d, noise);
    } else if (B.sched_n) {
        kc = paths_sched(d, noise, fp64, wide);
    } else if (fp64) {
        kc = paths_fp64(d, noise, wide);
    } else if (wide) {
        kc = paths_long(d, noise);
    } else if (noise == 0) {
        kc = d <= 16 ? paths_gauss_narrow(d) : paths_gauss_broad(d);
    } else {
        kc = d <= 16 ? paths_t_narrow(d) : paths_t_broad(d);
    }
    if (!kc.fn) return -5;
    if (kernel_width) *kernel_width = kc.D;
    hipLaunchKernelGGL(kc.fn, dim3(B.nblocks), dim3(kBlock), 0, stream, dev_desc, B);
    return hipGetLastError() == hipSuccess ? 0 : -3;
}

}  // namespace fw
