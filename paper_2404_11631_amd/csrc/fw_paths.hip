// fw_paths.hip -- the launch of the one-lane-per-replication kernels (fw_paths.hpp).
#include "fw_paths.hpp"

namespace fw {

// Returns 0 and launches, or a negative code: -5 unsupported shape, -3 launch failure.
// Feature-writing kernels exist for binary32 state and the 32-bit signature (T <= 92681).
int launch_fw_paths(const InstanceDesc &host_desc, const InstanceDesc *dev_desc, const RunBuffers &B,
                    bool fp64, hipStream_t stream, int *kernel_width)
{
    const bool wide = host_desc.T > kMaxNarrowT;
    const bool feat = (host_desc.flags & 4u) != 0;
    const uint32_t d = host_desc.d, noise = host_desc.noise;
    KernelChoice kc{nullptr, 0, false};
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
