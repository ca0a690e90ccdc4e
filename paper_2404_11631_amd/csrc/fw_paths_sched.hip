// fw_paths_sched.hip -- path kernels with per-epoch sample sizes.
#include "fw_paths.hpp"

namespace fw {

template <typename Real, typename WS>
static KernelChoice choose_sched(uint32_t d, uint32_t noise)
{
    return noise == 0 ? choose_generic<Real, 0, WS, false, true>(d) : choose_generic<Real, 1, WS, false, true>(d);
}

KernelChoice paths_sched(uint32_t d, uint32_t noise, bool fp64, bool wide)
{
    if (fp64) return wide ? choose_sched<double, uint64_t>(d, noise) : choose_sched<double, uint32_t>(d, noise);
    return wide ? choose_sched<float, uint64_t>(d, noise) : choose_sched<float, uint32_t>(d, noise);
}

}  // namespace fw
