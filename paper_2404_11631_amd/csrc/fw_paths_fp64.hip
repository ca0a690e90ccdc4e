// fw_paths_fp64.hip -- binary64 path kernels.
#include "fw_paths.hpp"

namespace fw {

// the widths of the named workloads, and the generic kernel for the others
template <typename Real, typename WS>
static KernelChoice choose_gauss(uint32_t d)
{
    KernelChoice kc = choose_exact<1, 6, Real, 0, WS, false>(d);
    if (d == 8) kc = choose_exact<8, 8, Real, 0, WS, false>(d);
    if (d == 10) kc = choose_exact<10, 10, Real, 0, WS, false>(d);
    if (d == 12) kc = choose_exact<12, 12, Real, 0, WS, false>(d);
    if (d == 16) kc = choose_exact<16, 16, Real, 0, WS, false>(d);
    return kc.fn ? kc : choose_generic<Real, 0, WS, false, false>(d);
}

KernelChoice paths_fp64(uint32_t d, uint32_t noise, bool wide)
{
    if (noise == 0) return wide ? choose_gauss<double, uint64_t>(d) : choose_gauss<double, uint32_t>(d);
    return wide ? choose_generic<double, 1, uint64_t, false, false>(d) : choose_generic<double, 1, uint32_t, false, false>(d);
}

}  // namespace fw
