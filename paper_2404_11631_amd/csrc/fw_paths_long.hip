// fw_paths_long.hip -- binary32 path kernels with the 64-bit signature (T > 92681).
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

KernelChoice paths_long(uint32_t d, uint32_t noise)
{
    return noise == 0 ? choose_gauss<float, uint64_t>(d) : choose_generic<float, 1, uint64_t, false, false>(d);
}

}  // namespace fw
