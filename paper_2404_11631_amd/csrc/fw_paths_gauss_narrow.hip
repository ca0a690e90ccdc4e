// fw_paths_gauss_narrow.hip -- binary32 Gaussian path kernels, 32-bit signature, up to 16 assets.
#include "fw_paths.hpp"

namespace fw {

KernelChoice paths_gauss_narrow(uint32_t d) { return choose_exact<1, 16, float, 0, uint32_t, false>(d); }

}  // namespace fw
