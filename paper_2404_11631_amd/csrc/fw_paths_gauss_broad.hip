// fw_paths_gauss_broad.hip -- binary32 Gaussian path kernels, 32-bit signature, 17 to 32 assets.
#include "fw_paths.hpp"

namespace fw {

KernelChoice paths_gauss_broad(uint32_t d) { return choose_exact<17, 32, float, 0, uint32_t, false>(d); }

}  // namespace fw
