// fw_paths_t_narrow.hip -- binary32 Student-t path kernels, 32-bit signature, up to 16 assets.
#include "fw_paths.hpp"

namespace fw {

KernelChoice paths_t_narrow(uint32_t d) { return choose_exact<1, 16, float, 1, uint32_t, false>(d); }

}  // namespace fw
