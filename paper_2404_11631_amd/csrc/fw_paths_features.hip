// fw_paths_features.hip -- path kernels that write the control-variate features.
#include "fw_paths.hpp"

namespace fw {

KernelChoice paths_features(uint32_t d, uint32_t noise)
{
    if (noise != 0) return choose_generic<float, 1, uint32_t, true, false>(d);
    return choose_exact<1, 32, float, 0, uint32_t, true>(d);
}

}  // namespace fw
