// fw_paths_split_narrow.hip -- binary32 Gaussian runs of few replications, up to 16 assets (fw_paths_split.hpp).
#include "fw_paths_split.hpp"

namespace fw {

KernelFn paths_split_narrow(uint32_t d) { return choose_split<1, 16, false>(d); }

}  // namespace fw
