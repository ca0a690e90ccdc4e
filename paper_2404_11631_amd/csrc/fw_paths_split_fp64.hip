// fw_paths_split_fp64.hip -- binary64 Gaussian runs of few replications (fw_paths_split.hpp).
#include "fw_paths_split.hpp"

namespace fw {

KernelFn paths_split_fp64(uint32_t d) { return choose_split<1, 16, false, 3, double>(d); }

}  // namespace fw
