// fw_paths_split_features.hip -- the same with control-variate features (fw_paths_split.hpp).
#include "fw_paths_split.hpp"

namespace fw {

KernelFn paths_split_features(uint32_t d) { return choose_split<2, 32, true, 3>(d); }

}  // namespace fw
