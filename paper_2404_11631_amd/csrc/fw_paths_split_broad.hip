// fw_paths_split_broad.hip -- the same from 17 assets on (fw_paths_split.hpp).
#include "fw_paths_split.hpp"

namespace fw {

KernelFn paths_split_broad(uint32_t d) { return choose_split<17, 32, false>(d); }

}  // namespace fw
