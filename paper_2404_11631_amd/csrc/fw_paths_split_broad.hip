// fw_paths_split_broad.hip -- the same from 17 assets on (fw_paths_split.hpp).
#include "fw_paths_split.hpp"

namespace fw {

KernelFn paths_split_broad(uint32_t d, int draw) { return draw > 3 ? choose_split<17, 32, false, 7>(d) : choose_split<17, 32, false, 3>(d); }

}  // namespace fw
