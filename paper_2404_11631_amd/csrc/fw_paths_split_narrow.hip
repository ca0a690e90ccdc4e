// fw_paths_split_narrow.hip -- binary32 Gaussian runs of few replications, up to 16 assets (fw_paths_split.hpp).
#include "fw_paths_split.hpp"

namespace fw {

KernelFn paths_split_narrow(uint32_t d, int draw) { return draw > 3 ? choose_split<kSplitSevenFrom, 16, false, 7>(d) : choose_split<2, 16, false, 3>(d); }

}  // namespace fw
