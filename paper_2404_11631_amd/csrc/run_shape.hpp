// run_shape.hpp -- sizes shared by the cooperative runs (fw_newsvendor_run.hip, fw_wide_run.hip) and
// their hosts.
#pragma once

#include <stdint.h>

namespace fw {

// 64-bit words per workgroup for its vertex word: a 64-byte line for each parity. Workgroups that
// share a line slow one another's stores and polls: 157 of them exchange a word in 1.6 us at a line
// each, in 2.5 us at 8 bytes each.
constexpr uint32_t kRunLine = 16;
constexpr uint32_t kRunSteps = 1024;            // iterations per launch at most (the length of the logs)

// What a launcher of a cooperative run returns when the runtime refuses the launch; the host then takes the
// launch-by-launch form from the start.
constexpr int kRunRefused = 1;

}  // namespace fw
