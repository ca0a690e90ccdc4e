// newsvendor_device.hpp -- the general-constraint newsvendor's arithmetic shared by its kernels
// (fw_newsvendor.hip, fw_newsvendor_lp_run.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fw {

// x + gamma (s - x) with each operation rounded on its own (contraction into a fused multiply-add is
// off here), so that any other implementation of the same formula in FP64 gets the same bits.
__device__ __forceinline__ double nv_lp_move(double x, double s, double gamma)
{
#pragma clang fp contract(off)
    const double step = gamma * (s - x);
    return x + step;
}

// Eq. (9): (k - v) + ((h + v) count) / S, each operation rounded on its own.
__device__ __forceinline__ double nv_lp_grad(double km, double hv, uint32_t count, uint32_t S)
{
#pragma clang fp contract(off)
    const double part = (hv * static_cast<double>(count)) / static_cast<double>(S);
    return km + part;
}

}  // namespace fw
