// small_launch.hpp -- host entry of the split contraction with small tiles (gemm_small_inst.hip).
#pragma once
#include "gemm_kernel.hpp"
#include "splitk_plan.hpp"

namespace coda {
hipError_t launch_gemm_small(const SmallPlan &pl, int mode, bool f8, bool ak, bool bkc, const GemmParams &p, float *part, hipStream_t s);
}  // namespace coda
