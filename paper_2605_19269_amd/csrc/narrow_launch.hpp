// narrow_launch.hpp -- host entry of the 256 x 192 tiles (gemm_narrow_inst.hip).
#pragma once
#include "gemm_kernel.hpp"
#include "splitk_plan.hpp"

namespace coda {

// bf16, A [M x K], B [K x N], nothing shared; mode: EPI_LINEAR without row reductions, EPI_SWIGLU_FWD
hipError_t launch_gemm_narrow(int mode, const GemmParams &p, hipStream_t s);

}  // namespace coda
