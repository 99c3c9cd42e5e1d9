// small_launch.hpp -- host entries of the small-tile kernels (gemm_small_inst.hip, gemm_direct_inst_*.hip).
#pragma once
#include "gemm_kernel.hpp"
#include "splitk_plan.hpp"

namespace coda {

struct SmallParams;

// chain, rot_cols: see SmallParams; chain INT32_MAX: one chain
// divided along K: partials to `part`, then the epilogue kernel
hipError_t launch_gemm_small(const SmallPlan &pl, int mode, bool f8, bool ak, bool bkc, const GemmParams &p, int chain, float *part, hipStream_t s);

// undivided, one kernel; mode: any but EPI_RMSNORM_BWD; tile: a DirectTile the mode has
hipError_t launch_gemm_direct(int tile, int mode, bool f8, bool ak, bool bkc, const GemmParams &p, int chain, int rot_cols, hipStream_t s);

template <bool F8, bool AK, bool BKC>
hipError_t launch_small_direct(int tile, int mode, const GemmParams &g, const SmallParams &p, hipStream_t s);

}  // namespace coda
