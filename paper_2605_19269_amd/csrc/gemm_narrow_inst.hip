// 256 x 192 tiles (gemm_kernel.hpp): instantiations and host launcher.
#include "gemm_launch.hpp"
#include "narrow_launch.hpp"

namespace coda {

using NarrowCfg = DlCfg<256, 192, 2, 4, 4>;
static_assert(NarrowCfg::BN == NARROW_TILE_N, "the plan counts the kernel's tiles");

template <int EPI>
static hipError_t launch(const GemmParams &p, hipStream_t s)
{
    using C = NarrowCfg;
    const dim3 grid((unsigned)(p.tiles_m * p.tiles_n));
    if (p.M % C::BM || p.N % C::BN || p.K % TILE_K)
        hipLaunchKernelGGL((gemm_kernel_narrow<C, EPI, true>), grid, dim3(C::NT), 0, s, p);
    else
        hipLaunchKernelGGL((gemm_kernel_narrow<C, EPI, false>), grid, dim3(C::NT), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_gemm_narrow(int mode, const GemmParams &p_in, hipStream_t s)
{
    GemmParams p = p_in;
    p.tiles_m = (p.M + NarrowCfg::BM - 1) / NarrowCfg::BM;
    p.tiles_n = (p.N + NarrowCfg::BN - 1) / NarrowCfg::BN;
    switch (mode) {
    case EPI_LINEAR: return launch<EPI_LINEAR>(p, s);
    case EPI_SWIGLU_FWD: return launch<EPI_SWIGLU_FWD>(p, s);
    default: return hipErrorInvalidConfiguration;    // the plan gives no other program these tiles
    }
}

}  // namespace coda
