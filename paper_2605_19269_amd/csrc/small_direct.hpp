// small_direct.hpp -- launchers of the undivided small-tile kernels (gemm_small.hpp), instantiated per operand type and
// per layout of B in gemm_direct_inst_*.hip.
#pragma once
#include "gemm_small.hpp"
#include "small_launch.hpp"

namespace coda {

template <class C, bool AK, bool BKC, int EPI, bool CHAINS>
static hipError_t launch_direct(const GemmParams &g, SmallParams p, hipStream_t s)
{
    p.tiles_m = (p.M + C::BM - 1) / C::BM;
    p.tiles_n = (p.N + C::BN - 1) / C::BN;
    p.nsplit = 1;
    hipLaunchKernelGGL((gemm_small_direct<C, AK, BKC, EPI, CHAINS>), dim3((unsigned)(p.tiles_m * p.tiles_n)), dim3(C::NT), 0, s, g, p);
    return hipGetLastError();
}

// 64x256 and 128x256 without chains where there is one only (2 to 3 % at 128x256).
template <class C, bool AK, bool BKC, int EPI>
static hipError_t launch_wide(const GemmParams &g, const SmallParams &p, hipStream_t s)
{
    return p.chain == INT32_MAX ? launch_direct<C, AK, BKC, EPI, false>(g, p, s) : launch_direct<C, AK, BKC, EPI, true>(g, p, s);
}

template <bool F8, bool AK, bool BKC, int EPI>
static hipError_t direct_tile(int tile, const GemmParams &g, const SmallParams &p, hipStream_t s)
{
    if constexpr (AK && (EPI == EPI_LINEAR || EPI == EPI_SWIGLU_FWD))
        if (tile == DIRECT_64x64) return launch_direct<SmallCfg<64, 64, 2, 1, 4, F8>, AK, BKC, EPI, true>(g, p, s);
    if constexpr (AK && EPI == EPI_LINEAR) {
        if (tile == DIRECT_32x256) return launch_direct<SmallCfg<32, 256, 1, 4, 4, F8>, AK, BKC, EPI, false>(g, p, s);
        if (tile == DIRECT_64x256) return launch_wide<SmallCfg<64, 256, 2, 4, 3, F8>, AK, BKC, EPI>(g, p, s);
    }
    if constexpr (EPI == EPI_ACCUM)
        if (tile == DIRECT_128x128_PAIR) return launch_direct<SmallCfg<128, 128, 2, 2, 2, F8>, AK, BKC, EPI, false>(g, p, s);
    if constexpr (F8 && AK && (EPI == EPI_LINEAR || EPI == EPI_SWIGLU_FWD))
        if (tile == DIRECT_128x128 && reads_once<SmallCfg<128, 128, 4, 2, 4, F8>, BKC>(p, 1))
            return launch_direct<Once<SmallCfg<128, 128, 4, 2, 4, F8>>, AK, BKC, EPI, true>(g, p, s);
    if (tile == DIRECT_128x128) return launch_direct<SmallCfg<128, 128, 4, 2, 4, F8>, AK, BKC, EPI, true>(g, p, s);
    if (tile == DIRECT_128x256) return launch_wide<SmallCfg<128, 256, 2, 4, 3, F8>, AK, BKC, EPI>(g, p, s);
    return hipErrorInvalidConfiguration;             // a tile that the plan does not give this program
}

template <bool F8, bool AK, bool BKC>
hipError_t launch_small_direct(int tile, int mode, const GemmParams &g, const SmallParams &p, hipStream_t s)
{
    switch (mode) {
    case EPI_LINEAR: return direct_tile<F8, AK, BKC, EPI_LINEAR>(tile, g, p, s);
    case EPI_SWIGLU_FWD: return direct_tile<F8, AK, BKC, EPI_SWIGLU_FWD>(tile, g, p, s);
    case EPI_SWIGLU_BWD: return direct_tile<F8, AK, BKC, EPI_SWIGLU_BWD>(tile, g, p, s);
    default: return direct_tile<F8, AK, BKC, EPI_ACCUM>(tile, g, p, s);
    }
}

}  // namespace coda
