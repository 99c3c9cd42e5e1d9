// The split contraction with small output tiles (gemm_small.hpp) and the epilogue over its partials (epi_rows.hpp):
// instantiations and host launchers.
#include "gemm_small.hpp"
#include "epi_rows.hpp"
#include "small_launch.hpp"

namespace coda {

template <class C, bool AK, bool BKC>
static hipError_t launch_partial(const SmallParams &p, hipStream_t s)
{
    hipLaunchKernelGGL((gemm_small_partial<C, AK, BKC>), dim3((unsigned)(p.tiles_m * p.tiles_n * p.nsplit)), dim3(C::NT), 0, s, p);
    return hipGetLastError();
}
template <class C, bool AK, bool BKC>
static hipError_t launch_partial_once(const SmallParams &p, hipStream_t s)
{
    return reads_once<C, BKC>(p, p.nsplit) ? launch_partial<Once<C>, AK, BKC>(p, s) : launch_partial<C, AK, BKC>(p, s);
}
// Rings (measured at N x K = 28672 x 4096 bf16, 235 MB of weights): 32 rows, stages of 20 KB: two 58 us, three 45, four 48,
// seven 50 -- past the ~40 KB in flight that the latency of memory asks for, more only queue up; 64 rows, stages of 24 KB:
// two 62, three 50, six 50.  128 rows: eight waves, one workgroup per CU, four stages of 32 KB (two: 81, four: 58) or, for
// 256 columns, three of 48 KB.
template <bool BKC, bool F8>
static hipError_t launch_tile(const SmallPlan &pl, bool ak, const SmallParams &p, hipStream_t s)
{
    if (pl.bm == 32) return launch_partial_once<SmallCfg<32, 128, 1, 4, 3, F8>, true, BKC>(p, s);
    if (pl.bm == 64) return launch_partial_once<SmallCfg<64, 128, 1, 4, 3, F8>, true, BKC>(p, s);
    if (pl.bn == 256) return ak ? launch_partial<SmallCfg<128, 256, 2, 4, 3, F8>, true, BKC>(p, s) : launch_partial<SmallCfg<128, 256, 2, 4, 3, F8>, false, BKC>(p, s);
    return ak ? launch_partial<SmallCfg<128, 128, 2, 4, 4, F8>, true, BKC>(p, s) : launch_partial<SmallCfg<128, 128, 2, 4, 4, F8>, false, BKC>(p, s);
}

template <class C, bool BKC>
static hipError_t launch_stream_tile(int mode, const GemmParams &g, const SmallParams &p, hipStream_t s)
{
    const dim3 grid((unsigned)(p.tiles_m * p.tiles_n));
    if (mode == EPI_LINEAR)
        hipLaunchKernelGGL((gemm_small_stream<C, BKC, EPI_LINEAR>), grid, dim3(C::NT), 0, s, g, p);
    else
        hipLaunchKernelGGL((gemm_small_stream<C, BKC, EPI_SWIGLU_FWD>), grid, dim3(C::NT), 0, s, g, p);
    return hipGetLastError();
}

template <class C, bool BKC>
static hipError_t launch_stream(int mode, const GemmParams &g, const SmallParams &p, hipStream_t s)
{
    return reads_once<C, BKC>(p, 1) ? launch_stream_tile<Once<C>, BKC>(mode, g, p, s) : launch_stream_tile<C, BKC>(mode, g, p, s);
}

// Three stages (four: 46.2 us at 1 x 28672 x 4096, three 43.1: more in flight only queues up); 64 rows in four waves of 32 x 64 (two of
// 64 x 64: 1 to 5 % slower).
template <bool BKC, bool F8>
static hipError_t launch_fused(int bm, int mode, const GemmParams &g, const SmallParams &p, hipStream_t s)
{
    return bm == 32 ? launch_stream<SmallCfg<32, 128, 1, 2, 3, F8>, BKC>(mode, g, p, s) : launch_stream<SmallCfg<64, 128, 2, 2, 3, F8>, BKC>(mode, g, p, s);
}

template <int EPI>
static hipError_t launch_rows(const GemmParams &p, const float *part, int nsplit, hipStream_t s)
{
    if constexpr (EPI == EPI_RMSNORM_BWD)
        hipLaunchKernelGGL((epi_cols_kernel<EPI>), dim3((unsigned)((p.N + EPI_COLS - 1) / EPI_COLS), (unsigned)((p.M + 255) / 256)), dim3(1024), 0, s, p, part, nsplit);
    else
        hipLaunchKernelGGL((epi_rows_kernel<EPI>), dim3((unsigned)((p.N + 255) / 256), (unsigned)((p.M + EPI_ROWS - 1) / EPI_ROWS)), dim3(256), 0, s, p,
                           part, nsplit);
    return hipGetLastError();
}

static SmallParams small_params(const GemmParams &p, bool f8, int chain, int rot_cols)
{
    const int64_t esz = f8 ? 1 : 2;
    SmallParams q{};
    q.A = reinterpret_cast<const unsigned char *>(p.A);
    q.B = reinterpret_cast<const unsigned char *>(p.B);
    q.lda = p.lda * esz;
    q.ldb = p.ldb * esz;
    q.M = p.M; q.N = p.N; q.K = p.K;
    q.chain = chain;
    q.rot_cols = rot_cols;
    return q;
}

hipError_t launch_gemm_small(const SmallPlan &pl, int mode, bool f8, bool ak, bool bkc, const GemmParams &p, int chain, float *part, hipStream_t s)
{
    SmallParams q = small_params(p, f8, chain, (int)PLAN_TILE_N);
    q.tiles_m = (p.M + pl.bm - 1) / pl.bm;
    q.tiles_n = (p.N + pl.bn - 1) / pl.bn;
    q.nsplit = pl.nsplit;
    q.part = part;
    if (pl.fused) return f8 ? (bkc ? launch_fused<true, true>(pl.bm, mode, p, q, s) : launch_fused<false, true>(pl.bm, mode, p, q, s))
                            : (bkc ? launch_fused<true, false>(pl.bm, mode, p, q, s) : launch_fused<false, false>(pl.bm, mode, p, q, s));
    const hipError_t e = f8 ? (bkc ? launch_tile<true, true>(pl, ak, q, s) : launch_tile<false, true>(pl, ak, q, s))
                            : (bkc ? launch_tile<true, false>(pl, ak, q, s) : launch_tile<false, false>(pl, ak, q, s));
    if (e != hipSuccess) return e;
    switch (mode) {
    case EPI_LINEAR: return launch_rows<EPI_LINEAR>(p, part, pl.nsplit, s);
    case EPI_SWIGLU_FWD: return launch_rows<EPI_SWIGLU_FWD>(p, part, pl.nsplit, s);
    case EPI_SWIGLU_BWD: return launch_rows<EPI_SWIGLU_BWD>(p, part, pl.nsplit, s);
    case EPI_RMSNORM_BWD: return launch_rows<EPI_RMSNORM_BWD>(p, part, pl.nsplit, s);
    default: return launch_rows<EPI_ACCUM>(p, part, pl.nsplit, s);
    }
}

hipError_t launch_gemm_direct(int tile, int mode, bool f8, bool ak, bool bkc, const GemmParams &p, int chain, int rot_cols, hipStream_t s)
{
    const SmallParams q = small_params(p, f8, chain, rot_cols);
    if (f8)
        return ak ? (bkc ? launch_small_direct<true, true, true>(tile, mode, p, q, s) : launch_small_direct<true, true, false>(tile, mode, p, q, s))
                  : (bkc ? launch_small_direct<true, false, true>(tile, mode, p, q, s) : launch_small_direct<true, false, false>(tile, mode, p, q, s));
    return ak ? (bkc ? launch_small_direct<false, true, true>(tile, mode, p, q, s) : launch_small_direct<false, true, false>(tile, mode, p, q, s))
              : (bkc ? launch_small_direct<false, false, true>(tile, mode, p, q, s) : launch_small_direct<false, false, false>(tile, mode, p, q, s));
}

}  // namespace coda
