// epi_rows.hpp -- the epilogue program on a contraction that lies in the workspace as `nsplit` fp32 partial matrices
// [nsplit][M][N] (gemm_small.hpp): adds the partials up in range order and applies the program of GemmParams.
//
// One wave owns one row of a 256-column block, a lane four consecutive columns: loads and stores are row-contiguous
// without staging, the pairwise maps stay inside a lane, and a block's row reduction -- the 256-column granularity that
// the callers' partial buffers have -- is one wave reduction in a fixed order.  M / 4 x N / 256 workgroups, so even a
// few rows spread over the chip.  Bound by reading the partials (from the memory-side cache, where the first kernel left them):
// 509 x 2048 in four ranges, 21 MB with the residual and the result, 5.2 us; with one row by the latency of a few loads, 3.8 us.
//
// RMSNORM_BWD also reduces over the columns of 256-row blocks: there a workgroup owns 256 rows x 32 columns, 8 lanes a row.
#pragma once
#include "gemm_kernel.hpp"

namespace coda {

// The ranges' partials of four columns of R rows, each row's added up in range order, R * W loads in flight: with few rows there is
// nothing else to hide a load's latency under (4096 columns of 8 ranges, one row: 4.0 us with the last three loaded one by one).
template <int W, int R>
__device__ __forceinline__ void sum_parts_by(f32x4 (&v)[R], const float *const (&part)[R], int nsplit, int64_t stride)
{
    for (int s = 0; s < nsplit; s += W) {
        f32x4 t[R][W];
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int q = 0; q < W; ++q) t[r][q] = *reinterpret_cast<const f32x4 *>(part[r] + (s + q < nsplit ? s + q : nsplit - 1) * stride);
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int q = 0; q < W; ++q)
                if (s + q < nsplit) v[r] = s + q == 0 ? t[r][q] : v[r] + t[r][q];
    }
}
// No more loads than ranges, rounded up to 2, 4 or 8 (always eight: 509 x 2048 in four ranges 5.5 us, here 5.2)
template <int R>
__device__ __forceinline__ void sum_parts(f32x4 (&v)[R], const float *const (&part)[R], int nsplit, int64_t stride)
{
    if (nsplit <= 2) sum_parts_by<2>(v, part, nsplit, stride);
    else if (nsplit <= 4) sum_parts_by<4>(v, part, nsplit, stride);
    else sum_parts_by<8>(v, part, nsplit, stride);
}
__device__ __forceinline__ f32x4 unpack4(u32x2 c) { return f32x4{bf16_lo(c[0]), bf16_hi(c[0]), bf16_lo(c[1]), bf16_hi(c[1])}; }
__device__ __forceinline__ u32x2 pack4(f32x4 v) { return u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])}; }
__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

constexpr int EPI_ROWS = 4;    // rows (waves) per workgroup
constexpr int EPI_COLS = 32;   // columns per workgroup of epi_cols_kernel: 256 workgroups at 1000 x 2048 (64 columns: half the CUs idle)

template <int EPI>
__global__ __launch_bounds__(256) void epi_rows_kernel(const GemmParams p, const float *__restrict__ part, const int nsplit)
{
    static_assert(EPI != EPI_RMSNORM_BWD, "see epi_cols_kernel");
    const int lane = threadIdx.x & 63;
    const int m = blockIdx.y * EPI_ROWS + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), tn = blockIdx.x, n = tn * 256 + lane * 4;
    if (m >= p.M) return;
    const bool ok = n < p.N;
    const int64_t plane = (int64_t)p.M * p.N;
    // the program's own inputs travel with the partials
    float rs = 1.0f;
    u32x2 res = {0u, 0u};
    u32x4 z = {0u, 0u, 0u, 0u};
    int pos = 0;
    if ((EPI == EPI_LINEAR || EPI == EPI_SWIGLU_FWD) && p.row_scale) rs = p.row_scale[m];
    if (EPI == EPI_LINEAR && p.rope_cos) pos = clampi(p.rope_pos[m], 0, p.rope_T - 1);
    if (EPI == EPI_LINEAR && p.add && ok) res = *reinterpret_cast<const u32x2 *>(p.add + (int64_t)m * p.ld_add + n);
    if (EPI == EPI_SWIGLU_BWD && ok) z = *reinterpret_cast<const u32x4 *>(p.Z + (int64_t)m * p.ldz + 2 * n);
    f32x4 sum[1] = {{0.f, 0.f, 0.f, 0.f}};
    if (ok) sum_parts(sum, {part + (int64_t)m * p.N + n}, nsplit, plane);
    f32x4 v = sum[0];
    float red = 0.0f;

    if constexpr (EPI == EPI_ACCUM) {
        if (ok) {
            f32x4 *o = reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(p.out) + (int64_t)m * p.ld_out + n);
            *o += v;
        }
        return;
    } else if constexpr (EPI == EPI_SWIGLU_FWD) {
        if (!ok) return;
        v *= rs;
        const float h0 = v[0] * fast_sigmoid(v[0]) * v[1], h1 = v[2] * fast_sigmoid(v[2]) * v[3];
        *reinterpret_cast<uint32_t *>(reinterpret_cast<uint16_t *>(p.out) + (int64_t)m * p.ld_out + (n >> 1)) = pack_bf16x2(h0, h1);
        if (p.out2) *reinterpret_cast<u32x2 *>(p.out2 + (int64_t)m * p.ld_out2 + n) = pack4(v);
        return;
    } else if constexpr (EPI == EPI_SWIGLU_BWD) {
        if (ok) {
            u32x4 dz;
            f32x4 act;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float d = v[e], gg = bf16_lo(z[e]), uu = bf16_hi(z[e]);
                const float sg = fast_sigmoid(gg), sl = gg * sg;
                const float dU = d * sl, dG = d * uu * (sg + sl * (1.0f - sg));
                dz[e] = pack_bf16x2(dG, dU);
                red += gg * dG + uu * dU;
                act[e] = gg * sg * uu;
            }
            *reinterpret_cast<u32x4 *>(reinterpret_cast<uint16_t *>(p.out) + (int64_t)m * p.ld_out + 2 * n) = dz;
            if (p.out2) *reinterpret_cast<u32x2 *>(p.out2 + (int64_t)m * p.ld_out2 + n) = pack4(act);
        }
    } else {
        if (p.lse_max) {
            constexpr float NEG_INF = -__builtin_inff(), LOG2E = 1.4426950408889634f;
            const f32x4 s = v * rs;
            float mx = ok ? fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])) : NEG_INF;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
            const float c2 = rs * LOG2E, d2 = -mx * LOG2E;
            float sm = 0.0f;
            if (ok && mx != NEG_INF) {                    // a block of -inf only: (max, sum) = (-inf, 0)
#pragma unroll
                for (int e = 0; e < 4; ++e) sm += __builtin_amdgcn_exp2f(__builtin_fmaf(v[e], c2, d2));
            }
            sm = wave_sum(sm);
            const unsigned e = (unsigned)(p.lse_y[m] - n);
            if (ok && e < 4u) p.lse_tgt[m] = e == 0 ? s[0] : (e == 1 ? s[1] : (e == 2 ? s[2] : s[3]));
            if (lane == 0) {
                p.lse_max[(int64_t)tn * p.M + m] = mx;
                p.lse_sum[(int64_t)tn * p.M + m] = sm;
            }
        }
        v *= rs;
        if (ok) {
            if (p.rope_cos && n < p.rope_cols)
                rope_unit(v, p, (int64_t)pos * p.rope_half, (n >> 1) % p.rope_half);
            if (p.add) v += unpack4(res);
            red = v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
            if (p.side)
                *reinterpret_cast<u32x2 *>(p.side + (int64_t)m * p.ld_side + n) = pack4(v * *reinterpret_cast<const f32x4 *>(p.col_scale + n));
            if (p.out_f32) *reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(p.out) + (int64_t)m * p.ld_out + n) = v;
            else *reinterpret_cast<u32x2 *>(reinterpret_cast<uint16_t *>(p.out) + (int64_t)m * p.ld_out + n) = pack4(v);
        }
    }
    if (p.rowred_mode != ROWRED_NONE) {
        red = wave_sum(red);
        if (lane == 0) {
            if (p.rowred_mode == ROWRED_PARTIALS) p.rowred[(int64_t)tn * p.M + m] = red;
            else atomicAdd(p.rowred + m, red);
        }
    }
}

// R rows of the RMSNorm backward, EPI_STEP apart from m on, in four columns: what they read is in flight together.  Rows past M read the
// last row and are dropped.  What is fused is written out: one row at a time and two give the same bits.
constexpr int EPI_STEP = 128;
template <int R>
__device__ __forceinline__ void cols_rows(const GemmParams &p, const float *part, int nsplit, int m, int n, f32x4 gm, f32x4 &dg)
{
#pragma clang fp contract(off)
    float rr[R], zz[R];
    u32x2 c[R], res[R];
    f32x4 d[R];
    const float *at[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int64_t mi = min(m + i * EPI_STEP, p.M - 1);
        rr[i] = p.rn_r[mi];
        zz[i] = p.rn_z[mi] * p.rn_zscale;
        c[i] = *reinterpret_cast<const u32x2 *>(p.rn_c + mi * p.ld_rn_c + n);
        res[i] = u32x2{0u, 0u};
        if (p.add) res[i] = *reinterpret_cast<const u32x2 *>(p.add + mi * p.ld_add + n);
        at[i] = part + mi * p.N + n;
        d[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    sum_parts(d, at, nsplit, (int64_t)p.M * p.N);
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int64_t mi = m + i * EPI_STEP;
        if (mi >= p.M) continue;
        const f32x4 cn = unpack4(c[i]) * rr[i];
        f32x4 o = __builtin_elementwise_fma(d[i], gm, -(cn * zz[i])) * rr[i];
        if (p.add) o += unpack4(res[i]);
        dg = __builtin_elementwise_fma(d[i], cn, dg);
        *reinterpret_cast<u32x2 *>(reinterpret_cast<uint16_t *>(p.out) + mi * p.ld_out + n) = pack4(o);
        if (p.out2) *reinterpret_cast<u32x2 *>(p.out2 + mi * p.ld_out2 + n) = pack4(cn * gm);
    }
}

// RMSNORM_BWD: 256 rows x 32 columns, 16 waves of eight rows a step, 8 lanes x 4 columns a row.  A workgroup a CU, so what both steps
// read is in flight together: 1000 x 2048 in four ranges, 49 MB, 13.0 -> 10.8 us.  A wave reads no step that lies past M: with both
// steps read for every wave a few rows took 11.2 us that take 7.9 (one row, 416 x 3280; 30 rows, 1544 x 5056: 14.9, 12.0).
template <int EPI>
__global__ __launch_bounds__(1024) void epi_cols_kernel(const GemmParams p, const float *__restrict__ part, const int nsplit)
{
    constexpr int ROWS = 256, COLS = EPI_COLS;
    static_assert(ROWS == 2 * EPI_STEP, "two steps");
    __shared__ f32x4 cs[16][COLS / 4];
    const int rl = threadIdx.x >> 3, cl = threadIdx.x & 7, n = blockIdx.x * COLS + cl * 4, m = blockIdx.y * ROWS + rl;
    f32x4 dg = {0.f, 0.f, 0.f, 0.f};
    const int mw = m - (rl & 7);                     // the wave's first row
    if (n < p.N && mw < p.M) {
        const f32x4 gm = *reinterpret_cast<const f32x4 *>(p.rn_gamma + n);
        if (mw + EPI_STEP < p.M) cols_rows<2>(p, part, nsplit, m, n, gm, dg);
        else cols_rows<1>(p, part, nsplit, m, n, gm, dg);
    }
    if (p.colred_mode == ROWRED_NONE) return;
    // column sums: the eight rows of a wave, then the sixteen waves in order
#pragma unroll
    for (int off = 8; off < 64; off <<= 1)
#pragma unroll
        for (int e = 0; e < 4; ++e) dg[e] += __shfl_xor(dg[e], off, 64);
    if ((threadIdx.x & 63) < 8) cs[threadIdx.x >> 6][cl] = dg;
    __syncthreads();
    const int nc = blockIdx.x * COLS + threadIdx.x;
    if (threadIdx.x >= COLS || nc >= p.N) return;
    float t = 0.0f;
#pragma unroll
    for (int w = 0; w < 16; ++w) t += reinterpret_cast<const float *>(cs[w])[threadIdx.x];
    if (p.colred_mode == ROWRED_PARTIALS) p.colred[(int64_t)blockIdx.y * p.N + nc] = t;
    else atomicAdd(p.colred + nc, t);
}

}  // namespace coda
