// epi_rows.hpp -- the epilogue program on a contraction that lies in the workspace as `nsplit` fp32 partial matrices
// [nsplit][M][N] (gemm_small.hpp): adds the partials up in range order and applies the program of GemmParams.
//
// One wave owns one row of a 256-column block, a lane four consecutive columns: loads and stores are row-contiguous
// without staging, the pairwise maps stay inside a lane, and a block's row reduction -- the 256-column granularity that
// the callers' partial buffers have -- is one wave reduction in a fixed order.  M / 4 x N / 256 workgroups, so even a
// few rows spread over the chip.  Bound by reading the partials (from L2 and the memory-side cache, where the first
// kernel left them).
//
// RMSNORM_BWD also reduces over the columns of 256-row blocks: there a workgroup owns 256 rows x 64 columns, 16 lanes a row.
#pragma once
#include "gemm_kernel.hpp"

namespace coda {

__device__ __forceinline__ f32x4 sum_parts(const float *part, int nsplit, int64_t stride)
{
    // four loads in flight, added up in range order
    f32x4 v = *reinterpret_cast<const f32x4 *>(part);
    int s = 1;
    for (; s + 3 < nsplit; s += 4) {
        f32x4 t[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) t[q] = *reinterpret_cast<const f32x4 *>(part + (s + q) * stride);
#pragma unroll
        for (int q = 0; q < 4; ++q) v += t[q];
    }
    for (; s < nsplit; ++s) v += *reinterpret_cast<const f32x4 *>(part + s * stride);
    return v;
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

template <int EPI>
__global__ __launch_bounds__(256) void epi_rows_kernel(const GemmParams p, const float *__restrict__ part, const int nsplit)
{
    static_assert(EPI != EPI_RMSNORM_BWD, "see epi_cols_kernel");
    const int lane = threadIdx.x & 63;
    const int m = blockIdx.y * EPI_ROWS + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), tn = blockIdx.x, n = tn * 256 + lane * 4;
    if (m >= p.M) return;
    const bool ok = n < p.N;
    const int64_t plane = (int64_t)p.M * p.N;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (ok) v = sum_parts(part + (int64_t)m * p.N + n, nsplit, plane);
    float red = 0.0f;

    if constexpr (EPI == EPI_ACCUM) {
        if (ok) {
            f32x4 *o = reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(p.out) + (int64_t)m * p.ld_out + n);
            *o += v;
        }
        return;
    } else if constexpr (EPI == EPI_SWIGLU_FWD) {
        if (!ok) return;
        v *= p.row_scale ? p.row_scale[m] : 1.0f;
        const float h0 = v[0] * fast_sigmoid(v[0]) * v[1], h1 = v[2] * fast_sigmoid(v[2]) * v[3];
        *reinterpret_cast<uint32_t *>(reinterpret_cast<uint16_t *>(p.out) + (int64_t)m * p.ld_out + (n >> 1)) = pack_bf16x2(h0, h1);
        if (p.out2) *reinterpret_cast<u32x2 *>(p.out2 + (int64_t)m * p.ld_out2 + n) = pack4(v);
        return;
    } else if constexpr (EPI == EPI_SWIGLU_BWD) {
        if (ok) {
            const u32x4 z = *reinterpret_cast<const u32x4 *>(p.Z + (int64_t)m * p.ldz + 2 * n);
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
        const float rs = p.row_scale ? p.row_scale[m] : 1.0f;
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
                rope_unit(v, p, (int64_t)clampi(p.rope_pos[m], 0, p.rope_T - 1) * p.rope_half, (n >> 1) % p.rope_half);
            if (p.add) v += unpack4(*reinterpret_cast<const u32x2 *>(p.add + (int64_t)m * p.ld_add + n));
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

// RMSNORM_BWD: 16 waves; 16 lanes x 4 columns a row, 64 rows per step of the workgroup.
template <int EPI>
__global__ __launch_bounds__(1024) void epi_cols_kernel(const GemmParams p, const float *__restrict__ part, const int nsplit)
{
    constexpr int ROWS = 256, COLS = 64, STEP = 64;
    __shared__ f32x4 cs[STEP][COLS / 4];
    const int rl = threadIdx.x >> 4, cl = threadIdx.x & 15, n = blockIdx.x * COLS + cl * 4;
    const bool nok = n < p.N;
    const int64_t plane = (int64_t)p.M * p.N;
    f32x4 dg = {0.f, 0.f, 0.f, 0.f}, gm = dg;
    if (nok) gm = *reinterpret_cast<const f32x4 *>(p.rn_gamma + n);
#pragma unroll
    for (int st = 0; st < ROWS / STEP; ++st) {
        const int m = blockIdx.y * ROWS + st * STEP + rl;
        if (m >= p.M || !nok) continue;
        const float rr = p.rn_r[m], zz = p.rn_z[m] * p.rn_zscale;
        const f32x4 d = sum_parts(part + (int64_t)m * p.N + n, nsplit, plane);
        const f32x4 cn = unpack4(*reinterpret_cast<const u32x2 *>(p.rn_c + (int64_t)m * p.ld_rn_c + n)) * rr;
        f32x4 o = (d * gm - cn * zz) * rr;
        if (p.add) o += unpack4(*reinterpret_cast<const u32x2 *>(p.add + (int64_t)m * p.ld_add + n));
        dg += d * cn;
        *reinterpret_cast<u32x2 *>(reinterpret_cast<uint16_t *>(p.out) + (int64_t)m * p.ld_out + n) = pack4(o);
        if (p.out2) *reinterpret_cast<u32x2 *>(p.out2 + (int64_t)m * p.ld_out2 + n) = pack4(cn * gm);
    }
    if (p.colred_mode == ROWRED_NONE) return;
    cs[rl][cl] = dg;
    __syncthreads();
    if (threadIdx.x >= COLS) return;
    float t = 0.0f;
#pragma unroll 8
    for (int r = 0; r < STEP; ++r) t += reinterpret_cast<const float *>(cs[r])[threadIdx.x];
    const int nc = blockIdx.x * COLS + threadIdx.x;
    if (nc >= p.N) return;
    if (p.colred_mode == ROWRED_PARTIALS) p.colred[(int64_t)blockIdx.y * p.N + nc] = t;
    else atomicAdd(p.colred + nc, t);
}

}  // namespace coda
