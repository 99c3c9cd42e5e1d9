"""GPU parity of the small-tile contraction and of the row-wise epilogue behind it: every tile, at the edges of M, N and K, every epilogue program, all layouts, bf16 and 8-bit operands, against the
oracle with the bounds of gpu_util."""
import numpy as np
import pytest
import torch

from paper_2605_19269_amd import synth
from tests import gpu_util as G
from tests import small_plan

pytestmark = pytest.mark.gpu

coda = None


@pytest.fixture(scope="module", autouse=True)
def _lib():
    global coda
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2605_19269_amd import coda as _c
    coda = _c
    yield
    torch.cuda.synchronize()


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    return small_plan.load(tmp_path_factory.mktemp("small_plan"))


def workspace(M, N, K):
    return torch.empty(coda.coda_gemm_workspace_bytes(M, N, K, []), dtype=torch.uint8, device="cuda").fill_(0xA5)


def operands(oracle, g, M, N, K, ta, tb, f8, a_std=1.0, b_std=0.05):
    sa, sb = ((K, M) if ta else (M, K)), ((N, K) if tb else (K, N))
    if f8:
        A, B = synth.normal_f8e4m3(g, sa, 1.0), synth.normal_f8e4m3(g, sb, 1.0)
        return torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), oracle.f8e4m3_to_bf16_bits(A), oracle.f8e4m3_to_bf16_bits(B)
    A, B = synth.normal_bf16(g, sa, a_std), synth.normal_bf16(g, sb, b_std)
    return G.dev_bf16(A), G.dev_bf16(B), A, B


# (M, N, K, f8, A transposed, B transposed, expected tile): one row; a full tile row; one row past it; ragged
# widths; K past a whole stage by 8 (bf16), 16 (8-bit); two tile rows; both widths of the 128-row tiles; all layouts
CASES = [(1, 264, 4104, False, False, False, (32, 128)), (32, 1000, 6144, False, False, True, (32, 128)), (33, 520, 4168, False, False, False, (64, 128)),
         (64, 256, 8192, False, False, True, (64, 128)), (65, 776, 4104, False, False, False, (128, 128)), (200, 1032, 4096, False, False, True, (128, 128)),
         (72, 520, 4168, False, True, False, (128, 128)), (128, 256, 4096, False, True, True, (128, 128)), (1000, 2056, 11272, False, False, True, (128, 256)), (1000, 1032, 8200, False, False, False, (128, 256)), (504, 2056, 11272, False, True, False, (128, 256)), (504, 2056, 11272, False, True, True, (128, 256)),
         (8, 256, 4112, True, False, True, (32, 128)), (31, 528, 4096, True, False, False, (32, 128)), (50, 520, 4112, True, False, True, (64, 128)),
         (96, 784, 4112, True, False, False, (128, 128)), (112, 272, 4096, True, True, False, (128, 128)), (144, 264, 4112, True, True, True, (128, 128)),
         (1000, 2056, 11280, True, False, True, (128, 256)), (1000, 2064, 11280, True, False, False, (128, 256)), (1008, 2064, 11280, True, True, False, (128, 256)), (1008, 2064, 11280, True, True, True, (128, 256))]


@pytest.mark.parametrize("M,N,K,f8,ta,tb,expect", CASES)
def test_linear_program(oracle, plans, M, N, K, f8, ta, tb, expect):
    bm, bn, ns = small_plan.plan(plans, M, N, K, f8, not ta, tb)
    assert ns > 0 and (bm, bn) == expect
    g = np.random.Generator(np.random.PCG64(4000 + M + N + K + 2 * ta + tb))
    dA, dB, A, B = operands(oracle, g, M, N, K, ta, tb, f8)
    C, r, gamma = synth.normal_bf16(g, (M, N), 1.0), synth.uniform_f32(g, (M,), 0.02, 0.06), synth.uniform_f32(g, (N,), 0.5, 1.5)
    dr, dC, dg, ws = G.dev_f32(r), G.dev_bf16(C), G.dev_f32(gamma), workspace(M, N, K)
    nblk = coda.coda_row_partial_blocks(N)
    outs = []
    for _ in range(2):
        Y, S = G.Guarded(M, N, torch.bfloat16), G.Guarded(M, N, torch.bfloat16)
        part = torch.full((nblk, M), G.SENTINEL_F32, dtype=torch.float32, device="cuda")
        coda.coda_gemm(dA, dB, [coda.row_scale(dr), coda.add_tile(dC), coda.row_sumsq(part), coda.col_scale_side(dg, S.t), coda.store(Y.t)],
                       transA=ta, transB=tb, workspace=ws)
        torch.cuda.synchronize()
        Y.check_guards(); Y.written(); S.check_guards(); S.written()
        outs.append((Y.t.clone(), part.clone()))
    refD, refss, refS = oracle.gemm_residual_sumsq(A, B, r=r.astype(np.float64), C=C, gamma=gamma.astype(np.float64), transA=ta, transB=tb, want_scaled=True)
    G.assert_bf16_close(G.host_f64(outs[0][0]), refD, "row scale + residual")
    G.assert_bf16_close(G.host_f64(S.t), refS, "column-scaled side output")
    G.assert_sumsq_close(G.host_f64(outs[0][1]).sum(axis=0), refss, "row sum of squares")
    for b in range(nblk):                                                # every 256-column block by itself
        G.assert_sumsq_close(G.host_f64(outs[0][1][b]), (refD[:, 256 * b:256 * b + 256] ** 2).sum(axis=1), "block %d" % b)
    assert torch.equal(outs[0][0].view(torch.int16), outs[1][0].view(torch.int16)) and torch.equal(outs[0][1], outs[1][1])


@pytest.mark.parametrize("M,N,K", [(1, 264, 4104), (40, 520, 4096), (200, 1032, 4168)])
def test_every_program(oracle, plans, M, N, K):
    assert small_plan.plan(plans, M, N, K)[2] > 0
    g = np.random.Generator(np.random.PCG64(4500 + M))
    dA, dB, A, B = operands(oracle, g, M, N, K, False, False, False)
    r, ws, nblk = synth.uniform_f32(g, (M,), 0.5, 1.5), workspace(M, N, K), coda.coda_row_partial_blocks(N)
    dr, r64 = G.dev_f32(r), r.astype(np.float64)

    def gemm(ops, a=dA, b=dB, **kw):
        coda.coda_gemm(a, b, ops, workspace=ws, **kw)
        torch.cuda.synchronize()

    # plain store in fp32
    F = G.Guarded(M, N, torch.float32, pad_cols=4)
    gemm([coda.row_scale(dr), coda.store(F.t, f32=True)])
    F.check_guards(); F.written()
    ref = oracle.gemm_rowscale(A, B, r=r64)
    G.assert_f32_signed_close(G.host_f64(F.t), ref, "f32 store")
    # RoPE: a head size that is no multiple of the block and a rotated width inside the matrix
    hd, rc, T = 24, 240, 50
    cos, sin = synth.rope_tables(T, hd)
    pos = np.ascontiguousarray(g.integers(0, T, M), dtype=np.int32)
    dcos, dsin, dpos = G.dev_f32(cos), G.dev_f32(sin), torch.from_numpy(pos).cuda()
    Q = G.Guarded(M, N, torch.bfloat16)
    gemm([coda.row_scale(dr), coda.rope(dcos, dsin, dpos, hd, rc), coda.store(Q.t)])
    Q.check_guards(); Q.written()
    G.assert_bf16_close(G.host_f64(Q.t), oracle.gemm_rowscale_rope(A, B, cos, sin, pos, hd, rc, r=r64), "rope")
    # log-sum-exp
    y = np.ascontiguousarray(g.integers(0, N, M), dtype=np.int32)
    dy = torch.from_numpy(y).cuda()
    L = G.Guarded(M, N, torch.bfloat16)
    pmax, psum = (torch.full((nblk, M), G.SENTINEL_F32, device="cuda") for _ in range(2))
    zt, lse, loss = (torch.full((M,), G.SENTINEL_F32, device="cuda") for _ in range(3))
    gemm([coda.row_scale(dr), coda.lse_partial(dy, pmax, psum, zt), coda.store(L.t)])
    coda.coda_lse_finalize(pmax, psum, M, nblk, ztgt=zt, lse_out=lse, loss_out=loss)
    torch.cuda.synchronize()
    refZ, refzt, reflse = oracle.gemm_rowscale_lse(A, B, y, r=r64)
    G.assert_bf16_close(G.host_f64(L.t), refZ, "logits")
    G.assert_f32_signed_close(G.host_f64(zt), refzt, "target logit")
    G.assert_f32_signed_close(G.host_f64(lse), reflse, "lse")
    G.assert_f32_signed_close(G.host_f64(loss), reflse - refzt, "loss")
    # SwiGLU forward with the pre-activation
    H, Zs = G.Guarded(M, N // 2, torch.bfloat16), G.Guarded(M, N, torch.bfloat16)
    gemm([coda.row_scale(dr), coda.swiglu_fwd(Zs.t), coda.store(H.t)])
    refH, refP = oracle.gemm_rowscale_swiglu(A, B, r=r64, want_preact=True)
    H.check_guards(); H.written(); Zs.check_guards(); Zs.written()
    G.assert_bf16_close(G.host_f64(H.t), refH, "swiglu forward")
    G.assert_bf16_close(G.host_f64(Zs.t), refP, "pre-activation")
    # SwiGLU backward with the activation and the row statistic
    dA2, dB2, A2, B2 = operands(oracle, g, M, N, K, False, True, False, a_std=1e-2, b_std=0.02)
    Z = synth.normal_bf16(g, (M, 2 * N), 1.0)
    dZin, dZ, O = G.dev_bf16(Z), G.Guarded(M, 2 * N, torch.bfloat16), G.Guarded(M, N, torch.bfloat16)
    part = torch.full((nblk, M), G.SENTINEL_F32, dtype=torch.float32, device="cuda")
    gemm([coda.swiglu_bwd(dZin, act_out=O.t, stat_out=part), coda.store(dZ.t)], dA2, dB2, transB=True)
    refdZ, refO, refstat = oracle.gemm_swiglu_bwd(A2, B2, Z, transB=True)
    dZ.check_guards(); dZ.written(); O.check_guards(); O.written()
    G.assert_bf16_close(G.host_f64(dZ.t), refdZ, "dZ")
    G.assert_bf16_close(G.host_f64(O.t), refO, "activation")
    G.assert_f32_signed_close(G.host_f64(part).sum(axis=0), refstat, "row statistic")
    # accumulation into an fp32 gradient
    Gin = synth.normal_f32(g, (M, N), 1e-1)
    buf = G.Guarded(M, N, torch.float32, pad_cols=4)
    buf.t.copy_(torch.from_numpy(Gin))
    buf.ref = buf.full.clone()
    gemm([coda.accum_f32(buf.t)])
    buf.check_guards()
    G.assert_f32_signed_close(G.host_f64(buf.t), oracle.gemm_accumulate(A, B, Gin), "accumulate")
    # RMSNorm backward, column partials per 256 rows
    Cb, Oin, z = synth.normal_bf16(g, (M, N), 1.0), synth.normal_bf16(g, (M, N), 1.0), synth.normal_f32(g, (M,), 0.3)
    gamma = synth.uniform_f32(g, (N,), 0.5, 1.5)
    Oout, Cout = G.Guarded(M, N, torch.bfloat16), G.Guarded(M, N, torch.bfloat16)
    dgp = torch.full((coda.coda_col_partial_blocks(M), N), G.SENTINEL_F32, dtype=torch.float32, device="cuda")
    dC, dz, dgm, dO = G.dev_bf16(Cb), G.dev_f32(z), G.dev_f32(gamma), G.dev_bf16(Oin)
    gemm([coda.rmsnorm_bwd(dC, dr, dz, dgm, c_out=Cout.t, dgamma_out=dgp), coda.add_tile(dO), coda.store(Oout.t)])
    refO, refC, refdg = oracle.gemm_rmsnorm_bwd(A, B, Cb, r64, z.astype(np.float64), gamma.astype(np.float64), Oin=Oin)
    Oout.check_guards(); Oout.written(); Cout.check_guards(); Cout.written()
    G.assert_bf16_close(G.host_f64(Oout.t), refO, "O_out")
    G.assert_bf16_close(G.host_f64(Cout.t), refC, "C_out")
    G.assert_f32_signed_close(G.host_f64(dgp).sum(axis=0), refdg, "dgamma")


# undivided launches: (M, N, K, f8, A transposed, B transposed, program, row reduction, tile): every tile with a ragged M, N and K, in
# bf16 and 8 bits, both layouts of B (128-row tiles: all four), and one whole shape of the tiles that skip bounds checks
DIRECT = [(1, 200, 72, False, False, False, "linear", False, "64x64"), (70, 520, 1000, False, False, True, "linear", False, "64x64"),
          (33, 336, 1040, True, False, False, "linear", False, "64x64"), (100, 264, 272, True, False, True, "linear", False, "64x64"),
          (1, 264, 8, False, False, False, "linear", True, "32x256"), (40, 520, 1000, False, False, True, "linear", True, "32x256"),
          (33, 528, 1040, True, False, False, "linear", True, "32x256"), (20, 264, 272, True, False, True, "linear", True, "32x256"),
          (2040, 2040, 1000, False, False, False, "linear", True, "64x256"), (2040, 2040, 1000, False, False, True, "linear", True, "64x256"),
          (2040, 2032, 1040, True, False, False, "linear", True, "64x256"), (2040, 2032, 1040, True, False, True, "linear", True, "64x256"),
          (8, 200, 72, False, False, False, "swiglu_fwd", False, "64x64"), (300, 1040, 1040, True, False, False, "swiglu_fwd", False, "64x64"),
          (500, 6160, 1000, False, False, False, "swiglu_fwd", False, "128x128"), (512, 6144, 1024, False, False, True, "swiglu_fwd", False, "128x128"),
          (500, 6160, 2064, True, False, False, "swiglu_fwd", False, "128x128"), (500, 6160, 2064, True, False, True, "swiglu_fwd", False, "128x128"),
          (72, 520, 200, False, True, False, "linear", False, "128x128"), (72, 520, 200, False, True, True, "linear", False, "128x128"),
          (80, 528, 400, True, True, False, "linear", False, "128x128"), (80, 528, 400, True, True, True, "linear", False, "128x128"),
          (500, 16376, 1000, False, False, False, "swiglu_fwd", False, "128x256"), (512, 16384, 1024, False, False, False, "swiglu_fwd", False, "128x256"),
          (500, 1032, 1000, False, False, True, "swiglu_bwd", True, "128x256"), (512, 1024, 1024, False, False, True, "swiglu_bwd", True, "128x256"),
          (80, 528, 400, True, True, False, "linear", True, "128x256"), (80, 528, 400, True, True, True, "linear", True, "128x256"),
          (504, 1032, 1000, False, True, True, "linear", True, "128x256"), (504, 1032, 1000, False, True, False, "linear", True, "128x256"),
          (500, 1040, 1040, True, False, False, "swiglu_bwd", True, "128x256"), (500, 1040, 1040, True, False, True, "swiglu_bwd", True, "128x256"),
          (1000, 2056, 504, False, True, False, "accum", False, "128x128"), (2048, 11264, 512, False, True, False, "accum", False, "128x128_PAIR"),
          (2040, 11272, 504, False, True, True, "accum", False, "128x128_PAIR"), (2032, 11280, 1040, True, True, False, "accum", False, "128x128_PAIR")]


@pytest.mark.parametrize("M,N,K,f8,ta,tb,prog,red,tile", DIRECT)
def test_undivided(oracle, plans, M, N, K, f8, ta, tb, prog, red, tile):
    assert small_plan.direct_tile(plans, M, N, K, f8, not ta, prog, red) == tile
    g = np.random.Generator(np.random.PCG64(5000 + M + N + K + 2 * ta + tb))
    dA, dB, A, B = operands(oracle, g, M, N, K, ta, tb, f8, a_std=1e-2 if prog == "swiglu_bwd" else 1.0)
    rows = None if M <= 300 else np.unique(np.concatenate([np.arange(0, M, 97), np.arange(0, M, 128), [M - 2, M - 1]]))
    idx = torch.arange(M).cuda() if rows is None else torch.from_numpy(rows).cuda()
    pick = lambda t: G.host_f64(t[idx])
    r = synth.uniform_f32(g, (M,), 0.02, 0.06) if f8 else synth.uniform_f32(g, (M,), 0.5, 1.5)
    dr, r64, nblk = G.dev_f32(r), r.astype(np.float64), coda.coda_row_partial_blocks(N)
    part = torch.full((nblk, M), G.SENTINEL_F32, dtype=torch.float32, device="cuda")
    kw = dict(transA=ta, transB=tb)
    if prog == "linear":
        C = synth.normal_bf16(g, (M, N), 1.0)
        dC, Y = G.dev_bf16(C), G.Guarded(M, N, torch.bfloat16)
        coda.coda_gemm(dA, dB, [coda.row_scale(dr), coda.add_tile(dC)] + ([coda.row_sumsq(part)] if red else []) + [coda.store(Y.t)], **kw)
        torch.cuda.synchronize()
        Y.check_guards(); Y.written()
        ref, refss = oracle.gemm_residual_sumsq(A, B, r=r64, C=C, rows=rows, **kw)[:2]
        G.assert_bf16_close(pick(Y.t), ref, "row scale + residual")
        if red:
            for b in range(nblk):
                G.assert_sumsq_close(pick(part[b]), (ref[:, 256 * b:256 * b + 256] ** 2).sum(axis=1), "row sum of squares, block %d" % b)
            y = np.ascontiguousarray(g.integers(0, N, M), dtype=np.int32)
            dy, L = torch.from_numpy(y).cuda(), G.Guarded(M, N, torch.bfloat16)
            pmax, psum = (torch.full((nblk, M), G.SENTINEL_F32, device="cuda") for _ in range(2))
            zt, lse = (torch.full((M,), G.SENTINEL_F32, device="cuda") for _ in range(2))
            coda.coda_gemm(dA, dB, [coda.row_scale(dr), coda.lse_partial(dy, pmax, psum, zt), coda.store(L.t)], **kw)
            coda.coda_lse_finalize(pmax, psum, M, nblk, lse_out=lse)
            torch.cuda.synchronize()
            refZ, refzt, reflse = oracle.gemm_rowscale_lse(A, B, y, r=r64, rows=rows, **kw)
            L.check_guards(); L.written()
            G.assert_bf16_close(pick(L.t), refZ, "logits")
            G.assert_f32_signed_close(pick(zt), refzt, "target logit")
            G.assert_f32_signed_close(pick(lse), reflse, "lse")
        else:
            hd, T = 24, 50
            cos, sin = synth.rope_tables(T, hd)
            pos = np.ascontiguousarray(g.integers(0, T, M), dtype=np.int32)
            dcos, dsin, dpos, Q = G.dev_f32(cos), G.dev_f32(sin), torch.from_numpy(pos).cuda(), G.Guarded(M, N, torch.bfloat16)
            coda.coda_gemm(dA, dB, [coda.row_scale(dr), coda.rope(dcos, dsin, dpos, hd, N - 8), coda.store(Q.t)], **kw)
            torch.cuda.synchronize()
            Q.check_guards(); Q.written()
            G.assert_bf16_close(pick(Q.t), oracle.gemm_rowscale_rope(A, B, cos, sin, pos, hd, N - 8, r=r64, rows=rows, **kw), "rope")
    elif prog == "swiglu_fwd":
        H, Z = G.Guarded(M, N // 2, torch.bfloat16), G.Guarded(M, N, torch.bfloat16)
        coda.coda_gemm(dA, dB, [coda.row_scale(dr), coda.swiglu_fwd(Z.t), coda.store(H.t)], **kw)
        torch.cuda.synchronize()
        H.check_guards(); H.written(); Z.check_guards(); Z.written()
        refH, refZ = oracle.gemm_rowscale_swiglu(A, B, r=r64, want_preact=True, rows=rows, **kw)
        G.assert_bf16_close(pick(H.t), refH, "swiglu forward")
        G.assert_bf16_close(pick(Z.t), refZ, "pre-activation")
    elif prog == "swiglu_bwd":
        Zin = synth.normal_bf16(g, (M, 2 * N), 1.0)
        dZin, dZ, O = G.dev_bf16(Zin), G.Guarded(M, 2 * N, torch.bfloat16), G.Guarded(M, N, torch.bfloat16)
        coda.coda_gemm(dA, dB, [coda.swiglu_bwd(dZin, act_out=O.t, stat_out=part), coda.store(dZ.t)], **kw)
        torch.cuda.synchronize()
        dZ.check_guards(); dZ.written(); O.check_guards(); O.written()
        refdZ, refO, refstat = oracle.gemm_swiglu_bwd(A, B, Zin, rows=rows, **kw)
        G.assert_bf16_close(pick(dZ.t), refdZ, "dZ")
        G.assert_bf16_close(pick(O.t), refO, "activation")
        G.assert_f32_signed_close(G.host_f64(part[:, idx]).sum(axis=0), refstat, "row statistic")
    else:
        Gin = synth.normal_f32(g, (M, N), 1e-1)
        buf = G.Guarded(M, N, torch.float32, pad_cols=4)
        buf.t.copy_(torch.from_numpy(Gin))
        buf.ref = buf.full.clone()
        coda.coda_gemm(dA, dB, [coda.accum_f32(buf.t)], **kw)
        torch.cuda.synchronize()
        buf.check_guards()
        G.assert_f32_signed_close(pick(buf.t), oracle.gemm_accumulate(A, B, Gin, rows=rows, **kw), "accumulate")
