"""The 256 x 192 tiles: which calls take them (on the host), and on the GPU every program they have at the edges of the tile, against
float64 and, bit for bit, against the 256 x 256 tiles that the same shape takes for a program with a row reduction."""
import ctypes
import os
import subprocess

import pytest
import torch

from tests import gpu_util as G
from tests import small_plan

LINEAR, SWIGLU_FWD, SWIGLU_BWD, ACCUM, RMSNORM_BWD = range(5)


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("narrow") / "narrow_plan_host.so")
    subprocess.run([small_plan.HIPCC, "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-shared", "-Wno-inline-asm", "-o", so,
                    os.path.join(small_plan.ROOT, "tests", "narrow_plan_host.hip")], check=True, capture_output=True)
    return ctypes.CDLL(so)


@pytest.fixture(scope="module")
def narrow(host):
    fn = host.host_narrow
    fn.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_int] * 6
    return lambda M, N, K, prog=LINEAR, f8=False, ta=False, tb=False, wide=False, ws=True: bool(
        fn(M, N, K, int(f8), int(not ta), int(tb), prog, int(wide), int(ws)))


# microseconds on 256 x 256 tiles (the last two: on 128 x 256) and on 256 x 192
FASTER = [(2560, 3776, 512), (1728, 5184, 8192), (2048, 6144, 4096), (7680, 4608, 1024), (3072, 5760, 2048), (1536, 12864, 2048)]   # 19.3 15.6, 160 136, 92 82, 80.7 70.6, 88 80, 91 83
SLOWER = [(1728, 23552, 4096), (6912, 25344, 2048), (1664, 7680, 5120), (8192, 16384, 2048), (1024, 6912, 4096), (512, 3072, 512)]   # 295 303, 602 630, 122 170, 419 471, 58 64, 9.5 16.5


@pytest.mark.parametrize("M,N,K", FASTER)
def test_taken_where_faster_by_programs_that_fit(narrow, M, N, K):
    for ws in (True, False):
        assert narrow(M, N, K, ws=ws) and narrow(M, N, K, SWIGLU_FWD, ws=ws)
        for other in (dict(wide=True), dict(f8=True), dict(ta=True), dict(tb=True), dict(prog=ACCUM), dict(prog=SWIGLU_BWD), dict(prog=RMSNORM_BWD)):
            assert not narrow(M, N, K, ws=ws, **other)


@pytest.mark.parametrize("M,N,K", SLOWER)
def test_not_taken_where_slower(narrow, M, N, K):
    assert not narrow(M, N, K) and not narrow(M, N, K, SWIGLU_FWD)


# one round of 128 x 256 tiles that half a round of narrow ones would replace: microseconds on either
HALF = [(2996, 1288, 7664), (7559, 528, 13216), (11518, 320, 13128), (256, 16576, 8640), (1670, 2320, 12904), (193, 17176, 11464)]   # 108 123, 156 185, 192 272, 116 126, 151 192, 177 202


@pytest.mark.parametrize("M,N,K", HALF)
def test_not_taken_for_half_a_round(narrow, M, N, K):
    for prog in (LINEAR, SWIGLU_FWD):
        assert not narrow(M, N, K, prog, ws=False)


def test_a_shape_that_a_workspace_divides_stays_divided(narrow):
    assert not narrow(1000, 2048, 11264) and not narrow(2048, 4096, 14336)


# whole tiles; one row, eight columns and eight of K past a tile; eight short of one; K of one pair of K-steps, four and more than the ring
GPU = [(2048, 6144, 64), (2560, 3840, 512), (1409, 6152, 72), (1535, 6136, 136), (3072, 3848, 200), (769, 11704, 320)]


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", GPU)
def test_programs_on_narrow_tiles(narrow, M, N, K):
    from paper_2605_19269_amd import coda
    assert narrow(M, N, K) and narrow(M, N, K, SWIGLU_FWD) and not narrow(M, N, K, wide=True)
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    A, B, R = (torch.randn(s, device="cuda", generator=g).mul_(w).bfloat16() for s, w in (((M, K), 1.0), ((K, N), K ** -0.5), ((M, N), 1.0)))
    r = torch.rand(M, device="cuda", generator=g) + 0.5
    gamma = torch.rand(N, device="cuda", generator=g) + 0.5
    D = (A.double() @ B.double()) * r.double()[:, None]
    nblk = coda.coda_row_partial_blocks(N)

    def run(*ops):
        coda.coda_gemm(A, B, [coda.row_scale(r), *ops])
        torch.cuda.synchronize()

    def check(out, ref, what):
        out.check_guards(); out.written()
        # bf16: half a step of rounding, 2^-9 of the value, and the fp32 sums behind it; five times that
        bound = 1e-2 if out.t.dtype == torch.bfloat16 else 1e-5
        assert ((out.t.double() - ref).abs() <= bound * (ref.abs() + ref.square().mean().sqrt())).all(), what

    Y, W, part = G.Guarded(M, N, torch.bfloat16, pad_cols=8), G.Guarded(M, N, torch.bfloat16, pad_cols=8), torch.empty(nblk, M, device="cuda")
    run(coda.store(Y.t))
    run(coda.row_sumsq(part), coda.store(W.t))                    # 256 x 256 or other tiles
    check(Y, D, "store")
    assert torch.equal(Y.t, W.t)
    F, S = G.Guarded(M, N, torch.float32, pad_cols=4), G.Guarded(M, N, torch.bfloat16, pad_cols=8)
    run(coda.add_tile(R), coda.store(F.t, f32=True))
    check(F, D + R.double(), "residual, fp32")
    run(coda.add_tile(R), coda.col_scale_side(gamma, S.t), coda.store(Y.t))
    check(Y, D + R.double(), "residual")
    check(S, (D + R.double()) * gamma.double(), "side output")
    H, Z = G.Guarded(M, N // 2, torch.bfloat16, pad_cols=8), G.Guarded(M, N, torch.bfloat16, pad_cols=8)
    act = torch.nn.functional.silu(D[:, 0::2]) * D[:, 1::2]
    run(coda.swiglu_fwd(), coda.store(H.t))
    check(H, act, "SwiGLU")
    run(coda.swiglu_fwd(Z.t), coda.store(H.t))
    check(H, act, "SwiGLU")
    check(Z, D, "pre-activation")
    for hd in (128, 48, 8):                                       # heads wider than a wave's 48 columns, as wide, narrower
        cols = N * 3 // 4 // hd * hd
        cos, sin = (torch.randn(70, hd // 2, device="cuda", generator=g) for _ in range(2))
        pos = torch.randint(0, 70, (M,), device="cuda", dtype=torch.int32, generator=g)
        run(coda.rope(cos, sin, pos, hd, cols), coda.store(Y.t))
        c, s = (t.double()[pos.long()].repeat(1, cols // hd) for t in (cos, sin))
        ref = D.clone()
        ref[:, 0:cols:2], ref[:, 1:cols:2] = D[:, 0:cols:2] * c - D[:, 1:cols:2] * s, D[:, 0:cols:2] * s + D[:, 1:cols:2] * c
        check(Y, ref, "RoPE, heads of %d" % hd)


def test_rope_tables_are_read_at_the_alignment_that_is_asked_of_them(host):
    from paper_2605_19269_amd import coda
    P, X, W = 0x10000, coda.coda_mat(0x10000, 0, 32, 32, 0, coda.CODA_BF16), coda.coda_mat(0x10000, 32, 64, 64, 0, coda.CODA_BF16)      # no rows: nothing is launched
    st = coda.coda_epi_op(coda.CODA_EPI_STORE, out=P, ld_out=64)
    for at in range(0, 32, 4):
        for cos, sin in ((P + at, P), (P, P + at)):
            rope = coda.coda_epi_op(coda.CODA_EPI_ROPE, in_=cos, in2=sin, in3=P, ld_in=128, i0=16, i1=32)
            assert coda.coda_gemm_raw(None, 0, 64, 32, X, W, [rope, st]) == (coda.CODA_ERR_ALIGN if at % host.host_rope_align() else coda.CODA_OK)


# narrow tiles; 256 x 256 tiles, whose heads of 64 and 128 take the same loads
@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(2560, 3840, 512), (1409, 6152, 72), (8192, 4096, 64)])
@pytest.mark.parametrize("hd", [128, 64, 48, 8])
def test_rope_tables_off_sixteen_bytes(narrow, M, N, K, hd):
    from paper_2605_19269_amd import coda
    assert narrow(M, N, K) == (M != 8192)
    g = torch.Generator(device="cuda").manual_seed(M + N + hd)
    A, B = (torch.randn(s, device="cuda", generator=g).bfloat16() for s in ((M, K), (K, N)))
    pos = torch.randint(0, 70, (M,), device="cuda", dtype=torch.int32, generator=g)
    tables = [torch.randn(70 * hd // 2 + 4, device="cuda", generator=g) for _ in range(2)]
    off = [t[2:2 + 70 * hd // 2].view(70, hd // 2) for t in tables]
    outs = []
    for (cos, sin), at in ((off, 8), ([t.clone() for t in off], 0)):
        assert (cos.data_ptr() % 16, sin.data_ptr() % 16) == (at, at)
        Y = G.Guarded(M, N, torch.bfloat16, pad_cols=8)
        coda.coda_gemm(A, B, [coda.rope(cos, sin, pos, hd, N // hd * hd), coda.store(Y.t)])
        torch.cuda.synchronize()
        Y.check_guards(); Y.written()
        outs.append(Y.t.clone())
    assert torch.equal(*outs)
