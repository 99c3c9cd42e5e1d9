"""Programs over the partials of a divided contraction: one to sixteen ranges (loads in batches of two, four and eight), rows at the edges of
the 128-row steps and 256-row blocks of the RMSNorm backward.  Against float64."""
import pytest
import torch

from tests import gpu_util as G
from tests import small_plan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    return small_plan.load(tmp_path_factory.mktemp("small_plan"))


CASES = [(864, 6016, 3304, 1), (769, 4104, 4104, 2), (385, 2056, 4104, 3), (256, 1032, 4104, 4), (257, 2056, 4104, 5), (129, 2056, 4104, 7), (504, 776, 6152, 8),
         (127, 2056, 4104, 9), (1, 264, 4104, 16)]


@pytest.mark.parametrize("M,N,K,ranges", CASES)
def test_ranges(plans, M, N, K, ranges):
    from paper_2605_19269_amd import coda
    route = small_plan.Route(plans, M, N, K, False, True, True, "rmsnorm_bwd", False, True)
    assert (route.kind, route.ranges) == ("divided", ranges)
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)
    A, B, C, R = rnd(M, K).bfloat16(), rnd(N, K).mul_(K ** -0.5).bfloat16(), rnd(M, N).bfloat16(), rnd(M, N).bfloat16()
    r, z, gamma = rnd(M).abs() + 0.5, rnd(M), rnd(N).abs() + 0.5
    ws = torch.empty(coda.coda_gemm_workspace_bytes(M, N, K, []), dtype=torch.uint8, device="cuda").fill_(0xA5)
    D = A.double() @ B.double().t()

    def check(out, ref, what, bound=1e-2):
        # bf16: half a step of rounding, 2^-9 of the value, and the fp32 sums behind it; five times that
        assert ((out.double() - ref).abs() <= bound * (ref.abs() + ref.square().mean().sqrt())).all(), what

    X, O = G.Guarded(M, N, torch.bfloat16, pad_cols=8), G.Guarded(M, N, torch.bfloat16, pad_cols=8)
    blocks = coda.coda_col_partial_blocks(M)
    dg = torch.full((blocks, N), G.SENTINEL_F32, device="cuda")
    coda.coda_gemm(A, B, [coda.rmsnorm_bwd(C, r, z, gamma, c_out=X.t, dgamma_out=dg), coda.add_tile(R), coda.store(O.t)], transB=True, workspace=ws)
    cn = C.double() * r.double()[:, None]
    torch.cuda.synchronize()
    for out in (X, O):
        out.check_guards(); out.written()
    check(X.t, cn * gamma.double(), "C_out")
    check(O.t, (D * gamma.double() - cn * z.double()[:, None]) * r.double()[:, None] + R.double(), "O_out")
    for b in range(blocks):
        # fp32 sums of up to 256 products of fp32 sums over K, in units of the terms' root of the sum of squares: 2^-24 * sqrt(256 + K) = 4e-6 expected; twenty times that
        t = (D * cn)[256 * b:256 * b + 256]
        assert ((dg[b].double() - t.sum(0)).abs() <= 1e-4 * (t.square().sum(0).sqrt() + 1.0)).all(), "dgamma"
    F, S = G.Guarded(M, N, torch.float32, pad_cols=4), torch.full((coda.coda_row_partial_blocks(N), M), G.SENTINEL_F32, device="cuda")
    coda.coda_gemm(A, B, [coda.row_scale(r), coda.row_sumsq(S), coda.store(F.t, f32=True)], transB=True, workspace=ws)
    torch.cuda.synchronize()
    F.check_guards(); F.written()
    ref = D * r.double()[:, None]
    check(F.t, ref, "fp32", 1e-5)
    assert ((S.double().sum(0) - ref.square().sum(1)).abs() <= 1e-5 * ref.square().sum(1)).all(), "row sum of squares"


@pytest.mark.parametrize("M,N,K", [(1, 416, 3280), (127, 2056, 4104), (129, 2056, 4104), (257, 2056, 4104), (864, 6016, 3304)])
def test_rmsnorm_backward_rounds_the_same_in_one_step_and_in_two(M, N, K):
    """Rows whose wave has a row 128 further on and rows whose wave has none: D * gamma fused with the product that is subtracted, everything
    else rounded by itself.  The 64-bit product of two fp32 is exact, and its sum with a third rounds to fp32 as the fused operation does but for one case in 2^29."""
    from paper_2605_19269_amd import coda
    g = torch.Generator(device="cuda").manual_seed(M + N)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)
    A, B, C, R = rnd(M, K).bfloat16(), rnd(K, N).mul_(K ** -0.5).bfloat16(), rnd(M, N).bfloat16(), rnd(M, N).bfloat16()
    r, z, gamma = (rnd(M).abs() + 0.5)[:, None], rnd(M)[:, None], rnd(N)
    ws = torch.empty(coda.coda_gemm_workspace_bytes(M, N, K, []), dtype=torch.uint8, device="cuda")
    D, O = torch.empty(M, N, device="cuda"), torch.empty(M, N, device="cuda", dtype=torch.bfloat16)
    coda.coda_gemm(A, B, [coda.store(D, f32=True)], workspace=ws)
    coda.coda_gemm(A, B, [coda.rmsnorm_bwd(C, r.view(M), z.view(M), gamma), coda.add_tile(R), coda.store(O)], workspace=ws)
    torch.cuda.synchronize()
    sub = (C.float() * r) * z
    fused = (D.double() * gamma.double() - sub.double()).float()
    assert torch.equal(O, (fused * r + R.float()).bfloat16())
