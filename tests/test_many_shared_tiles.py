"""Shapes of 70 to 128 tiles of 256 x 256 that a workspace divides: which of them take small tiles instead of shared ones (on the host),
and on the GPU every program of those that do, against float64 and with one D behind all of them."""
import pytest
import torch

from tests import gpu_util as G
from tests import small_plan


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    return small_plan.load(tmp_path_factory.mktemp("small_plan"))


# microseconds on shared tiles, on small ones
SMALL = [(1232, 5568, 15040, False, False), (1072, 3840, 11072, False, False), (960, 5376, 10432, False, False), (1024, 8192, 4096, False, False),
         (2304, 2304, 10240, False, True), (2045, 3392, 4480, True, True)]                   # 329 213, 176 119, 174 127, 77 62, 189 149, 53 34
SHARED = [(2048, 4096, 14336, False, False), (1440, 4096, 14336, False, False), (384, 16384, 14336, False, True), (512, 16384, 14336, False, False)]    # 179 189, 164 181, 189 228, 188 203


@pytest.mark.parametrize("M,N,K,f8,tb", SMALL)
def test_small_tiles_where_they_are_faster(plans, M, N, K, f8, tb):
    for prog, wide in (("linear", False), ("linear", True), ("swiglu_fwd", False), ("swiglu_bwd", True), ("accum", False), ("rmsnorm_bwd", False)):
        assert small_plan.Route(plans, M, N, K, f8, True, tb, prog, wide, True).kind in ("direct", "divided")


# microseconds on one range of 128 x 128, on two of 128 x 256: 24.2 29.4, 33.5 38.1, 26.3 29.7
@pytest.mark.parametrize("M,N,K,tb", [(99, 22016, 4096, True), (606, 6144, 5632, False), (117, 22016, 4096, False)])
def test_one_range_of_128_columns_where_it_is_faster(plans, M, N, K, tb):
    for prog in ("linear", "swiglu_fwd"):
        assert small_plan.Route(plans, M, N, K, True, True, tb, prog, False, True).tile == "128x128"


@pytest.mark.parametrize("M,N,K,f8,tb", SHARED)
def test_shared_tiles_where_they_are_faster(plans, M, N, K, f8, tb):
    assert small_plan.Route(plans, M, N, K, f8, True, tb, "linear", True, True).kind == "shared"


def test_the_line_lies_at_seventy_tiles(plans):
    for N, kinds in ((17664, {"shared"}), (17920, {"direct", "divided"})):          # 69 and 70
        assert -(-N // 256) == (69 if kinds == {"shared"} else 70)
        assert {small_plan.Route(plans, 256, N, 8192, False, True, False, p, w, True).kind for p, w in (("linear", False), ("linear", True), ("rmsnorm_bwd", False))} <= kinds


# A B^T whose K is no whole number of lines: on shared tiles, on small ones (RMSNorm backward), microseconds
RAGGED = [(1128, 4160, 12648, False, True), (2201, 1808, 15264, False, False), (244, 24768, 5552, True, False), (768, 6848, 7184, True, True)]   # 201 248, 199 234, 74 88, 70 85


@pytest.mark.parametrize("M,N,K,f8,ta", RAGGED)
def test_rows_of_broken_lines_stay_shared(plans, M, N, K, f8, ta):
    for prog, wide in (("linear", False), ("linear", True), ("swiglu_bwd", True), ("accum", False), ("rmsnorm_bwd", False)):
        assert small_plan.Route(plans, M, N, K, f8, not ta, True, prog, wide, True).kind == "shared"
        assert small_plan.Route(plans, M, N, K // 128 * 128, f8, not ta, True, prog, wide, True).kind in ("direct", "divided")


# one and two ranges; edges of the 128-row, 128- and 256-column tiles; K past a whole stage; all layouts
GPU = [(1281, 3720, 4104, False, False, False), (2304, 2304, 4160, False, False, True), (2040, 2312, 6152, False, True, False), (3832, 1288, 6152, False, True, True),
       (1537, 3856, 4112, True, False, False), (2048, 2304, 8208, True, False, True)]


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,f8,ta,tb", GPU)
def test_one_product_behind_all_programs(plans, M, N, K, f8, ta, tb):
    from paper_2605_19269_amd import coda
    kinds = {small_plan.Route(plans, M, N, K, f8, not ta, tb, p, w, True).kind for p, w in (("linear", False), ("linear", True), ("rmsnorm_bwd", False))}
    assert kinds <= {"direct", "divided"}
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    A, B = (torch.randn(s, device="cuda", generator=g).mul_(w) for s, w in (((K, M) if ta else (M, K), 1.0), ((N, K) if tb else (K, N), 1.0 if f8 else K ** -0.5)))
    A, B = ((t.to(torch.float8_e4m3fn) if f8 else t.bfloat16()) for t in (A, B))
    ws = torch.empty(coda.coda_gemm_workspace_bytes(M, N, K, []), dtype=torch.uint8, device="cuda").fill_(0xA5)
    assert ws.numel() > 0
    a, b = A.double(), B.double()
    D = (a.t() if ta else a) @ (b.t() if tb else b)

    def run(*ops):
        coda.coda_gemm(A, B, list(ops), transA=ta, transB=tb, workspace=ws)
        torch.cuda.synchronize()

    F = G.Guarded(M, N, torch.float32, pad_cols=4)
    run(coda.store(F.t, f32=True))
    F.check_guards(); F.written()
    # fp32 sums of K terms; 8-bit products round inside the MFMA
    assert ((F.t.double() - D).abs() <= (1e-3 if f8 else 1e-5) * (D.abs() + D.square().mean().sqrt())).all()
    exact = F.t.clone()
    Y, part = G.Guarded(M, N, torch.bfloat16, pad_cols=8), torch.empty(coda.coda_row_partial_blocks(N), M, device="cuda")
    run(coda.row_sumsq(part), coda.store(Y.t))
    assert torch.equal(Y.t, exact.bfloat16())
    assert ((part.sum(0).double() - exact.double().square().sum(1)).abs() <= 1e-3 * exact.double().square().sum(1)).all()
    S = torch.randn(M, N, device="cuda", generator=g)
    acc = S.clone()
    run(coda.accum_f32(acc))
    assert torch.equal(acc, S + exact)
    H, Z = G.Guarded(M, N // 2, torch.bfloat16, pad_cols=8), G.Guarded(M, N, torch.bfloat16, pad_cols=8)
    run(coda.swiglu_fwd(Z.t), coda.store(H.t))
    assert torch.equal(Z.t, exact.bfloat16())
    ref = torch.nn.functional.silu(exact.double()[:, 0::2]) * exact.double()[:, 1::2]
    assert ((H.t.double() - ref).abs() <= 1e-2 * (ref.abs() + ref.square().mean().sqrt())).all()
    C, r, gamma = torch.randn(M, N, device="cuda", generator=g).bfloat16(), torch.rand(M, device="cuda", generator=g) + 0.5, torch.rand(N, device="cuda", generator=g) + 0.5
    dg = torch.empty(coda.coda_col_partial_blocks(M), N, device="cuda")
    run(coda.rmsnorm_bwd(C, r, r, gamma, dgamma_out=dg), coda.store(Y.t))
    cn = C.double() * r.double()[:, None]
    ref = (exact.double() * gamma.double() - cn * r.double()[:, None]) * r.double()[:, None]
    assert ((Y.t.double() - ref).abs() <= 1e-2 * (ref.abs() + ref.square().mean().sqrt())).all()
    ref = (exact.double() * cn).sum(0)
    assert ((dg.sum(0).double() - ref).abs() <= 1e-3 * (ref.abs() + ref.square().mean().sqrt())).all()
