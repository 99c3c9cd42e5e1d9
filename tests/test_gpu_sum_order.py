"""The order of the additions behind an element of D does not depend on the program: D taken out of every program, bit for bit.  The sizes
are ones whose programs run on different kernels (asserted), in every layout that has an order of its own."""
import pytest
import torch

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


# M, N, K, f8, A transposed, B transposed, workspace, tiles of the programs.  In turn: tiles of different widths; few rows of A B^T, which
# start by column, next to a 256 x 256 tile, bf16 and 8-bit; a whole shape of A B^T, which starts by XCD; ragged K; A^T B;
# 8-bit on all tiles; one range, taken over by an undivided tile; several ranges; ranges that straddle tiles
CASES = [(300, 11008, 3000, False, False, False, False, {"64x256", "128x256", "256x256"}),
         (40, 2048, 1024, False, False, True, False, {"32x256", "64x64", "128x256", "128x128", "256x256"}),
         (40, 2048, 1024, True, False, True, False, {"32x256", "64x64", "128x256", "128x128", "256x256"}),
         (512, 2048, 1024, False, False, True, False, {"32x256", "64x64", "128x256", "128x128", "256x256"}),
         (300, 2064, 1000, False, False, True, False, {"32x256", "64x64", "128x256", "128x128", "256x256"}),
         (2048, 3072, 512, False, True, False, False, {"128x256", "128x128_PAIR", "256x256"}),
         (200, 4096, 2000, True, False, False, False, {"32x256", "64x64", "128x256", "128x128", "256x256"}),
         (96, 28672, 4096, True, False, True, True, {"64x256", "128x128"}),
         (32, 28672, 4096, False, False, True, True, {"32x128", "128x128"}),
         (32, 28672, 4096, False, False, False, True, {"32x128", "128x128"}),
         (809, 4096, 4096, False, False, False, True, {"128x256"}), (1168, 3248, 6160, False, False, True, True, {"256x256"}), (768, 5632, 12288, True, False, False, True, {"256x256"})]


@pytest.mark.parametrize("M,N,K,f8,ta,tb,ws,tiles", CASES)
def test_every_program_has_the_same_d(plans, M, N, K, f8, ta, tb, ws, tiles):
    progs = [("linear", False), ("linear", True), ("swiglu_fwd", False), ("swiglu_bwd", False), ("swiglu_bwd", True), ("accum", False), ("rmsnorm_bwd", False)]
    routes = [small_plan.Route(plans, M, N, K, f8, not ta, tb, prog, wide, ws) for prog, wide in progs]
    assert {r.tile for r in routes} == tiles
    assert len({r.kind for r in routes}) > 1 or routes[0].ranges > 1 or routes[0].kind == "shared"
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    draw = lambda shape, std: torch.randn(shape, device="cuda", generator=g) * std
    A, B = draw((K, M) if ta else (M, K), 1.0), draw((N, K) if tb else (K, N), 1.0 if f8 else 0.05)
    A, B = ((t.to(torch.float8_e4m3fn).view(torch.uint8) if f8 else t.bfloat16()) for t in (A, B))
    work = torch.empty(coda.coda_gemm_workspace_bytes(M, N, K, []), dtype=torch.uint8, device="cuda") if ws else None
    f32 = lambda *shape: torch.zeros(shape, dtype=torch.float32, device="cuda")
    b16 = lambda *shape, value=0.0: torch.full(shape, value, dtype=torch.bfloat16, device="cuda")
    nblk = coda.coda_row_partial_blocks(N)

    def gemm(*ops):
        coda.coda_gemm(A, B, list(ops), transA=ta, transB=tb, workspace=work)

    D = f32(M, N)
    gemm(coda.store(D, f32=True))
    Db = D.bfloat16()
    X = f32(M, N)
    gemm(coda.row_sumsq(f32(nblk, M)), coda.store(X, f32=True))
    assert torch.equal(X, D), "row sum of squares"
    X = f32(M, N)
    gemm(coda.lse_partial(torch.zeros(M, dtype=torch.int32, device="cuda"), f32(nblk, M), f32(nblk, M), f32(M)), coda.store(X, f32=True))
    assert torch.equal(X, D), "log-sum-exp"
    X = f32(M, N)
    gemm(coda.accum_f32(X))
    assert torch.equal(X, D), "accumulation into zeros"
    Z = b16(M, N)
    gemm(coda.swiglu_fwd(Z), coda.store(b16(M, N // 2)))
    assert torch.equal(Z, Db), "pre-activation"
    # gate = up = 64: silu(64) = 64 in fp32, so dU = 64 D
    for stat in (None, f32(nblk, M)):
        dZ = b16(M, 2 * N)
        gemm(coda.swiglu_bwd(b16(M, 2 * N, value=64.0), stat_out=stat), coda.store(dZ))
        assert torch.equal(dZ[:, 1::2].float() / 64, Db.float()), "SwiGLU backward"
    # C = 0, r = gamma = 1: O = D
    O, one = b16(M, N), torch.ones(max(M, N), device="cuda")
    gemm(coda.rmsnorm_bwd(b16(M, N), one[:M], f32(M), one[:N]), coda.store(O))
    assert torch.equal(O, Db), "RMSNorm backward"


# M, N, K, f8: undivided tiles in place of one range (all that fold, with and without row sums), the divided tiles with one and several
# ranges; chains that divide a range and that do not
CHAINED = [(32, 28672, 4096, False), (96, 28672, 4096, True), (40, 20480, 8192, False), (512, 14336, 6144, True), (200, 28672, 4096, False), (200, 28672, 4096, True),
           (2, 16400, 23040, True), (1000, 4096, 4096, True), (509, 2048, 8192, False), (1000, 2048, 11264, True), (1000, 2048, 11264, False)]


@pytest.mark.parametrize("M,N,K,f8", CHAINED)
def test_long_sums_fold_at_the_length_of_the_shared_ranges(plans, M, N, K, f8):
    """A large value in the first stage swallows the small products that follow it in its chain, one MFMA step at a time (each is less than
    half its last place), and none of those in other chains, whose sums are added as a whole."""
    stage = 128 if f8 else 64
    stages = K // stage
    assert K % stage == 0
    if f8:                                     # 128 x 448^2 < 2^25: last place 2; a step of 64 products adds 2^-1, a stage 1
        A, B = torch.full((M, K), 2.0 ** -3), torch.full((K, N), 2.0 ** -4)
        A[:, :stage], B[:stage] = 448.0, 448.0
        A, B = (t.to(torch.float8_e4m3fn).view(torch.uint8).cuda() for t in (A, B))
        big, ulp, per_stage = 128 * 448.0 ** 2, 2.0, 1.0
    else:                                      # 2^30: last place 128; a step of 32 products adds 32, a stage 64
        A, B = torch.ones(M, K), torch.ones(K, N)
        A[:, 0], B[0] = 2.0 ** 15, 2.0 ** 15
        A, B = (t.bfloat16().cuda() for t in (A, B))
        big, ulp, per_stage = 2.0 ** 30, 128.0, 64.0
    work = torch.empty(coda.coda_gemm_workspace_bytes(M, N, K, []), dtype=torch.uint8, device="cuda")
    for wide in (False, True):
        route = small_plan.Route(plans, M, N, K, f8, True, False, "linear", wide, True)
        ranges, chain = route.order[:2]
        assert chain < stages, "a range of its own would not show it"
        first = min(chain, stages // ranges)                       # stages of the chain with the large value
        others = (stages - first) * per_stage
        folds = ranges * -(-stages // ranges // chain) + ranges
        D = torch.zeros(M, N, dtype=torch.float32, device="cuda")
        ops = [coda.row_sumsq(torch.zeros(coda.coda_row_partial_blocks(N), M, device="cuda"))] if wide else []
        coda.coda_gemm(A, B, ops + [coda.store(D, f32=True)], workspace=work)
        tol = 0.5 * ulp * folds                                    # half a last place for each sum that is added to the large one
        assert others > 2 * tol
        err = (D.double() - (big + others)).abs().max().item()
        assert err <= tol, (route.kind, route.tile, route.order, err, tol)
