"""Few rows against weights of 129 to 256 tiles: contraction and epilogue in one kernel.  Against float64, and bit for bit against the
partials and the second kernel that a program with a row reduction takes on the same shape."""
import pytest
import torch

from tests import gpu_util as G
from tests import small_plan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    return small_plan.load(tmp_path_factory.mktemp("small_plan"))


# one row; one short of, at and past 32; 64; 129 tiles with 8 columns in the last, 256 whole ones; K past a whole stage by 8 (16), more than the ring
CASES = [(1, 16392, 4104, False, False), (31, 32768, 4096, False, True), (32, 20480, 4096, False, False), (33, 16520, 4168, False, True), (64, 24576, 4096, False, False),
         (1, 16400, 4112, True, True), (32, 32768, 4096, True, False), (50, 16528, 4176, True, False), (64, 28672, 4096, True, True)]


@pytest.mark.parametrize("M,N,K,f8,tb", CASES)
def test_one_kernel(plans, M, N, K, f8, tb):
    from paper_2605_19269_amd import coda
    for prog in ("linear", "swiglu_fwd"):
        route = small_plan.Route(plans, M, N, K, f8, True, tb, prog, False, True)
        assert (route.kind, route.tile, route.ranges) == ("divided", "32x128" if M <= 32 else "64x128", 1)
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    A, B = (torch.randn(s, device="cuda", generator=g).mul_(w) for s, w in (((M, K), 1.0), ((N, K) if tb else (K, N), 1.0 if f8 else K ** -0.5)))
    A, B = ((t.to(torch.float8_e4m3fn) if f8 else t.bfloat16()) for t in (A, B))
    ws = torch.empty(coda.coda_gemm_workspace_bytes(M, N, K, []), dtype=torch.uint8, device="cuda").fill_(0xA5)
    r = (torch.rand(M, device="cuda", generator=g) + 0.5) * (K ** -0.5 if f8 else 1.0)
    R = torch.randn(M, N, device="cuda", generator=g).bfloat16()
    b64 = B.double()
    D = (A.double() @ (b64.t() if tb else b64)) * r.double()[:, None]
    part = torch.empty(coda.coda_row_partial_blocks(N), M, device="cuda")

    def run(*ops):
        coda.coda_gemm(A, B, [coda.row_scale(r), *ops], transB=tb, workspace=ws)
        torch.cuda.synchronize()

    def check(out, ref, what, bound=1e-2):
        # bf16: half a step of rounding, 2^-9 of the value, and the fp32 sums behind it; five times that.  fp32: 8-bit products round inside the MFMA
        out.check_guards(); out.written()
        assert ((out.t.double() - ref).abs() <= bound * (ref.abs() + ref.square().mean().sqrt())).all(), what

    Y, W = G.Guarded(M, N, torch.bfloat16, pad_cols=8), G.Guarded(M, N, torch.bfloat16, pad_cols=8)
    run(coda.store(Y.t))
    run(coda.row_sumsq(part), coda.store(W.t))
    check(Y, D, "store")
    assert torch.equal(Y.t, W.t)
    F = G.Guarded(M, N, torch.float32, pad_cols=4)
    run(coda.add_tile(R), coda.store(F.t, f32=True))
    check(F, D + R.double(), "residual, fp32", 1e-3 if f8 else 1e-5)
    H, Z = G.Guarded(M, N // 2, torch.bfloat16, pad_cols=8), G.Guarded(M, N, torch.bfloat16, pad_cols=8)
    run(coda.swiglu_fwd(Z.t), coda.store(H.t))
    check(Z, D, "pre-activation")
    check(H, torch.nn.functional.silu(D[:, 0::2]) * D[:, 1::2], "SwiGLU")
    cos, sin = (torch.randn(70, 64, device="cuda", generator=g) for _ in range(2))
    pos = torch.randint(0, 70, (M,), device="cuda", dtype=torch.int32, generator=g)
    cols = N * 3 // 4 // 128 * 128
    run(coda.rope(cos, sin, pos, 128, cols), coda.store(Y.t))
    c, s = (t.double()[pos.long()].repeat(1, cols // 128) for t in (cos, sin))
    ref = D.clone()
    ref[:, 0:cols:2], ref[:, 1:cols:2] = D[:, 0:cols:2] * c - D[:, 1:cols:2] * s, D[:, 0:cols:2] * s + D[:, 1:cols:2] * c
    check(Y, ref, "RoPE")
