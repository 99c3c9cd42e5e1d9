"""GPU parity of every epilogue program on every kind of kernel that a call can take: 256 x 256 tiles (whole rounds, ragged), shared
256 x 256 tiles (equal parts and ranges that straddle tiles, in all tiles and behind whole rounds), divided and undivided small tiles.
The kind is asserted, so that a change of the plan cannot empty the test.

The contraction D of a shape is checked on sampled rows against the oracle.  Every program is then checked on all elements against
float64 PyTorch of its definition on that D: the same D, bit for bit, is behind every program (test_gpu_sum_order.py)."""
import numpy as np
import pytest
import torch

from paper_2605_19269_amd import synth
from tests import gpu_util as G
from tests import small_plan

pytestmark = pytest.mark.gpu

coda = None
PROGRAMS = [("linear", False), ("linear", True), ("swiglu_fwd", False), ("swiglu_bwd", True), ("accum", False), ("rmsnorm_bwd", False)]


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


def close(got, ref, what, bf16=True):
    """The bounds of gpu_util on the GPU: bf16 outputs 1e-2 of the value and of the rms, fp32 ones 1e-3."""
    bound = 1e-2 if bf16 else 1e-3
    d, rms = (got.double() - ref).abs(), ref.square().mean().sqrt()
    limit = bound * (rms + ref.abs()) if bf16 else bound * torch.maximum(ref.abs(), rms)
    assert (d <= limit).all(), "%s: max delta %.3g, rms %.3g" % (what, d.max().item(), rms.item())


class Problem:
    def __init__(self, oracle, M, N, K, f8, ta, tb, ws, seed):
        self.M, self.N, self.ta, self.tb = M, N, ta, tb
        self.g = torch.Generator(device="cuda").manual_seed(seed)
        A, B = self.normal((K, M) if ta else (M, K)), self.normal((N, K) if tb else (K, N), 1.0 if f8 else 0.05)
        self.A, self.B = ((t.to(torch.float8_e4m3fn).view(torch.uint8) if f8 else t.bfloat16()) for t in (A, B))
        need = coda.coda_gemm_workspace_bytes(M, N, K, []) if ws else 0
        self.ws = torch.empty(need, dtype=torch.uint8, device="cuda").fill_(0xA5) if ws else None
        self.nblk = coda.coda_row_partial_blocks(N)
        D = G.Guarded(M, N, torch.float32, pad_cols=4)
        self.gemm(coda.store(D.t, f32=True))
        D.check_guards(); D.written()
        bits = oracle.f8e4m3_to_bf16_bits if f8 else lambda t: t
        a, b = (bits(t.cpu().numpy()) if f8 else G.host_bits(t) for t in (self.A, self.B))
        rows = np.unique(np.concatenate([synth.sample_rows_per_tile(M, 1, seed=seed) if M > 256 else np.arange(0, M, max(1, M // 8)), [0, M - 1]]))
        G.assert_f32_signed_close(G.host_f64(D.t[torch.from_numpy(rows).cuda()]), oracle.gemm_rowscale(a, b, transA=ta, transB=tb, rows=rows), "D")
        self.D = D.t.double()

    def normal(self, shape, std=1.0):
        return torch.randn(shape, device="cuda", generator=self.g) * std

    def uniform(self, n, lo=0.5, hi=1.5):
        return torch.rand(n, device="cuda", generator=self.g) * (hi - lo) + lo

    def gemm(self, *ops):
        coda.coda_gemm(self.A, self.B, list(ops), transA=self.ta, transB=self.tb, workspace=self.ws)

    def out(self, cols, dtype=torch.bfloat16):
        return G.Guarded(self.M, cols, dtype, pad_cols=8 if dtype == torch.bfloat16 else 4)

    def blocks(self, v, reduce):
        """[M x N] -> [column blocks of 256 x M]"""
        return torch.stack([reduce(v[:, c:c + 256]) for c in range(0, self.N, 256)])

    def partials(self):
        return torch.full((self.nblk, self.M), G.SENTINEL_F32, device="cuda")


def done(*outs):
    torch.cuda.synchronize()
    for o in outs:
        o.check_guards()
        o.written()


def check_linear(p):
    r, C, gamma = p.uniform(p.M), p.normal((p.M, p.N)).bfloat16(), p.uniform(p.N)
    Y, S, part = p.out(p.N), p.out(p.N), p.partials()
    p.gemm(coda.row_scale(r), coda.add_tile(C), coda.row_sumsq(part), coda.col_scale_side(gamma, S.t), coda.store(Y.t))
    done(Y, S)
    v = p.D * r.double()[:, None] + C.double()
    close(Y.t, v, "row scale + residual")
    close(S.t, v * gamma.double(), "column-scaled side output")
    close(part, p.blocks(v, lambda b: b.square().sum(1)), "row sums of squares", bf16=False)
    # atomic sums on top of what is there; a program without a row reduction may run on other tiles
    total = torch.ones(p.M, device="cuda")
    p.gemm(coda.row_sumsq(total, atomic=True), coda.store(Y.t))
    close(total, 1.0 + p.D.square().sum(1), "atomic row sum of squares", bf16=False)
    p.gemm(coda.row_scale(r), coda.add_tile(C), coda.store(Y.t))
    done(Y)
    close(Y.t, v, "without a row reduction")


def check_rope(p):
    hd, T = 128, 50
    cols = p.N // hd * hd
    cos, sin = p.normal((T, hd // 2)), p.normal((T, hd // 2))
    pos = torch.randint(0, T, (p.M,), device="cuda", dtype=torch.int32, generator=p.g)
    Y = p.out(p.N)
    p.gemm(coda.rope(cos, sin, pos, hd, cols), coda.store(Y.t))
    done(Y)
    ref = p.D.clone()
    c, s = (t.double()[pos.long()].repeat(1, cols // hd) for t in (cos, sin))
    a, b = p.D[:, 0:cols:2], p.D[:, 1:cols:2]
    ref[:, 0:cols:2], ref[:, 1:cols:2] = a * c - b * s, a * s + b * c
    close(Y.t, ref, "rope")


def check_log_sum_exp(p):
    # row scales of both signs, logits of order one
    r = p.uniform(p.M) / p.D.square().mean().sqrt().float()
    r[::3] *= -1.0
    y = torch.randint(0, p.N, (p.M,), device="cuda", dtype=torch.int32, generator=p.g)
    L, pmax, psum = p.out(p.N), p.partials(), p.partials()
    zt, lse = torch.full((p.M,), G.SENTINEL_F32, device="cuda"), torch.empty(p.M, device="cuda")
    p.gemm(coda.row_scale(r), coda.lse_partial(y, pmax, psum, zt), coda.store(L.t))
    coda.coda_lse_finalize(pmax, psum, p.M, p.nblk, lse_out=lse)
    done(L)
    v = p.D * r.double()[:, None]
    top = p.blocks(v, lambda b: b.amax(1))
    close(L.t, v, "logits")
    close(pmax, top, "block maxima", bf16=False)
    close(psum, p.blocks(v, lambda b: (b - b.amax(1, keepdim=True)).exp().sum(1)), "block sums", bf16=False)
    close(zt, v.gather(1, y.long()[:, None])[:, 0], "target logits", bf16=False)
    close(lse, v.logsumexp(1), "log-sum-exp", bf16=False)


def check_swiglu(p):
    scale = (1.0 / p.D.square().mean().sqrt()).float()
    r = p.uniform(p.M) * scale
    H, Z = p.out(p.N // 2), p.out(p.N)
    p.gemm(coda.row_scale(r), coda.swiglu_fwd(Z.t), coda.store(H.t))
    done(H, Z)
    v = p.D * r.double()[:, None]
    close(Z.t, v, "pre-activation")
    close(H.t, v[:, 0::2] * torch.sigmoid(v[:, 0::2]) * v[:, 1::2], "swiglu forward")
    Zin = p.normal((p.M, 2 * p.N)).bfloat16()
    g, u = Zin.double()[:, 0::2], Zin.double()[:, 1::2]
    sg = torch.sigmoid(g)
    dU, dG = p.D * g * sg, p.D * u * (sg + g * sg * (1.0 - sg))
    stat = g * dG + u * dU
    dZ, O, part = p.out(2 * p.N), p.out(p.N), p.partials()
    p.gemm(coda.swiglu_bwd(Zin, act_out=O.t, stat_out=part), coda.store(dZ.t))
    done(dZ, O)
    close(dZ.t, torch.stack([dG, dU], 2).reshape(p.M, 2 * p.N), "dZ")
    close(O.t, g * sg * u, "activation")
    close(part, p.blocks(stat, lambda b: b.sum(1)), "row statistic", bf16=False)
    total = torch.zeros(p.M, device="cuda")
    p.gemm(coda.swiglu_bwd(Zin, stat_out=total, atomic=True), coda.store(dZ.t))
    close(total, stat.sum(1), "atomic row statistic", bf16=False)


def check_accumulate(p):
    start = p.normal((p.M, p.N))
    buf = p.out(p.N, torch.float32)
    buf.t.copy_(start)
    buf.ref = buf.full.clone()
    p.gemm(coda.accum_f32(buf.t))
    torch.cuda.synchronize()
    buf.check_guards()
    close(buf.t, start.double() + p.D, "accumulate", bf16=False)


def check_rmsnorm_backward(p):
    C, Oin = p.normal((p.M, p.N)).bfloat16(), p.normal((p.M, p.N)).bfloat16()
    r, z, gamma = p.uniform(p.M), p.normal((p.M,), 0.3), p.uniform(p.N)
    O, Cn = p.out(p.N), p.out(p.N)
    dg = torch.full((coda.coda_col_partial_blocks(p.M), p.N), G.SENTINEL_F32, device="cuda")
    p.gemm(coda.rmsnorm_bwd(C, r, z, gamma, c_out=Cn.t, dgamma_out=dg), coda.add_tile(Oin), coda.store(O.t))
    done(O, Cn)
    rr, cn = r.double()[:, None], C.double() * r.double()[:, None]
    close(O.t, (p.D * gamma.double() - cn * z.double()[:, None]) * rr + Oin.double(), "O")
    close(Cn.t, cn * gamma.double(), "C")
    ref = p.D * cn
    close(dg, torch.stack([ref[m:m + 256].sum(0) for m in range(0, p.M, 256)]), "dgamma partials", bf16=False)
    total = torch.zeros(p.N, device="cuda")
    p.gemm(coda.rmsnorm_bwd(C, r, z, gamma, dgamma_out=total, atomic=True), coda.store(O.t))
    close(total, ref.sum(0), "atomic dgamma", bf16=False)


# M, N, K, 8-bit, A transposed, B transposed, workspace, kind of kernel
WHOLE = [(1680, 14000, 528, False, False, False), (1680, 14000, 1040, False, False, True), (1680, 14000, 528, False, True, False), (1680, 14000, 1040, False, True, True),
         (656, 10928, 144, False, False, True), (912, 13232, 128, False, True, True), (1280, 10496, 128, False, False, False),
         (1680, 14000, 528, True, False, True), (1424, 13744, 2064, True, False, False), (1680, 14000, 1040, True, True, False), (1424, 13744, 2064, True, True, True)]
# ... and whether ranges straddle tiles, whether whole rounds come first
SHARED = [(1280, 3328, 3072, False, False, False, False, False), (768, 5632, 6144, False, False, True, True, False), (1168, 3248, 6160, False, True, False, True, False),
          (8336, 432, 3088, False, True, True, False, False), (11008, 1536, 3072, False, False, True, False, True), (9616, 2224, 3088, False, False, False, True, True),
          (3584, 5888, 4096, False, True, False, True, True),
          (1280, 3328, 4096, True, False, True, False, False), (768, 5632, 12288, True, False, False, True, False), (1168, 3248, 12304, True, True, False, True, False),
          (8336, 432, 6160, True, True, True, False, False), (11008, 1536, 4096, True, True, False, False, True), (9616, 2224, 6160, True, False, True, True, True)]
DIVIDED = [(1, 264, 4104, False, False, False), (33, 520, 4096, False, False, True), (200, 1032, 4168, False, False, False), (504, 2056, 11272, False, True, False),
           (31, 528, 4096, True, False, True), (300, 1040, 4112, True, False, False), (1008, 2064, 11280, True, True, False)]
SMALL = [(40, 1040, 1000, False, False, False), (100, 2064, 1024, False, False, True), (300, 11008, 3000, False, False, False), (504, 1040, 1000, False, True, True),
         (40, 1040, 1040, True, False, True), (500, 6160, 1040, True, False, False), (512, 2064, 400, True, True, False)]
CASES = ([c + (False, "whole") for c in WHOLE] + [c[:6] + (True, "shared") for c in SHARED] + [c + (True, "divided") for c in DIVIDED] + [c + (False, "direct") for c in SMALL])


@pytest.mark.parametrize("M,N,K,f8,ta,tb,ws,kind", CASES)
def test_every_program(oracle, plans, M, N, K, f8, ta, tb, ws, kind):
    for prog, wide in PROGRAMS:
        r = small_plan.Route(plans, M, N, K, f8, not ta, tb, prog, wide, ws)
        assert r.kind == kind or (kind, prog, r.kind) == ("direct", "rmsnorm_bwd", "whole"), (prog, wide, r.kind, r.tile)
    p = Problem(oracle, M, N, K, f8, ta, tb, ws, seed=M + N + K)
    for check in (check_linear, check_rope, check_log_sum_exp, check_swiglu, check_accumulate, check_rmsnorm_backward):
        check(p)


@pytest.mark.parametrize("M,N,K,f8,ta,tb,straddling,behind", SHARED)
def test_shared_plans_are_of_every_kind(plans, M, N, K, f8, ta, tb, straddling, behind):
    first, tail, chunks, pieces = small_plan.shared(plans, M, N, K, f8)
    assert chunks > tail and (pieces > 1) == straddling and (first > 0) == behind


@pytest.mark.parametrize("M,N,K,kind", [(40, 520, 4096, "divided"), (100, 520, 1024, "direct"), (1680, 14000, 528, "whole")])
def test_log_sum_exp_of_blocks_without_a_finite_logit(plans, M, N, K, kind):
    """A block of -inf only has (max, sum) = (-inf, 0) and does not disturb the others."""
    ws = kind == "divided"
    assert small_plan.Route(plans, M, N, K, prog="linear", wide=True, workspace=ws).kind == kind
    A, B = torch.rand(M, K, device="cuda").bfloat16() + 0.5, (torch.randn(K, N, device="cuda") * 0.05).bfloat16()
    B[0, 256:512] = float("-inf")
    work = torch.empty(coda.coda_gemm_workspace_bytes(M, N, K, []), dtype=torch.uint8, device="cuda") if ws else None
    nblk = coda.coda_row_partial_blocks(N)
    pmax, psum = (torch.full((nblk, M), G.SENTINEL_F32, device="cuda") for _ in range(2))
    zt, lse, L = torch.zeros(M, device="cuda"), torch.empty(M, device="cuda"), torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
    y = torch.zeros(M, dtype=torch.int32, device="cuda")
    coda.coda_gemm(A, B, [coda.lse_partial(y, pmax, psum, zt), coda.store(L)], workspace=work)
    coda.coda_lse_finalize(pmax, psum, M, nblk, lse_out=lse)
    assert (pmax[1] == float("-inf")).all() and (psum[1] == 0).all()
    keep = torch.ones(N, dtype=torch.bool, device="cuda")
    keep[256:512] = False
    close(lse, (A.double() @ B[:, keep].double()).logsumexp(1), "log-sum-exp", bf16=False)


@pytest.mark.parametrize("M,N,K,f8", [(11008, 1536, 3072, False), (10896, 1456, 4112, True)])
def test_shared_tiles_in_a_graph_and_in_the_static_scratch(plans, M, N, K, f8):
    """The ticket counters of shared 256 x 256 tiles are cleared by a kernel inside the captured sequence.  Replays with eager work and
    poisoned memory between them, the caller's workspace and the static array all give the same bits."""
    assert small_plan.Route(plans, M, N, K, f8, workspace=True).kind == "shared"
    need = coda.coda_gemm_workspace_bytes(M, N, K, [])
    assert 0 < need <= coda.CODA_STATIC_WS_BYTES
    A, B = torch.randn(M, K, device="cuda"), torch.randn(K, N, device="cuda")
    A, B = ((t.to(torch.float8_e4m3fn).view(torch.uint8) if f8 else t.bfloat16()) for t in (A, B))
    work = torch.empty(need, dtype=torch.uint8, device="cuda").fill_(0xA5)
    eager, static, captured = (torch.zeros(M, N, device="cuda") for _ in range(3))
    coda.coda_gemm(A, B, [coda.store(eager, f32=True)], workspace=work)
    for _ in range(2):
        static.zero_()
        coda.coda_gemm_static_ws(A, B, [coda.store(static, f32=True)])
        assert torch.equal(eager, static)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        coda.coda_gemm(A, B, [coda.store(captured, f32=True)], workspace=work)
    torch.cuda.synchronize()
    for _ in range(3):
        captured.fill_(float("nan"))
        work.fill_(0xA5)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(eager, captured)
