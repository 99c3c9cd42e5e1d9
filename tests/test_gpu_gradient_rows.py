"""GPU parity of the gradient program's rows of D: whole 128-byte lines, rows that start inside a line, the longest rows (past 2^31 bytes from row 128 on), by way of
the caches and past them, on every tile that has the program, whole and with edges of M and N that end inside a pass of 32 rows.  The tile is asserted, so that a
change of the plan cannot empty the test.

The contraction is checked on all elements against float64; D is then what it was, in random numbers, plus that contraction, bit for bit (the order of its sums does
not depend on the program), and nothing beside D changes."""
import numpy as np
import pytest
import torch

from paper_2605_19269_amd import synth
from tests import gpu_util as G
from tests import small_plan

pytestmark = pytest.mark.gpu

# tile, M, N, K, 8-bit, A transposed, B transposed
SHAPES = [("128x128", 256, 512, 64, False, True, False), ("128x128", 264, 520, 72, False, True, False), ("128x128", 8, 264, 64, False, True, False),
          ("128x128", 1032, 520, 40, False, True, True), ("128x128", 272, 528, 144, True, True, False), ("128x128", 1280, 1024, 128, True, False, True),
          ("128x128", 1280, 1024, 128, False, True, False), ("128x128", 1032, 520, 40, False, True, False), ("128x128", 1280, 1024, 128, True, True, False),
          ("128x128_PAIR", 2304, 2048, 128, False, True, False), ("128x128_PAIR", 2040, 2312, 72, False, True, False), ("128x128_PAIR", 4400, 504, 32, False, False, False),
          ("128x128_PAIR", 256, 8704, 128, True, True, False), ("128x128_PAIR", 1600, 1392, 32, True, False, True),
          ("128x256", 1024, 5120, 3072, False, True, False), ("128x256", 1296, 3856, 4352, False, True, False), ("128x256", 136, 17008, 1040, False, False, True),
          ("256x256", 4096, 4096, 128, False, True, False), ("256x256", 2136, 5664, 200, False, True, False), ("256x256", 136, 39064, 80, False, False, True),
          ("256x256", 256, 33024, 384, True, True, False), ("256x256", 144, 39776, 160, True, True, False)]
# D that does not stay in the caches
LARGE = [("128x128_PAIR", 4096, 17920, 128, True, True, True), ("128x128_PAIR", 4416, 16896, 32, True, True, False), ("128x128_PAIR", 14016, 5376, 32, False, True, False),
         ("256x256", 3840, 19712, 256, False, True, False), ("256x256", 2712, 27264, 200, False, True, False), ("256x256", 11280, 6624, 400, True, True, False)]
LONG = 1 << 22          # the longest row that is accepted
# rows of D: pitch over whole lines of 32 values, first element
ROWS = {"lines": (32, 0), "inside a line": (4, 0), "base inside a line": (32, 4), "long": (None, 0)}


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    return small_plan.load(tmp_path_factory.mktemp("small_plan"))


@pytest.mark.parametrize("tile,M,N,K,f8,ta,tb", SHAPES + LARGE)
def test_gradient_rows(plans, tile, M, N, K, f8, ta, tb):
    from paper_2605_19269_amd import coda
    assert torch.cuda.is_available(), "these tests need the MI355X"
    route, plain = (small_plan.Route(plans, M, N, K, f8, not ta, tb, p) for p in ("accum", "linear"))
    assert (route.kind, route.tile) in (("direct", tile), ("whole", tile)) and route.order == plain.order
    g = torch.Generator(device="cuda").manual_seed(900 + M + N + K)
    A, B = (torch.randn(s, device="cuda", generator=g) for s in ((K, M) if ta else (M, K), (N, K) if tb else (K, N)))
    A, B = ((t.to(torch.float8_e4m3fn) if f8 else t.bfloat16()) for t in (A, B))
    F = torch.full((M, N), G.SENTINEL_F32, device="cuda")
    coda.coda_gemm(A, B, [coda.store(F, f32=True)], transA=ta, transB=tb)
    a, b = A.double(), B.double()
    ref = (a.t() if ta else a) @ (b.t() if tb else b)
    # fp32 sums of K terms; 8-bit products round inside the MFMA
    assert ((F.double() - ref).abs() <= (1e-3 if f8 else 1e-5) * (ref.abs() + ref.square().mean().sqrt())).all()
    del ref
    lines, past = -(-N // 32) * 32, (tile, M, N, K, f8, ta, tb) in LARGE
    for rows, (over, base) in ROWS.items():
        if rows == "long" and M > 300:
            continue
        ld = LONG if over is None else lines + over
        # a row before D and one behind it, and what lies between its rows
        store = torch.full(((M + 2) * ld + 64,), G.SENTINEL_F32, device="cuda")
        D = store.as_strided((M, N), (ld, 1), ld + base)
        aligned = D.data_ptr() % 128 == 0 and ld % 32 == 0
        assert D.data_ptr() % 16 == 0 and aligned == (rows in ("lines", "long"))
        assert bool(plans.host_gradient_once(M, N, ld * 4, D.data_ptr())) == (past and aligned)
        old = torch.randn(M, N, device="cuda", generator=g)
        D.copy_(old)
        coda.coda_gemm(A, B, [coda.accum_f32(D)], transA=ta, transB=tb)
        torch.cuda.synchronize()
        assert torch.equal(D, old + F), rows
        D.fill_(G.SENTINEL_F32)
        assert bool((store == G.SENTINEL_F32).all()), rows
        del store, D, old


@pytest.mark.parametrize("M,N,K,tile", [(14336, 4096, 504, "128x128_PAIR"), (2048, 11264, 1544, "128x128_PAIR"), (2048, 16384, 504, "256x256"), (11008, 4096, 504, "256x256"), (4096, 4096, 256, "256x256")])
def test_rounds_of_tiles(oracle, plans, M, N, K, tile):
    """Shapes of several rounds, on either side of where the plan goes from 256 x 256 tiles to 128 x 128, two a CU, against the oracle: a row of every pass of the
    first tiles, and of an inner and the last one."""
    from paper_2605_19269_amd import coda
    assert small_plan.Route(plans, M, N, K, False, False, False, "accum").tile == tile
    g = np.random.Generator(np.random.PCG64(950 + K))
    A, B = synth.normal_bf16(g, (K, M), 1.0), synth.normal_bf16(g, (K, N), 0.05)
    rows = np.unique(np.concatenate([np.arange(5, 256, 32), [0, 127, 128, M // 2 + 5, M - 129, M - 1]]))
    D = torch.randn(M, N, device="cuda", generator=torch.Generator(device="cuda").manual_seed(K))
    old = D.cpu().numpy()
    coda.coda_gemm(G.dev_bf16(A), G.dev_bf16(B), [coda.accum_f32(D)], transA=True)
    torch.cuda.synchronize()
    G.assert_f32_signed_close(G.host_f64(D)[rows], oracle.gemm_accumulate(A, B, old, rows=rows, transA=True), "accumulate")
