"""GPU parity of the gradient program's rows of D: whole 128-byte lines (past the caches), rows that start inside a line, the longest rows, on every tile that has the program, at edges of M and N and of
a pass of 32 rows, against the oracle with the bound of gpu_util."""
import numpy as np
import pytest
import torch

from paper_2605_19269_amd import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

# (M, N, K, 8-bit): 256 x 256 tiles, whole and ragged; 128 x 128 two a CU, whole and ragged; one row of tiles that ends inside a pass
SHAPES = [(256, 512, 64, False), (264, 520, 72, False), (1280, 1024, 128, False), (1032, 520, 40, False), (8, 264, 64, False), (272, 528, 144, True), (1280, 1024, 128, True)]
ROWS = ["lines", "inside a line", "base inside a line", "long"]


@pytest.mark.parametrize("M,N,K,f8,rows", [s + (r,) for s in SHAPES for r in ROWS if r != "long" or s[0] == 8])
def test_gradient_rows(oracle, M, N, K, f8, rows):
    from paper_2605_19269_amd import coda
    assert torch.cuda.is_available(), "these tests need the MI355X"
    g = np.random.Generator(np.random.PCG64(900 + M + N + K))
    if f8:
        A, B = synth.normal_f8e4m3(g, (K, M), 1.0), synth.normal_f8e4m3(g, (K, N), 1.0)
        dA, dB, A, B = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), oracle.f8e4m3_to_bf16_bits(A), oracle.f8e4m3_to_bf16_bits(B)
    else:
        A, B = synth.normal_bf16(g, (K, M), 1.0), synth.normal_bf16(g, (K, N), 0.05)
        dA, dB = G.dev_bf16(A), G.dev_bf16(B)
    lines = -(-N // 32) * 32
    ld, base = {"lines": (lines + 32, 0), "inside a line": (lines + 4, 0), "base inside a line": (lines + 32, 4), "long": (1 << 22, 0)}[rows]
    store = torch.empty((M - 1) * ld + lines + 36, device="cuda")
    D = store.as_strided((M, N), (ld, 1), base)
    beside = store.as_strided((M, 4), (ld, 1), base + N)         # the four values behind a row stay what they are
    assert D.data_ptr() % 16 == 0 and (D.data_ptr() % 128 != 0) == (base != 0)
    old = synth.normal_f32(g, (M, N), 1e-1)
    D.copy_(torch.from_numpy(old))
    beside.fill_(G.SENTINEL_F32)
    coda.coda_gemm(dA, dB, [coda.accum_f32(D)], transA=True)
    torch.cuda.synchronize()
    G.assert_f32_signed_close(G.host_f64(D), oracle.gemm_accumulate(A, B, old, transA=True), "accumulate")
    assert bool((beside == G.SENTINEL_F32).all())


@pytest.mark.parametrize("M,N,K", [(11008, 4096, 504), (2048, 11264, 1544), (4096, 4096, 256)])
def test_rounds_of_tiles(oracle, M, N, K):
    """Shapes of several rounds, on either side of where the plan goes from 256 x 256 tiles to 128 x 128, two a CU: rows of the first, an
    inner and the last tile."""
    from paper_2605_19269_amd import coda
    g = np.random.Generator(np.random.PCG64(950 + K))
    A, B = synth.normal_bf16(g, (K, M), 1.0), synth.normal_bf16(g, (K, N), 0.05)
    rows = np.array([0, 127, 128, M // 2 + 5, M - 129, M - 1])
    D = torch.full((M, N), 0.125, device="cuda")
    coda.coda_gemm(G.dev_bf16(A), G.dev_bf16(B), [coda.accum_f32(D)], transA=True)
    torch.cuda.synchronize()
    ref = oracle.gemm_accumulate(A, B, np.full((M, N), 0.125, np.float32), rows=rows, transA=True)
    G.assert_f32_signed_close(G.host_f64(D)[rows], ref, "accumulate")
