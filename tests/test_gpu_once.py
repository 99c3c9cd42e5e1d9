"""Weights fetched past the caches (one row of tiles, matrices from STREAM_BYTES on, whole lines) against the ordinary loads, which a row pitch
that is no multiple of a line takes: the same bits; and against float64."""
import pytest
import torch

from tests import gpu_util as G

pytestmark = pytest.mark.gpu

# divided (32 and 64 rows), one kernel (both), undivided 8-bit 128 x 128; full and ragged rows, columns and K
CASES = [(1, 4096, 14336, False, False), (64, 14344, 4104, False, True), (50, 14336, 4096, False, False), (32, 28680, 4104, False, False), (64, 28672, 4096, False, True),
         (8, 4096, 28688, True, True), (33, 28688, 4112, True, False), (96, 28688, 4112, True, True), (128, 28672, 4096, True, False)]


@pytest.mark.parametrize("M,N,K,f8,tb", CASES)
def test_same_bits(M, N, K, f8, tb):
    from paper_2605_19269_amd import coda
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    typ, esz = (torch.float8_e4m3fn, 1) if f8 else (torch.bfloat16, 2)
    A = torch.randn(M, K, device="cuda", generator=g).to(typ)
    rows, cols = (N, K) if tb else (K, N)
    V = torch.randn(rows, cols, device="cuda", generator=g).mul_(1.0 if f8 else K ** -0.5).to(typ)
    r = (torch.rand(M, device="cuda", generator=g) + 0.5) * (K ** -0.5 if f8 else 1.0)
    ws = torch.empty(coda.coda_gemm_workspace_bytes(M, N, K, []), dtype=torch.uint8, device="cuda")
    line = 128 // esz
    whole = (cols + line - 1) // line * line
    outs = []
    for pitch in (whole, whole + 16 // esz):
        B = torch.zeros(rows, pitch, device="cuda", dtype=torch.uint8 if f8 else typ)
        B[:, :cols] = V.view(torch.uint8) if f8 else V
        assert (B.data_ptr() % 128, pitch * esz % 128) == (0, 0 if pitch == whole else 16)
        Y = G.Guarded(M, N, torch.float32, pad_cols=4)
        coda.coda_gemm(A, B[:, :cols], [coda.row_scale(r), coda.store(Y.t, f32=True)], transB=tb, workspace=ws)
        torch.cuda.synchronize()
        Y.check_guards(); Y.written()
        outs.append(Y.t.clone())
    assert torch.equal(outs[0], outs[1])
    D = (A.double() @ (V.double().t() if tb else V.double())) * r.double()[:, None]
    # fp32 sums; 8-bit products round inside the MFMA
    assert ((outs[0].double() - D).abs() <= (1e-3 if f8 else 1e-5) * (D.abs() + D.square().mean().sqrt())).all()
