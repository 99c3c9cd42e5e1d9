"""Weights fetched past the caches (reads_once): which launches do that (on the host), and on the GPU against the ordinary loads, which a row pitch
that is no multiple of a line takes: the same bits; and against float64."""
import pytest
import torch

from tests import gpu_util as G
from tests import small_plan

@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    return small_plan.load(tmp_path_factory.mktemp("small_plan"))


def once(plans, M, N, K, f8, tb, pitch=None, at=0):
    """Whether a call's kernel fetches its weights past the caches."""
    r = small_plan.Route(plans, M, N, K, f8, True, tb, workspace=True)
    bm = int(r.tile.split("x")[0])
    esz = 1 if f8 else 2
    hinted = (r.kind == "divided" and bm <= 64) or (r.kind == "direct" and r.tile == "128x128" and f8)      # the kernels there are
    return hinted and bool(plans.host_reads_once(M, N, K, int(f8), int(tb), bm, r.ranges, pitch or (K if tb else N) * esz, at))


# microseconds with ordinary loads and with the hint, other weights in between; the same matrix again and again
TAKEN = [(1, 28672, 4096, False, False),     # 42.2 38.6, 36.3 37.4
         (32, 14336, 4096, False, True),     # 26.5 23.9, 22.0 22.9
         (32, 28672, 4096, True, False),     # 26.6 25.3, 21.8 22.4
         (64, 28672, 4096, False, True),     # 42.3 39.3, 35.7 38.8
         (96, 28672, 4096, True, True),      # 28.4 25.8, 21.6 26.3
         (1, 24576, 8192, False, False),     # 70.0 67.2, 70.0 66.2
         (64, 8192, 20480, False, True)]     # 66.1 61.0, 65.9 60.4
LEFT = [(128, 28672, 4096, True, False),     # 33.4 31.2, 23.2 28.3
        (64, 14336, 4096, False, False),     # 29.1 29.7, 25.2 29.1
        (64, 6144, 8192, False, False),      # 25.9 26.4, 23.0 25.7
        (1, 22016, 4096, False, False),      # 35.6 34.9, 29.7 33.8
        (32, 18432, 4608, False, False),     # 40.1 39.3, 28.6 38.0
        (64, 12288, 12288, True, False),     # 41.5 40.9, 31.1 40.3
        (1, 8192, 4096, False, False), (128, 28672, 4096, False, True)]


@pytest.mark.parametrize("M,N,K,f8,tb", TAKEN)
def test_taken_where_other_weights_come_between(plans, M, N, K, f8, tb):
    assert once(plans, M, N, K, f8, tb)
    pitch = (K if tb else N) * (1 if f8 else 2)
    assert not once(plans, M, N, K, f8, tb, pitch=pitch + 16) and not once(plans, M, N, K, f8, tb, at=64)       # whole lines


@pytest.mark.parametrize("M,N,K,f8,tb", LEFT)
def test_not_taken_where_a_lone_matrix_would_pay_more(plans, M, N, K, f8, tb):
    assert not once(plans, M, N, K, f8, tb)


def test_more_than_one_row_of_tiles_reads_weights_again(plans):
    for bm in (32, 64, 128):
        for M in (bm, bm + 1):
            assert bool(plans.host_reads_once(M, 28672, 8192, 1, 1, bm, 1, 8192, 0)) == (M == bm)
            for tb in (0, 1):
                assert bool(plans.host_reads_once(M, 32768, 9216, 1, tb, bm, 1, 32768, 0)) == (M == bm)      # in either layout


# divided (32 and 64 rows), one kernel (both), undivided 8-bit 128 x 128; full and ragged rows, columns and K
CASES = [(1, 4096, 14336, False, False), (64, 14344, 4104, False, True), (50, 14336, 4096, False, False), (32, 28680, 4104, False, False), (64, 28672, 4096, False, True),
         (8, 4096, 28688, True, True), (33, 28688, 4112, True, False), (96, 28688, 4112, True, True), (128, 28672, 4096, True, False),
         (50, 8200, 20488, False, False), (64, 12304, 24592, True, True), (128, 28672, 4096, True, True)]
ORDINARY = [(64, 14344, 4104, False, True), (50, 14336, 4096, False, False), (128, 28672, 4096, True, False)]


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,f8,tb", CASES)
def test_same_bits(plans, M, N, K, f8, tb):
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
        assert once(plans, M, N, K, f8, tb, pitch * esz, B.data_ptr()) == (pitch == whole and (M, N, K, f8, tb) not in ORDINARY)
        Y = G.Guarded(M, N, torch.float32, pad_cols=4)
        coda.coda_gemm(A, B[:, :cols], [coda.row_scale(r), coda.store(Y.t, f32=True)], transB=tb, workspace=ws)
        torch.cuda.synchronize()
        Y.check_guards(); Y.written()
        outs.append(Y.t.clone())
    assert torch.equal(outs[0], outs[1])
    D = (A.double() @ (V.double().t() if tb else V.double())) * r.double()[:, None]
    # fp32 sums; 8-bit products round inside the MFMA
    assert ((outs[0].double() - D).abs() <= (1e-3 if f8 else 1e-5) * (D.abs() + D.square().mean().sqrt())).all()
