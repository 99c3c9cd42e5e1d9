"""Host checks of where the plan of the small tiles draws its lines: sizes at which both sides were timed on the GPU, with the faster one
(microseconds, 256 x 256 tiles first)."""
import pytest

from tests import small_plan


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return small_plan.load(tmp_path_factory.mktemp("small_plan"))


# M, N, K, 8-bit, A transposed, B transposed, program, row reduction
LARGE = [(4096, 4096, 32, False, True, False, "accum", False),              # 27.0, 29.2 two 128x128 a CU
         (4096, 4096, 192, False, True, False, "accum", False),             # 30.0, 31.9
         (2248, 5912, 96, False, True, False, "accum", False),              # 25.3, 26.8
         (3426, 2832, 160, True, False, False, "linear", False),            # 14.7, 17.7 three rounds of 128x128
         (292, 46864, 3920, True, False, True, "linear", True),             # 118.7, 137.7 three rounds of 128x256
         (1915, 12816, 4752, True, False, False, "swiglu_fwd", False),      # 115.0, 133.5
         (384, 58320, 15968, True, False, False, "swiglu_fwd", False),      # 402, 480
         (4096, 4096, 1000, False, True, False, "accum", False),            # 54.9, 59.7 two 128x128 a CU
         (8192, 2048, 1000, False, True, False, "accum", False),            # 52.8, 60.7
         (5632, 2048, 504, False, True, False, "accum", False),             # 34.0, 35.2
         (2048, 16384, 504, False, True, False, "accum", False),            # 85.6, 92.8
         (4096, 6144, 3072, False, True, False, "accum", False),            # 160, 175
         (4096, 6144, 3080, False, True, False, "accum", False),            # 171, 177
         (4096, 28672, 424, False, True, False, "accum", False),            # 222, 252: D past the caches
         (4096, 22016, 704, False, True, True, "accum", False)]             # 229, 266
SMALL = [(897, 19712, 200, False, False, False, "swiglu_fwd", False, "128x256"),     # 26.6, 23.6 (128x128 28.2)
         (32, 55056, 176, True, True, False, "accum", False, "128x128_PAIR"),        # 10.0, 8.3 (128x128 11.9)
         (768, 8784, 96, False, False, True, "swiglu_fwd", False, "128x256"),        # 10.6, 7.7 (128x128 9.7)
         (3598, 5456, 352, True, False, True, "linear", True, "128x256"),            # 44.8, 36.9
         (6144, 4096, 96, False, True, False, "accum", False, "128x128_PAIR"),       # 46.4, 41.2
         (2048, 8192, 128, True, True, False, "accum", False, "128x128_PAIR"),       # 33.5, 30.5
         (2048, 11264, 1000, False, True, False, "accum", False, "128x128_PAIR"),    # 87.7, 81.4
         (2048, 11264, 2000, False, True, False, "accum", False, "128x128_PAIR"),    # 126, 120
         (14336, 4096, 504, False, True, False, "accum", False, "128x128_PAIR"),     # 140, 125
         (10240, 5120, 1000, False, True, False, "accum", False, "128x128_PAIR"),    # 172, 157
         (1000, 4048, 504, False, True, False, "accum", False, "128x128"),           # 28.0, 17.4 (two a CU 18.7)
         (3184, 1016, 352, False, True, False, "accum", False, "128x128")]           # 25.3, 15.4 (16.0)


@pytest.mark.parametrize("M,N,K,f8,ta,tb,prog,red", LARGE)
def test_large_tiles_where_they_are_faster(lib, M, N, K, f8, ta, tb, prog, red):
    assert small_plan.Route(lib, M, N, K, f8, not ta, tb, prog, red).kind == "whole"


@pytest.mark.parametrize("M,N,K,f8,ta,tb,prog,red,tile", SMALL)
def test_small_tiles_where_they_are_faster(lib, M, N, K, f8, ta, tb, prog, red, tile):
    r = small_plan.Route(lib, M, N, K, f8, not ta, tb, prog, red)
    assert (r.kind, r.tile) == ("direct", tile)


# M, N and microseconds of one D again and again: ordinary, past the caches
@pytest.mark.parametrize("M,N", [(2048, 5632), (4096, 4096), (2048, 11264), (4096, 8192), (4096, 11008)])     # 36 40, 28 33, 65 68, 65 69, 117 151
def test_gradients_that_may_stay_go_through_the_caches(lib, M, N):
    assert not lib.host_gradient_once(M, N, N * 4, 0)


@pytest.mark.parametrize("M,N", [(4096, 18432), (4096, 20480), (8192, 16384)])                                # 222 216, 214 169, 416 349
def test_gradients_that_never_stay_go_past_the_caches(lib, M, N):
    assert lib.host_gradient_once(M, N, N * 4, 0) and lib.host_gradient_once(M, N, (N + 32) * 4, 128)
    assert not lib.host_gradient_once(M, N, (N + 4) * 4, 0) and not lib.host_gradient_once(M, N, N * 4, 16)
