"""Host checks of the small-tile contraction: its plan stays inside the workspace and the shapes that the shared large
tiles are planned for, and its workgroup map reaches every (range, tile) exactly once."""
import ctypes
import random

import numpy as np
import pytest

from tests import small_plan


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return small_plan.load(tmp_path_factory.mktemp("small_plan"))


def test_plans_fit_the_workspace_of_the_shape(lib):
    from paper_2605_19269_amd import coda
    rng = random.Random(5)
    taken = 0
    for _ in range(4000):
        M, N, K = (int(2 ** rng.uniform(0, 14)), 8 * int(2 ** rng.uniform(0, 12.5)), 16 * int(2 ** rng.uniform(3, 10.5)))
        for f8 in (False, True):
            for ak, bkc in ((True, False), (True, True), (False, False), (False, True)):
                bm, bn, ns = small_plan.plan(lib, M, N, K, f8, ak, bkc)
                if ns == 0:
                    continue
                taken += 1
                esz = 1 if f8 else 2
                assert ns * M * N * 4 <= coda.coda_gemm_workspace_bytes(M, N, K, [])
                assert 1 <= ns <= -(-K * esz // 128), "every range has a stage"
                assert bm == (128 if M > 64 or not ak else 64 if M > 32 else 32) and bn in ((128, 256) if bm == 128 else (128,))
                assert -(-M // 256) * -(-N // 256) < 256, "whole rounds of large tiles stay on them"
    assert taken > 500


@pytest.mark.parametrize("tiles_m,tiles_n,ns", [(1, 1, 1), (1, 48, 5), (1, 224, 1), (2, 17, 7), (9, 3, 4), (20, 11, 1), (17, 5, 3)])
def test_map_is_a_bijection(lib, tiles_m, tiles_n, ns):
    n = tiles_m * tiles_n * ns
    out = (ctypes.c_int * (3 * n))()
    lib.host_small_map(tiles_m, tiles_n, ns, out)
    m = np.array(out).reshape(n, 3)
    assert (m.min(axis=0) >= 0).all() and (m.max(axis=0) == [tiles_m - 1, tiles_n - 1, ns - 1]).all()
    assert len({tuple(r) for r in m}) == n


def test_undivided_tiles_suit_the_program(lib):
    """Row reductions take 256-wide tiles, A not contiguous in K 128 rows; large launches keep the 256 x 256 tiles."""
    rng = random.Random(6)
    seen = set()
    for _ in range(4000):
        M, N, K = 8 * int(2 ** rng.uniform(0, 11)), 16 * int(2 ** rng.uniform(0, 10.5)), 16 * int(2 ** rng.uniform(0, 9))
        for prog in small_plan.PROGRAMS:
            for f8 in (False, True):
                for ak in (True, False):
                    for wide in (False, True) if prog in ("linear", "swiglu_bwd") else (False,):
                        t = small_plan.direct_tile(lib, M, N, K, f8, ak, prog, wide)
                        seen.add(t)
                        if wide:
                            assert t.endswith("x256")
                        if not ak or prog in ("swiglu_bwd", "accum"):
                            assert t.startswith(("128x", "256x"))
                        if prog == "swiglu_fwd":
                            assert t not in ("32x256", "64x256")
                        assert (t != "128x128_PAIR") or prog == "accum"
    assert seen == set(small_plan.TILES)
    for M, N, K in ((8192, 16384, 2048), (16384, 6144, 4096), (8192, 32768, 4096), (8192, 8192, 8192)):
        assert small_plan.direct_tile(lib, M, N, K) == "256x256"
