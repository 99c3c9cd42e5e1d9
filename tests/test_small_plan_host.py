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
            for ak in (True, False):
                bm, ns, dense = small_plan.plan(lib, M, N, K, f8, ak)
                if ns == 0:
                    continue
                taken += 1
                esz = 1 if f8 else 2
                assert ns * M * N * 4 <= coda.coda_gemm_workspace_bytes(M, N, K, [])
                assert 1 <= ns <= -(-K * esz // 128), "every range has a stage"
                assert bm == (128 if M > 64 or not ak else 64 if M > 32 else 32) and (bm == 128 or not dense)
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
