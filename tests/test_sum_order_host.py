"""Host checks of the promise that the order of the additions behind an element of D does not depend on the program: every program of
a shape gets kernels of one order."""
import random

import pytest

from tests import small_plan

ALL = [("linear", False), ("linear", True), ("swiglu_fwd", False), ("swiglu_bwd", False), ("swiglu_bwd", True), ("accum", False), ("rmsnorm_bwd", False)]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return small_plan.load(tmp_path_factory.mktemp("small_plan"))


def test_programs_of_a_shape_share_one_order(lib):
    rng = random.Random(11)
    mixed = set()
    for _ in range(3000):
        M, N, K = 16 * int(2 ** rng.uniform(0, 9)), 16 * int(2 ** rng.uniform(0, 12)), 16 * int(2 ** rng.uniform(0, 10))
        if rng.random() < 0.3:
            M, N, K = -(-M // 256) * 256, -(-N // 256) * 256, -(-K // 128) * 128
        for f8 in (False, True):
            for ak in (True, False):
                for bkc in (True, False):
                    for ws in (True, False):
                        routes = [small_plan.Route(lib, M, N, K, f8, ak, bkc, prog, wide, ws) for prog, wide in ALL]
                        assert len({r.order for r in routes}) == 1, (M, N, K, f8, ak, bkc, ws, [(r.kind, r.tile, r.order) for r in routes])
                        if len({r.kind for r in routes}) > 1:
                            mixed.add((ws, tuple(sorted({r.kind for r in routes}))))
    assert {(False, ("direct", "whole")), (True, ("direct", "divided"))} <= mixed       # the sizes are not of one kernel each


def test_chains_are_as_short_as_the_pieces_of_a_shared_tile(lib):
    """Where small tiles take over a shape that would be shared, their chains are no longer than a shared tile's stages over the ranges
    that reach into it, straddling or not."""
    rng = random.Random(12)
    straddling = 0
    for _ in range(6000):
        M, N, K = int(2 ** rng.uniform(0, 12)), 16 * int(2 ** rng.uniform(0, 11)), 16 * int(2 ** rng.uniform(7, 10.5))
        f8 = rng.random() < 0.5
        first, tail, chunks, pieces = small_plan.shared(lib, M, N, K, f8)
        r = small_plan.Route(lib, M, N, K, f8, workspace=True)
        if not chunks or r.kind == "shared":
            continue
        assert first == 0
        straddling += pieces > 1
        stages = -(-K * (1 if f8 else 2) // 128)
        # range c holds the stages (of all tiles, end to end) from c * tail * stages / chunks on
        starts = [c * tail * stages // chunks for c in range(chunks)]
        reach = max(sum(1 for c in range(chunks) if starts[c] < (t + 1) * stages and (starts + [tail * stages])[c + 1] > t * stages) for t in range(tail))
        assert r.order[1] == -(-stages // reach), (M, N, K, f8)
    assert straddling > 20


@pytest.mark.parametrize("M,N,K,f8", [(8144, 720, 6448, False), (12088, 384, 8448, False), (1000, 6016, 7280, False), (4000, 1520, 4528, False), (543, 8192, 8192, False),
                                      (736, 8016, 16208, True)])
def test_no_longer_chains_on_shared_tiles(lib, M, N, K, f8):
    """96 tiles in 256 ranges, B K-contiguous: the longest range is 1.4 to 1.5 times as long as the chains that small tiles fold at."""
    first, tail, chunks, pieces = small_plan.shared(lib, M, N, K, f8)
    stages = -(-K * (1 if f8 else 2) // 128)
    assert (first, tail, chunks, pieces) == (0, 96, 256, 2)
    for prog, wide in ALL:
        r = small_plan.Route(lib, M, N, K, f8, True, True, prog, wide, True)
        assert r.kind in ("direct", "divided") and r.order[1] < 0.72 * -(-tail * stages // chunks), (r.kind, r.order)


@pytest.mark.parametrize("tiles_m", [1, 2, 3, 7, 8, 9, 16, 21])
def test_small_tiles_know_the_xcd_of_their_large_tile(lib, tiles_m):
    for tiles_n in (1, 2, 3, 5, 8, 13, 40):
        assert lib.host_tile_xcd_ok(tiles_m, tiles_n)
