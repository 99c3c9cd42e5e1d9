"""Host check of what the compiler reported for the small-tile kernels and the epilogue kernels behind them: they depend on a compiler
option that keeps the accumulators in ordinary registers and run two waves a SIMD, so a small edit can start spills."""
import os
import re

import pytest

from paper_2605_19269_amd import build as B


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(B.RESOURCES):
        B.build(force=True)
    rows = {"partial": {}, "direct": {}, "rows": {}, "cols": {}, "stream": {}, "once partial": {}, "once direct": {}, "once stream": {}}
    cfg = r"SmallCfgILi(\d+)ELi(\d+)ELi(\d)ELi(\d)ELi(\d)ELb([01])EEE"
    for line in open(B.RESOURCES):
        name, vgpr, agpr, scratch, spill, lds = line.split()
        r = dict(vgpr=int(vgpr), agpr=int(agpr), scratch=int(scratch), spill=int(spill), lds=int(lds))
        m = re.search(r"gemm_small_(partial|direct|stream)INS_(4OnceINS_)?\d+" + cfg, name)
        if m:
            rows[("once " if m.group(2) else "") + m.group(1)][name] = dict(r, tile=(int(m.group(3)), int(m.group(4))), waves=int(m.group(5)) * int(m.group(6)))
        m = re.search(r"epi_(rows|cols)_kernel", name)
        if m:
            rows[m.group(1)][name] = r
    return rows


def test_every_instance_is_there(kernels):
    """Divided: 32 and 64 rows with A K-contiguous, 128 x 128 and 128 x 256, in two layouts of B and two operand types.  Undivided: 64x64
    for two programs, 32x256 and 64x256 (with chains and without) for one, 128x128 and 128x256 (likewise) for four in all layouts,
    128x128 two a CU for the gradient.  One kernel for one range: 32 and 64 rows, two layouts of B, two operand types, two programs.  With
    the weights past the caches: 32 and 64 rows of the divided ones and of those, 8-bit 128x128 undivided for two programs."""
    assert len(kernels["partial"]) == (1 + 1 + 2 + 2) * 2 * 2
    assert len(kernels["direct"]) == 2 * (2 * 2 + 2 + 2 * 2 + 4 * 4 * (1 + 2) + 4)
    assert len(kernels["rows"]) == 4 and len(kernels["cols"]) == 1
    assert len(kernels["stream"]) == len(kernels["once stream"]) == 2 * 2 * 2 * 2
    assert len(kernels["once partial"]) == 2 * 2 * 2 and len(kernels["once direct"]) == 2 * 2


def test_no_spills_and_two_waves_a_simd(kernels):
    for group in kernels.values():
        for name, r in group.items():
            assert r["scratch"] == 0 and r["spill"] == 0 and r["agpr"] == 0, (name, r)
            assert r["vgpr"] <= 256, (name, r)


def test_local_memory(kernels):
    for name, r in [i for group in kernels.values() for i in group.items() if "tile" in i[1]]:
        assert r["lds"] <= 160 * 1024, (name, r)
        if r["tile"][0] <= 64 and r["tile"][1] <= 128 or r["waves"] == 4 and r["tile"] == (128, 128):
            assert r["lds"] <= 80 * 1024, (name, r)              # two workgroups a CU
