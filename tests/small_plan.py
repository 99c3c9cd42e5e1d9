"""ctypes access to the host build of the small-tile plan (tests/small_plan_host.hip)."""
import ctypes
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def load(folder):
    so = str(folder / "small_plan_host.so")
    subprocess.run([HIPCC, "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-shared", "-Wno-inline-asm", "-o", so,
                    os.path.join(ROOT, "tests", "small_plan_host.hip")], check=True, capture_output=True)
    lib = ctypes.CDLL(so)
    lib.host_small_plan.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_int] * 3 + [ctypes.POINTER(ctypes.c_int)]
    lib.host_direct_tile.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_int] * 4
    lib.host_route.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_int] * 6 + [ctypes.POINTER(ctypes.c_int)]
    lib.host_reads_once.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_int] * 4 + [ctypes.c_int64, ctypes.c_uint64]
    lib.host_gradient_once.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_uint64]
    lib.host_split_plan.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_int, ctypes.POINTER(ctypes.c_int)]
    lib.host_small_map.argtypes = [ctypes.c_int] * 3 + [ctypes.POINTER(ctypes.c_int)]
    return lib


def plan(lib, M, N, K, f8=False, ak=True, bkc=False):
    """(tile rows, tile columns, ranges); ranges = 0: the shape runs on the large tiles."""
    out = (ctypes.c_int * 3)()
    lib.host_small_plan(M, N, K, int(f8), int(ak), int(bkc), out)
    return tuple(out)


def shared(lib, M, N, K, f8=False):
    """(first shared 256 x 256 tile, shared tiles, ranges, workgroups a range); no ranges: nothing is shared."""
    out = (ctypes.c_int * 4)()
    lib.host_split_plan(M, N, K, int(f8), out)
    return tuple(out)


TILES = ["256x256", "64x64", "32x256", "64x256", "128x128", "128x128_PAIR", "128x256"]     # coda::DirectTile
PROGRAMS = ["linear", "swiglu_fwd", "swiglu_bwd", "accum"]                                 # coda::DirectProgram, whose last is RMSNorm backward
KINDS = ["whole", "shared", "divided", "direct"]                                           # coda::RouteKind


def direct_tile(lib, M, N, K, f8=False, ak=True, prog="linear", wide=False):
    """The tile of an undivided launch; wide: the program reduces over rows."""
    return TILES[lib.host_direct_tile(M, N, K, int(f8), int(ak), PROGRAMS.index(prog), int(wide))]


class Route:
    """The kernels of a call.  kind: "whole" (256 x 256 tiles), "shared", "divided" or "direct"; tile: its tile; order: what the order of
    the additions behind an element depends on."""

    def __init__(self, lib, M, N, K, f8=False, ak=True, bkc=False, prog="linear", wide=False, workspace=False):
        out = (ctypes.c_int * 7)()
        lib.host_route(M, N, K, int(f8), int(ak), int(bkc), (PROGRAMS + ["rmsnorm_bwd"]).index(prog), int(wide), int(workspace), out)
        kind, tile, chain, rot, ns, bm, bn = out
        self.kind, self.ranges = KINDS[kind], ns if KINDS[kind] == "divided" else 1
        self.tile = {"divided": "%dx%d" % (bm, bn), "direct": TILES[tile]}.get(self.kind, "256x256")
        self.order = ("shared",) if self.kind == "shared" else (self.ranges, chain, rot)
