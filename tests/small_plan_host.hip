// Host build of the small-tile plan and of its workgroup -> (range, tile) map, for tests/test_small_plan_host.py and
// tests/test_gpu_small_tiles.py.  Compiled for the host only; nothing here touches a GPU.
#include "../paper_2605_19269_amd/csrc/gemm_small.hpp"
#include "../paper_2605_19269_amd/csrc/splitk_plan.hpp"

extern "C" {

// plan[0..2] = tile rows, tile columns, ranges (0: large tiles)
__attribute__((visibility("default"))) void host_small_plan(int64_t M, int64_t N, int64_t K, int f8, int ak, int bkc, int *plan)
{
    const coda::SmallPlan pl = coda::plan_small(M, N, K, f8 != 0, ak != 0, bkc != 0, coda::plan_splitk(M, N, K, f8 != 0));
    plan[0] = pl.bm; plan[1] = pl.bn; plan[2] = pl.nsplit;
}

// the undivided small tile of a program (coda::DirectTile; 0: 256 x 256 tiles)
__attribute__((visibility("default"))) int host_direct_tile(int64_t M, int64_t N, int64_t K, int f8, int ak, int prog, int wide)
{
    return coda::plan_direct(M, N, K, f8 != 0, ak != 0, (coda::DirectProgram)prog, wide != 0, coda::plan_splitk(M, N, K, f8 != 0)).tile;
}

// route[0..6] = coda::RouteKind, tile, chain, rot_cols, ranges, tile rows and columns of a divided launch
__attribute__((visibility("default"))) void host_route(int64_t M, int64_t N, int64_t K, int f8, int ak, int bkc, int prog, int wide, int workspace, int *route)
{
    const coda::Route r = coda::plan_route(M, N, K, f8 != 0, ak != 0, bkc != 0, (coda::DirectProgram)prog, wide != 0, workspace != 0);
    route[0] = r.kind; route[1] = r.tile; route[2] = r.chain; route[3] = r.rot_cols;
    route[4] = r.small.nsplit; route[5] = r.small.bm; route[6] = r.small.bn;
}

// plan[0..3] = coda::SplitPlan: first shared tile, shared tiles, ranges, workgroups a range
__attribute__((visibility("default"))) void host_split_plan(int64_t M, int64_t N, int64_t K, int f8, int *plan)
{
    const coda::SplitPlan pl = coda::plan_splitk(M, N, K, f8 != 0);
    plan[0] = pl.first; plan[1] = pl.tail; plan[2] = pl.chunks; plan[3] = pl.pieces;
}

// whether tiles of bm rows in `ranges` ranges fetch B past the caches
__attribute__((visibility("default"))) int host_reads_once(int64_t M, int64_t N, int64_t K, int f8, int bkc, int bm, int ranges, int64_t ldb_bytes, uint64_t at)
{
    return coda::reads_once(M, N, K, f8 != 0, bkc != 0, bm, ranges, ldb_bytes, at);
}

// whether the gradient program reads and writes D past the caches
__attribute__((visibility("default"))) int host_gradient_once(int64_t M, int64_t N, int64_t ld_bytes, uint64_t at)
{
    return coda::gradient_once(M, N, ld_bytes, at);
}

// whether tile_xcd() inverts tile_coords() on a grid of tiles
__attribute__((visibility("default"))) int host_tile_xcd_ok(int tiles_m, int tiles_n)
{
    for (int bid = 0; bid < tiles_m * tiles_n; ++bid) {
        int tm, tn;
        coda::tile_coords(bid, tiles_m * tiles_n, tiles_m, tiles_n, tm, tn);
        if (coda::tile_xcd(tm, tn, tiles_m, tiles_n) != bid % 8) return 0;
    }
    return 1;
}

// out[3 * bid ..] = tile row, tile column, range
__attribute__((visibility("default"))) void host_small_map(int tiles_m, int tiles_n, int nsplit, int *out)
{
    for (int bid = 0; bid < tiles_m * tiles_n * nsplit; ++bid) coda::small_coords(bid, tiles_m, tiles_n, nsplit, out[3 * bid], out[3 * bid + 1], out[3 * bid + 2]);
}

}
