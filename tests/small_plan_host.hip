// Host build of the small-tile plan and of its workgroup -> (range, tile) map, for tests/test_small_plan_host.py and
// tests/test_gpu_small_tiles.py.  Compiled for the host only; nothing here touches a GPU.
#include "../paper_2605_19269_amd/csrc/gemm_small.hpp"
#include "../paper_2605_19269_amd/csrc/splitk_plan.hpp"

extern "C" {

// plan[0..2] = tile rows, tile columns, ranges (0: large tiles)
__attribute__((visibility("default"))) void host_small_plan(int64_t M, int64_t N, int64_t K, int f8, int ak, int *plan)
{
    const coda::SmallPlan pl = coda::plan_small(M, N, K, f8 != 0, ak != 0);
    plan[0] = pl.bm; plan[1] = pl.bn; plan[2] = pl.nsplit;
}

// the undivided small tile of a program (coda::DirectTile; 0: 256 x 256 tiles)
__attribute__((visibility("default"))) int host_direct_tile(int64_t M, int64_t N, int64_t K, int f8, int ak, int prog, int wide)
{
    return coda::plan_direct(M, N, K, f8 != 0, ak != 0, (coda::DirectProgram)prog, wide != 0).tile;
}

// out[3 * bid ..] = tile row, tile column, range
__attribute__((visibility("default"))) void host_small_map(int tiles_m, int tiles_n, int nsplit, int *out)
{
    for (int bid = 0; bid < tiles_m * tiles_n * nsplit; ++bid) coda::small_coords(bid, tiles_m, tiles_n, nsplit, out[3 * bid], out[3 * bid + 1], out[3 * bid + 2]);
}

}
