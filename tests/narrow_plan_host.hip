// Host build of the plan of the 256 x 192 tiles, for tests/test_narrow_tiles.py.  Compiled for the host only; nothing here touches a GPU.
#include "../paper_2605_19269_amd/csrc/gemm_kernel.hpp"
#include "../paper_2605_19269_amd/csrc/splitk_plan.hpp"

extern "C" __attribute__((visibility("default"))) int host_narrow(int64_t M, int64_t N, int64_t K, int f8, int ak, int bkc, int prog, int wide, int workspace)
{
    return coda::plan_route(M, N, K, f8 != 0, ak != 0, bkc != 0, (coda::DirectProgram)prog, wide != 0, workspace != 0).narrow;
}

// the alignment that the kernels assume of the RoPE tables
extern "C" __attribute__((visibility("default"))) int host_rope_align() { return (int)alignof(coda::rope_quad); }
