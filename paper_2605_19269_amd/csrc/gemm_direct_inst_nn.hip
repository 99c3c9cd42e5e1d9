// Undivided small-tile kernels for one operand type and layout pair (see small_direct.hpp).
#include "small_direct.hpp"
namespace coda {
template hipError_t launch_small_direct<false, true, false>(int, int, const GemmParams &, const SmallParams &, hipStream_t);
}
