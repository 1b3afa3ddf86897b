// Weight-gradient kernels for 1x1 filters (one translation unit per filter
// size, compiled in parallel); the kernel is in sparse_dw.hpp.
#define ISC_DW_INSTANTIATE
#include "sparse_dw.hpp"

namespace isc {
namespace dwk {

hipError_t launch_r1(const DwArgs &a, const DwPlan &p, hipStream_t s) { return launch_dw_table<1, kDwTiles1, 0, sizeof(kDwTiles1) / sizeof(kDwTiles1[0])>(a, p, s); }

}  // namespace dwk
}  // namespace isc
