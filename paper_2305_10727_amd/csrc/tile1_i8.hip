// The INT8 instantiations of the tile kernel with one workgroup per CU.
#include "tile1.h"

namespace gpusq {
gpusq_status launch_tile1_i8(const GemmArgs& a, const EvenPlan& plan, unsigned grid, hipStream_t s) { return launch_tile1_typed<true, false>(a, plan, grid, s); }
}  // namespace gpusq
