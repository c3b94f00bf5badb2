// The INT8 instantiations of the tile kernel with one workgroup per CU for a K that is no whole number of steps.
#include "tile1.h"

namespace gpusq {
gpusq_status launch_tile1_i8_ragged(const GemmArgs& a, const EvenPlan& plan, unsigned grid, hipStream_t s) { return launch_tile1_typed<true, true>(a, plan, grid, s); }
}  // namespace gpusq
