// The FP16 instantiations of the tile kernel with one workgroup per CU for a K that is no whole number of steps.
#include "tile1.h"

namespace gpusq {
gpusq_status launch_tile1_f16_ragged(const GemmArgs& a, const EvenPlan& plan, unsigned grid, hipStream_t s) { return launch_tile1_typed<false, true>(a, plan, grid, s); }
}  // namespace gpusq
