// k_step_f32.hip -- the binary32-mixed instances of the fused step kernels
// (ecr_period.hpp, ecr_single.hpp)
#include "ecr_period.hpp"

namespace ecr {

template void launch_period<float>(const StepBatch<float> &, uint32_t, bool, bool, bool, hipStream_t);
template void launch_step<float>(const StepBatch<float> &, bool, bool, bool, const CellGrids &, hipStream_t);

}  // namespace ecr
