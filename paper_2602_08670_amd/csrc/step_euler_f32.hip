// Euler steps in one launch, single precision.
#include "step_kernels.hpp"

namespace fvk {
template hipError_t step_go<float, EULER>(const StageDesc &, int, const StageArgs<float> &, hipStream_t);
template hipError_t step_load<float, EULER>();
}
