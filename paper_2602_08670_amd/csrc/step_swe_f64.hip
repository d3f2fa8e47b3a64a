// Shallow-water steps in one launch, double precision.
#include "step_kernels.hpp"

namespace fvk {
template hipError_t step_go<double, SWE>(const StageDesc &, int, const StageArgs<double> &, hipStream_t);
template hipError_t step_load<double, SWE>();
}
