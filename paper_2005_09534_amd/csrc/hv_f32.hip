// FP32 instantiations of the fused Chebyshev step (hv_kernels.h).
#include "hv_kernels.h"

namespace polfed {

template void launch_step<float>(hipStream_t, int, const StepArgs<float> &, const StepShape &,
                                 int);

}  // namespace polfed
