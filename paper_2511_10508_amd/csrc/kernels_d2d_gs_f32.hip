// 2D deep-tile kernels, FP32 storage: one (precision, kind) pair of the
// launcher in pf_deep2d_launch.h, instantiated in a file of its own.
#include "pf_deep2d_launch.h"

namespace pf {

template hipError_t launch_deep2d_kind<float, kGS>(const Launch &, const StepArgs<float> &, const DeepPlan &, bool,
                                                 hipStream_t);
template hipError_t launch_deep2d_batched_kind<float, kGS>(const Launch &, const BatchTable<float> &, int32_t, int32_t,
                                                         int32_t, hipStream_t);

}  // namespace pf
