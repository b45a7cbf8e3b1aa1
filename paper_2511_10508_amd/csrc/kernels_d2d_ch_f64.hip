// 2D deep-tile kernels, FP64 storage: one (precision, kind) pair of the
// launcher in pf_deep2d_launch.h, instantiated in a file of its own.
#include "pf_deep2d_launch.h"

namespace pf {

template hipError_t launch_deep2d_kind<double, kCH>(const Launch &, const StepArgs<double> &, const DeepPlan &, bool,
                                                 hipStream_t);
template hipError_t launch_deep2d_batched_kind<double, kCH>(const Launch &, const BatchTable<double> &, int32_t, int32_t,
                                                         int32_t, hipStream_t);

}  // namespace pf
