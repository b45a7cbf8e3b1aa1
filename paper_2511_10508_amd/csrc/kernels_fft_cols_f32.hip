// Column transforms of the spectral step, FP32 storage (pf_fft.h), in a file of
// their own so that they compile in parallel.
#include "pf_fft_launch.h"

namespace pf {

template hipError_t launch_fft_cols_t<float>(const SpecArgs &, const FftArgs &, int64_t, bool, int64_t, int,
                                             hipStream_t);

}  // namespace pf
