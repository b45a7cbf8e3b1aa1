// Row transforms of the spectral step, FP32 storage (pf_fft.h), in a file of their
// own so that they compile in parallel.
#include "pf_fft_launch.h"

namespace pf {

template hipError_t launch_fft_rows_t<float>(const StepArgs<float> &, const FftArgs &, bool, hipStream_t);

}  // namespace pf
