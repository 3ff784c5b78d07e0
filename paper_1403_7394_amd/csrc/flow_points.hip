// Row pass with several rows in flight, FP32 points mode (flowpass.h).
#include "flowpass.h"

namespace hap {

template hipError_t launch_flow<float, 2>(const SweepArgs<float> &, int, int, bool, bool, hipStream_t);
template hipError_t launch_flow<float, 3>(const SweepArgs<float> &, int, int, bool, bool, hipStream_t);

}  // namespace hap
