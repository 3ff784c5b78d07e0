// Row pass with several rows in flight, FP32 reading S (flowpass.h).
#include "flowpass.h"

namespace hap {

template hipError_t launch_flow<float, 0>(const SweepArgs<float> &, int, int, bool, bool, hipStream_t);
template hipError_t launch_flow<float, -1>(const SweepArgs<float> &, int, int, bool, bool, hipStream_t);

}  // namespace hap
