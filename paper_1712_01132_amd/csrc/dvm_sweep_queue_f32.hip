// The queue sweep in FP32.
#include "dvm_sweep_queue.h"

namespace pdvm {

template hipError_t launch_sweep_queue<float>(const Batch<float> &, hipStream_t, const Scratch &);

}  // namespace pdvm
