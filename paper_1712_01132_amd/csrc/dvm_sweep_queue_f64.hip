// The queue sweep in FP64.
#include "dvm_sweep_queue.h"

namespace pdvm {

template hipError_t launch_sweep_queue<double>(const Batch<double> &, hipStream_t, const Scratch &);

}  // namespace pdvm
