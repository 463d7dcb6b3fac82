// The per-diagonal sweep in FP32.
#include "dvm_sweep_diag.h"

namespace pdvm {

template hipError_t launch_sweep<float>(const Batch<float> &, int, hipStream_t);

}  // namespace pdvm
