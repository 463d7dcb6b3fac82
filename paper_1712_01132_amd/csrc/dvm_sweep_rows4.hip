// The row pipeline with 4 x 4 tiles (2D): instantiations and launcher.
#include "dvm_sweep_rows4.h"

namespace pdvm {

template <typename T, bool LOCAL>
void launch_rows4_local(const Batch<T> &B, dim3 grid, hipStream_t st, const Scratch &scr) {
#define PDVM_ROWS4(E)                                                                               \
  hipLaunchKernelGGL((sweep_rows4_kernel<T, LOCAL, band_waves(4), E>), grid, dim3(rows4_threads()), 0, st, B.d_geo, \
                     B.d_row_off, B.nprob, B.row_stride, scr.progress, scr.prog_pad, scr.xcc)
  // EXT: bit 0 tau fed back (psi), bit 1 Shakhov, bit 2 Maxwell walls
  if (B.maxwell) {
    if (B.shakhov) PDVM_ROWS4(7);
    else if (B.tau_fb) PDVM_ROWS4(5);
    else PDVM_ROWS4(4);
  } else if (B.shakhov) PDVM_ROWS4(3);
  else if (B.tau_fb) PDVM_ROWS4(1);
  else PDVM_ROWS4(0);
#undef PDVM_ROWS4
}

template <typename T>
hipError_t launch_sweep_rows4(const Batch<T> &B, bool local, hipStream_t st, const Scratch &scr) {
  const dim3 grid((unsigned)B.h_row_off[B.nprob]);
  if (local) launch_rows4_local<T, true>(B, grid, st, scr);
  else launch_rows4_local<T, false>(B, grid, st, scr);
  return hipGetLastError();
}

namespace {
template <typename T>
__global__ void rows4_reset_kernel(const Geo<T> *__restrict__ G, const int *__restrict__ off, int pad, int32_t *prog) {
  const int p = blockIdx.x;
  const int32_t below = (int32_t)((uint32_t)G[p].seq * (uint32_t)G[p].ntile[0]);
  for (int i = off[p] + threadIdx.x; i < off[p + 1]; i += blockDim.x) prog[(int64_t)i * pad] = below;
}
}  // namespace

template <typename T>
hipError_t launch_rows4_reset(const Batch<T> &B, const Scratch &scr, hipStream_t st) {
  hipLaunchKernelGGL((rows4_reset_kernel<T>), dim3((unsigned)B.nprob), dim3(256), 0, st, B.d_geo, B.d_row_off,
                     scr.prog_pad, scr.progress);
  return hipGetLastError();
}

template hipError_t launch_rows4_reset<double>(const Batch<double> &, const Scratch &, hipStream_t);
template hipError_t launch_rows4_reset<float>(const Batch<float> &, const Scratch &, hipStream_t);
template hipError_t launch_sweep_rows4<double>(const Batch<double> &, bool, hipStream_t, const Scratch &);
template hipError_t launch_sweep_rows4<float>(const Batch<float> &, bool, hipStream_t, const Scratch &);

}  // namespace pdvm
