// The sweep as one launch per diagonal of tiles (launch_sweep).
#pragma once
#include "dvm_sweep_tile.h"

namespace pdvm {
namespace {

// Step (i) for one diagonal of tiles: block = (octant, group, tile of the
// diagonal). In 2D the tiles (a, b) with a + b = diag are computed, the same
// for every octant; in 3D they come per octant from the table of tiles
// holding fluid.
template <typename T, int DIM, int TT, bool Y2WALL, int EXT>
__global__ void __launch_bounds__(kWave)
    sweep_kernel(const Geo<T> *__restrict__ G, const int *__restrict__ item_off, int nprob, int diag) {
  __shared__ TileLds<T, DIM, TT, EXT> L;
  const int p = nprob > 1 ? owner_of(item_off, nprob, blockIdx.x) : 0;
  const Geo<T> &G_ = G[p];
  if (!G_.run) return;  // converged problems retire
  const int ngroups = G_.ngroups;
  int item = nprob > 1 ? blockIdx.x - item_off[p] : blockIdx.x;
  int t, grp, o, tpos[3] = {0, 0, 0};
  if (DIM == 2) {
    const int amin = max(0, diag - (G_.ntile[1] - 1)), amax = min(diag, G_.ntile[0] - 1);
    const int ntd = amax - amin + 1;
    t = item % ntd;
    item /= ntd;
    grp = item % ngroups;
    o = item / ngroups;
    tpos[0] = amin + t;
    tpos[1] = diag - tpos[0];
#pragma unroll
    for (int j = 0; j < 2; ++j)
      if ((o >> j) & 1) tpos[j] = G_.ntile[j] - 1 - tpos[j];
  } else {
    const gptr<const int32_t> diag_off = as_global(G_.diag_off) + diag * 8;
    const int base = diag_off[0];
    o = 0;
#pragma unroll
    for (int k = 1; k < 8; ++k)
      if (item >= (diag_off[k] - base) * ngroups) o = k;
    const int d0 = diag_off[o], ntd = diag_off[o + 1] - d0;
    item -= (d0 - base) * ngroups;
    t = item % ntd;
    grp = item / ntd;
    const gptr<const int32_t> diag_tiles = as_global(G_.diag_tiles);
#pragma unroll
    for (int j = 0; j < 3; ++j) tpos[j] = diag_tiles[(d0 + t) * 4 + j];
  }
  sweep_tile<T, DIM, TT, Y2WALL, EXT>(G_, o, grp, tpos, L, [] {});
}

}  // namespace

template <typename T, bool Y2WALL>
void launch_sweep_rule(const Batch<T> &B, int diag, hipStream_t st) {
  const int items = B.h_item_off[(size_t)diag * (B.nprob + 1) + B.nprob];
  if (items == 0) return;
  const int *off = B.d_item_off + (size_t)diag * (B.nprob + 1);
#define PDVM_SWEEP_E(D, X, E)                                                                           \
  hipLaunchKernelGGL((sweep_kernel<T, D, X, Y2WALL, E>), dim3(items), dim3(kWave), 0, st, B.d_geo, off, \
                     B.nprob, diag)
#define PDVM_SWEEP_T(D, E)              \
  if (B.tile_edge <= 4) PDVM_SWEEP_E(D, 4, E); \
  else PDVM_SWEEP_E(D, 8, E)
  // EXT: bit 0 psi (2D with tau fed back), bit 1 Shakhov, bit 2 Maxwell walls
  // (stencil rule 1 only, so never with Y2WALL)
  if constexpr (!Y2WALL) {
    if (B.maxwell) {
      if (B.dim == 2) {
        if (B.shakhov) { PDVM_SWEEP_T(2, 7); }
        else if (B.psi) { PDVM_SWEEP_T(2, 5); }
        else { PDVM_SWEEP_T(2, 4); }
      } else {
        if (B.shakhov) { PDVM_SWEEP_T(3, 6); }
        else { PDVM_SWEEP_T(3, 4); }
      }
      return;
    }
  }
  if (B.dim == 2) {
    if (B.shakhov) { PDVM_SWEEP_T(2, 3); }
    else if (B.psi) { PDVM_SWEEP_T(2, 1); }
    else { PDVM_SWEEP_T(2, 0); }
  } else {
    if (B.shakhov) { PDVM_SWEEP_T(3, 2); }
    else { PDVM_SWEEP_T(3, 0); }
  }
#undef PDVM_SWEEP_T
#undef PDVM_SWEEP_E
}

template <typename T>
hipError_t launch_sweep(const Batch<T> &B, int diag, hipStream_t st) {
  if (B.y2wall) launch_sweep_rule<T, true>(B, diag, st);
  else launch_sweep_rule<T, false>(B, diag, st);
  return hipGetLastError();
}

}  // namespace pdvm
