// The sweep as one launch of persistent wavefronts that take tiles from
// per-XCD queues (launch_sweep_queue).
#pragma once
#include "dvm_sweep_tile.h"

namespace pdvm {
namespace {

// Step (i) as one launch: per XCD, kQueueSub queues of packed tile items (the
// velocity chains, i.e. problem x octant x group, are dealt to the XCDs and
// their sub-queues, each chain to one), ordered by tile diagonal. Every block
// takes items from the queues of the XCD it runs on (one claim ahead: the
// next item's counter update is in flight during a tile, and a claim only
// ever waits on items claimed before it); before a tile it waits for the done flags of
// its upstream tiles along each axis (same chain, so the same queue and XCD),
// and after it drains its stores into the L2 and stamps the tile's flag with
// the iteration's seq (flags are never reset). A wait only ever concerns an
// item taken earlier by a running wavefront, so the queue cannot deadlock.
// Producer and consumer share the XCD's L2: relaxed agent-scope flag stores
// and polls, no cache write-back or invalidation; the consumer's L1 holds no
// line of the tile before the flag (a chain's lines are read only by its own
// downstream tiles, and lanes past the octant read their own group's slot).
// Waits are bounded (Geo::wait_ticks) and flag ctl->fault; the blocks count
// the items they handled, and the reduction discards an iterate whose count
// falls short (a queue without blocks on its XCD).
// Item: bits 0-23 tile index (x1 fastest), 24-26 octant, 27-31 group,
// 32-47 problem, 48-53 waits: bit 2 j + k - 1 = wait for the k-th tile
// upstream along axis j (k = 2 where the first is one voxel thick).
// COL (3D): an item is a segment of Geo::col_tiles tiles of a column along x3
// (bits 0-23 the column's x1 + nt0 x2 tile index, 48-63 the segment), ordered
// by the diagonal of its first tile; one wavefront sweeps its tiles in turn,
// each with the waits of Geo::qtinfo and its own flag, keeping the
// x3-upstream planes in registers from tile to tile (no x3 halo loads but at
// the segment's start).
// Occupancy (FP32): 4 wavefronts per SIMD in 2D (the 64-problem batch sweeps in
// 2.21 ms instead of 2.29 with 3), 3 in 3D (at 4 the 4x4 tile spills its x3
// planes: 5.8 ms on the 96^3 pack instead of 4.3, measured with records in LDS). At 3
// (168 VGPRs) tile items of 4x4 with stencil rule 1 do not spill (Maxwell walls with
// Shakhov: one register); with rule 0 10 - 13 registers, columns 3 - 37, and 8x8 tiles
// 48 - 90 (per-diagonal launches of those, without the bound, spill none: 48 x 44 x 40 with
// 16^3 velocities 1.00 ms a sweep against 1.21 from the queue).
template <typename T, int DIM, int TT, bool Y2WALL, int EXT, bool COL>
__global__ void __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? (DIM == 2 ? 4 : 3) : 1)))
    sweep_queue_kernel(const Geo<T> *__restrict__ G, const uint64_t *__restrict__ items,
                       const int32_t *__restrict__ q_off, int32_t *__restrict__ qctr, int32_t *__restrict__ qflags,
                       int nprob) {
  __shared__ TileLds<T, DIM, TT, EXT> L;
  if (nprob == 1 && !G[0].run) return;  // a stopped problem (its reduction checks nothing)
  uint32_t xcc;
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
  xcc &= 7u;
  const int lane = threadIdx.x;
  int handled = 0;
  // the XCD's sub-queues holding items (the host fills them from the first
  // on), starting with one picked by the block index; a block that finds one
  // drained moves on to the next
  const int *const xo = q_off + xcc * kQueueSub;
  int used = 0;
  for (int i = 0; i < kQueueSub; ++i) used += xo[i + 1] > xo[i];
  const int sub0 = used ? (int)((blockIdx.x >> 3) % used) : 0;
  for (int si = 0; si < used; ++si) {
    const int qi = (int)xcc * kQueueSub + (sub0 + si) % used;
    const int qb = q_off[qi], qn = q_off[qi + 1] - qb;
    int32_t *const ctr = &qctr[qi * kCtrPad];
    // claims run two ahead: the item word of the next claim is loaded, and the
    // claim after it is in flight, while a tile runs
    auto claim = [&]() __attribute__((always_inline)) {
      int c = 0;
      if (lane == 0) c = __hip_atomic_fetch_add(ctr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return c;
    };
    int k = __builtin_amdgcn_readfirstlane(claim());
    int kn = claim();
    uint64_t it = k < qn ? items[qb + k] : 0;
    while (k < qn) {
      kn = __builtin_amdgcn_readfirstlane(kn);
      const uint64_t itn = kn < qn ? items[qb + kn] : 0;
      const int knn = claim();
      ++handled;
      const int tile = (int)(it & 0xFFFFFFu), o = (int)((it >> 24) & 7u), grp = (int)((it >> 27) & 31u);
      const int p = (int)((it >> 32) & 0xFFFFu), wm = (int)((it >> 48) & 63u);
      const Geo<T> &G_ = G[p];
      if (G_.run) {
        const int32_t stamp = G_.seq;
        const int nt0 = G_.ntile[0], nt1 = G_.ntile[1];
        int32_t *const fl = qflags + G_.qflag_off + (int64_t)(o * G_.ngroups + grp) * G_.ntiles_all;
        // the upstream tiles' flags of tile wt with waits ww, polled by lane
        // b < 2 DIM for wait b, all at once, while the tile's first records
        // are being loaded
        int wt = tile, ww = wm;
        auto wait_upstream = [&]() __attribute__((always_inline)) {
          if (!ww) return;
          const int j = lane >> 1, kk = (lane & 1) + 1;
          const bool mine = lane < 2 * DIM && ((ww >> lane) & 1);
          const int stride = j == 0 ? 1 : (j == 1 ? nt0 : nt0 * nt1);
          const int up = mine ? wt - (((o >> j) & 1) ? -kk : kk) * stride : wt;
          int32_t *const fault = &G_.ctl->fault;
          const int64_t wait_ticks = G_.wait_ticks;
          int n = 0;
          int64_t t0 = 0;
          for (;;) {
            const bool ok = !mine || __hip_atomic_load(&fl[up], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == stamp;
            if (__all(ok)) break;
            if ((++n & 63) == 0) {
              const int64_t tn = wall_clock64();
              if (__hip_atomic_load(fault, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) break;
              if (n == 64) {
                t0 = tn;
              } else if (tn - t0 > wait_ticks) {
                if (lane == 0) __hip_atomic_store(fault, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
              }
            }
            __builtin_amdgcn_s_sleep(1);
          }
          __atomic_signal_fence(__ATOMIC_SEQ_CST);  // no load outside the tile is moved above the polls
        };
        // after a tile: its stores drained into the L2, then its flag stamped
        auto publish = [&](int t) __attribute__((always_inline)) {
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
          __builtin_amdgcn_s_waitcnt(0);  // every store of the tile has reached the L2
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
          if (lane == 0) __hip_atomic_store(&fl[t], stamp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();  // the next tile's records overwrite this tile's
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        };
        if constexpr (!COL) {
          const int tpos[3] = {tile % nt0, (tile / nt0) % nt1, tile / (nt0 * nt1)};
          sweep_tile<T, DIM, TT, Y2WALL, EXT>(G_, o, grp, tpos, L, wait_upstream);
          publish(tile);
        } else {
          // a column (tile = x1 + nt0 x2 tile index), or the segment wm of
          // col_tiles tiles of it: its tiles holding fluid in the octant's x3
          // order; the planes below a tile come in registers from the tile
          // before it, and are loaded from h at the segment's start and after
          // a tile without fluid (which is skipped, its flag never stamped).
          // Waits along x3 only where the tile below is another segment's.
          const int nt2 = G_.ntile[2], ncol = nt0 * nt1, S = G_.col_tiles;
          const int seg = (int)((it >> 48) & 0xFFFFu);
          const int cb0 = seg * S, cb1 = min(nt2, cb0 + S);
          const bool down = (o >> 2) & 1;
          const gptr<const int32_t> info = as_global(G_.qtinfo) + (int64_t)o * G_.ntiles_all;
          T zc[2 * TileLds<T, DIM, TT, EXT>::ZN];
          bool zload = true;
          int t = tile + (down ? nt2 - 1 - cb0 : cb0) * ncol;
          int inf = info[t];
          for (int cb = cb0; cb < cb1; ++cb) {
            const int tn = t + (down ? -ncol : ncol);
            const int infn = info[cb + 1 < cb1 ? tn : t];  // the next tile's, loaded ahead
            if (inf & 128) {
              const int tpos[3] = {tile % nt0, tile / nt0, t / ncol};
              wt = t;
              ww = inf & (15 | (cb == cb0 ? 48 : (cb == cb0 + 1 ? 32 : 0)));
              sweep_tile<T, DIM, TT, Y2WALL, EXT, true>(G_, o, grp, tpos, L, wait_upstream, zc, zload);
              publish(t);
              zload = false;
            } else {
              zload = true;
            }
            t = tn;
            inf = infn;
          }
        }
      }
      k = kn;
      kn = knn;
      it = itn;
    }
  }
  if (lane == 0)
    __hip_atomic_fetch_add(&qctr[(8 * kQueueSub + xcc) * kCtrPad], handled, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}

// The queue counters (taken per sub-queue, handled per XCD) before a queue
// sweep: a fill kernel, so that a captured graph holds no memset node.
__global__ void queue_reset_kernel(int32_t *qctr) {
  for (int i = threadIdx.x; i < kQueueCounters; i += blockDim.x) qctr[i * kCtrPad] = 0;
}

}  // namespace

template <typename T, bool Y2WALL>
void launch_queue_rule(const Batch<T> &B, hipStream_t st, int32_t *qctr, int32_t *qflags) {
  hipLaunchKernelGGL(queue_reset_kernel, dim3(1), dim3(128), 0, st, qctr);
  const dim3 grid(kQueueBlocks);
#define PDVM_QUEUE_C(D, X, E, C)                                                                             \
  hipLaunchKernelGGL((sweep_queue_kernel<T, D, X, Y2WALL, E, C>), grid, dim3(kWave), 0, st, B.d_geo, B.d_qitems, \
                     B.d_q_off, qctr, qflags, B.nprob)
#define PDVM_QUEUE_E(D, X, E)                                   \
  if (D == 3 && B.use_columns) PDVM_QUEUE_C(D, X, E, D == 3); \
  else PDVM_QUEUE_C(D, X, E, false)
#define PDVM_QUEUE_T(D, E)                          \
  if (B.tile_edge <= 4) PDVM_QUEUE_E(D, 4, E);      \
  else PDVM_QUEUE_E(D, 8, E)
  if constexpr (!Y2WALL) {
    if (B.maxwell) {
      if (B.dim == 2) {
        if (B.shakhov) { PDVM_QUEUE_T(2, 7); }
        else if (B.psi) { PDVM_QUEUE_T(2, 5); }
        else { PDVM_QUEUE_T(2, 4); }
      } else {
        if (B.shakhov) { PDVM_QUEUE_T(3, 6); }
        else { PDVM_QUEUE_T(3, 4); }
      }
      return;
    }
  }
  if (B.dim == 2) {
    if (B.shakhov) { PDVM_QUEUE_T(2, 3); }
    else if (B.psi) { PDVM_QUEUE_T(2, 1); }
    else { PDVM_QUEUE_T(2, 0); }
  } else {
    if (B.shakhov) { PDVM_QUEUE_T(3, 2); }
    else { PDVM_QUEUE_T(3, 0); }
  }
#undef PDVM_QUEUE_T
#undef PDVM_QUEUE_E
#undef PDVM_QUEUE_C
}

template <typename T>
hipError_t launch_sweep_queue(const Batch<T> &B, hipStream_t st, const Scratch &scr) {
  int32_t *qctr = scr.qctr ? scr.qctr : B.d_qctr;
  int32_t *qflags = scr.qflags ? scr.qflags : B.d_qflags;
  if (B.y2wall) launch_queue_rule<T, true>(B, st, qctr, qflags);
  else launch_queue_rule<T, false>(B, st, qctr, qflags);
  return hipGetLastError();
}

}  // namespace pdvm
