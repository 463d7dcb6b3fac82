// Step (i) of the iteration (Sec. 3.1, Algorithm 1) on gfx950 for 2D problems:
// the row pipeline of dvm_sweep_rows.hip for 4 x 4 tiles, with the voxels'
// records broadcast between lanes instead of through LDS.
#pragma once
#include "dvm_device.h"

namespace pdvm {
namespace {

// The counter of a band and chain, `pad` ints each (more than 2^31 ints for the tallest
// problems that fit the memory: 280 M one-voxel rows, four chains).
__host__ __device__ constexpr int64_t counter_at(int band, int nchains, int c, int pad) {
  return ((int64_t)band * nchains + c) * pad;
}
static_assert(counter_at(35000000, 4, 3, kProgPad) == 4480000096ll, "counter offsets are 64-bit");

// The pipeline, its hand-overs, its waits and their protocols are those of
// sweep_rows_kernel. What differs:
//
// Records. A record is the same for all 64 velocities of a wavefront, but FMAs
// need it in every lane. Read from LDS, ten FP64 values a voxel are 5 KB of LDS
// return traffic (128 bytes per clock and CU: 40 clocks a voxel and wavefront,
// 320 for the CU's eight), which set the pace: 6200 clocks per tile step. A
// 4 x 4 tile has as many voxels as a DPP row has lanes, so here lane l holds
// the record of voxel l % 16 in registers, and the FMAs read voxel v's value as
// a row_newbcast operand: no LDS read, no extra instruction (a move where the
// value is an addend). LDS holds the reciprocal denominators and the ring.
//
// Stores. One buffer resource per voxel row; a voxel that is not stored (solid,
// or outside a ragged tile) takes an offset past its range, which the hardware
// drops. A tile always issues 16 stores with no branch around them, so a wait
// for the next tile's record data (loaded a tile ahead) is counted exactly and
// never waits for this tile's stores; a branch around each store made it drain
// them every tile.
//
// Bands. A wait for any load also waits for the wavefront's older stores (the
// counter of vector-memory operations is in order), so a wavefront that stores
// tiles cannot poll the band below, or load its halo, without draining them
// (2600 clocks a tile measured, as long as the tile). So a block has one more
// wavefront, the importer, which stores nothing: it polls the band below,
// loads the halo rows of the band's first row and hands them over through
// LDS, like every row to the next. A band's top wavefront publishes tile a - 1
// before it walks tile a (the stores have then reached the L2 with hardly a
// stall), each counter on a line of its own: with the counters of several
// chains, written from several XCDs, on one line a poll took over 1 us.
//
// Solid tiles. A tile without fluid hands on zeros, which only ever meet zero
// coefficients, without waiting for the row below: it costs a third of a tile,
// and the rows above it do not depend on those below it.
//
// Hand-overs read the counter and the data together (a wavefront's LDS
// accesses are performed in order) and look again only if the counter shows
// that the data came too late.
//
// What bounds it: the issue of about 500 instructions per tile and wavefront,
// two wavefronts to a SIMD (1.6 us per tile; one alone takes 1.2), and the 0.7
// us from a row to the next one above.
// Measured (MI355X, sweep per iteration, this kernel against sweep_rows_kernel
// with 4 x 4 tiles): 512^2 rock with 32 x 32 velocities FP64 664 -> 418 us,
// FP32 533 -> 322 us; 540^2 image with 8 x 8 velocities FP64 612 -> 406 us;
// 64^2 cell with 16 x 16 velocities FP64 73 -> 52 us, 203 x 157 with 16 x 16
// velocities, tau, Shakhov and Maxwell walls FP64 421 -> 233 us (one branch and one
// load after the other per voxel at a wall, against one round trip per axis of a tile).
template <typename T, bool LOCAL, int NW, int EXT>
__global__ void __launch_bounds__(kWave * (NW + 1))
    sweep_rows4_kernel(const Geo<T> *__restrict__ G, const int *__restrict__ row_off, int nprob, int stride,
                       int32_t *__restrict__ prog_scr, int pad, uint8_t *__restrict__ xcc_scr) {
  constexpr int DIM = 2, TT = 4, NC = 16;
  constexpr int RING = 2, RING_IN = 4;  // slots of each hand-over: from the row below, from the importer
  constexpr bool TAU = (EXT & 1) != 0, SH = (EXT & 2) != 0, MW = (EXT & 4) != 0;
  // 8 MiB past any row's range (1 GiB), so also from columns that a ragged or narrow
  // tile does not have, up to three voxels of 32 KiB before the row's start; the bits
  // of 4.0f, an inline constant (a literal costs the FP32 sweeps 1 %)
  constexpr uint32_t kDrop = 0x40800000u;
  __shared__ T rd_lds[4 * kWave];
  // wavefront w reads its bottom halo from slot a of ring_of(w)
  __shared__ T ring[(NW - 1) * RING + RING_IN][2 * TT][kWave];
  __shared__ int32_t made[NW], used[NW];
  const int p = nprob > 1 ? owner_of(row_off, nprob, blockIdx.x) : 0;
  const Geo<T> &G_ = G[p];
  if (!G_.run) return;
  const Dom<T> dm = dom_of(G_);
  const int ngroups = G_.ngroups, Ko = G_.Ko, Ko_pad = G_.Ko_pad;
  const int tile0 = G_.tile[0], tile1 = G_.tile[1];
  const int ntile0 = G_.ntile[0], ntile1 = G_.ntile[1];
  const gptr<T> hc = as_global(G_.hcur);
  const gptr<const T> hp = as_global(G_.hprev);
  const gptr<const T> src = as_global(G_.srccur);
  const gptr<const T> srct = as_global(G_.srctcur);
  const gptr<const T> srcq = as_global(G_.srcqcur);
  const gptr<const T> wall = as_global(G_.wallcur);
  const gptr<const uint32_t> flags = as_global(G_.flags);
  const int row0 = nprob > 1 ? row_off[p] : 0;
  const gptr<int32_t> progress = as_global(prog_scr ? prog_scr + (int64_t)row0 * pad : G_.progress);
  const gptr<int32_t> fault = as_global(&G_.ctl->fault);
  const uint32_t seq = (uint32_t)G_.seq;
  const int n0 = dm.n[0], n1 = dm.n[1];
  const int nchains = ngroups << DIM;
  const int local_b = blockIdx.x - row0;
  const int c = local_b % stride;
  const int band = local_b / stride;
  if (c >= nchains) return;  // padding of the band to a multiple of 8 blocks
  if (LOCAL && threadIdx.x == 0) {
    uint32_t xcc;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
    as_global(xcc_scr ? xcc_scr + row0 : G_.xcc_seen)[local_b] = (uint8_t)(xcc & 0xFFu);
  }
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const int j = band * NW + w;  // tile row in sweep order
  const int grp = c % ngroups;
  const int o = c / ngroups;
  const int q = grp * kWave + lane;
  const int qq = q < Ko ? q : Ko - 1;  // lanes past the octant copy its last slot
  int s[2], sidx[2], pin[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    sidx[k] = (o >> k) & 1;
    s[k] = sidx[k] ? -1 : 1;
    pin[k] = 1 - sidx[k];
  }
  const T ph = TAU ? as_global(G_.phm)[qq] : T(1);
  Dom<T> dv = dm;
  if (TAU) dv.jump = dm.jump * ph;
  T vv[2], aa[2], cq[2] = {T(0), T(0)}, am[2] = {T(0), T(0)};
  const T spec = G_.spec, alpha = G_.alpha;
  const T qs = SH ? as_global(G_.qsf)[qq] : T(0);
#pragma unroll
  for (int k = 0; k < DIM; ++k) {
    const T a = as_global(G_.absv)[k * Ko_pad + qq];
    const T av = a * ph;
    vv[k] = s[k] > 0 ? av : -av;
    aa[k] = as_global(G_.av)[k * Ko_pad + qq];
    if (SH) cq[k] = (s[k] > 0 ? a : -a) * qs;
    if (MW) am[k] = aa[k] * spec;
  }
  const T vsqm = TAU ? as_global(G_.vsqm)[qq] : T(0);
  if (w == 0) {
#pragma unroll
    for (int k = 0; k < 4; ++k) rd_lds[k * kWave + lane] = as_global(G_.rden)[k * Ko_pad + qq];
  }
  if (lane == 0 && w < NW) {
    made[w] = 0;
    used[w] = 0;
  }
  __syncthreads();          // the only block-wide barrier
  const int kofs = o * Ko_pad + qq;
  const uint32_t colb = (uint32_t)(dm.Kpad * (int64_t)sizeof(T));  // bytes per voxel
  const uint32_t dcol = s[0] > 0 ? colb : 0u - colb;               // and from one column to the next
  int kmir[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) kmir[k] = (o ^ (1 << k)) * Ko_pad + qq;
  const int64_t wait_ticks = G_.wait_ticks;
  // as in sweep_rows_kernel; LDS polls do not sleep (a hand-over is on the
  // critical path of every row above)
  auto bounded_wait = [&](auto ready, bool sleep) __attribute__((always_inline)) {
    if (ready()) return;
    int n = 0;
    int64_t t0 = 0;
    __builtin_amdgcn_s_setprio(0);  // a polling wavefront leaves the issue slots to the walking ones
    while (!ready()) {
      if ((++n & 127) == 0) {
        const int64_t t = wall_clock64();
        if (__hip_atomic_load(fault, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) break;
        if (n == 128) {
          t0 = t;
        } else if (t - t0 > wait_ticks) {
          __hip_atomic_store(fault, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          break;
        }
      }
      if (sleep) __builtin_amdgcn_s_sleep(1);
    }
    __builtin_amdgcn_s_setprio(2);
  };
  auto lds_get = [](int32_t *ctr) __attribute__((always_inline)) {
    const int32_t v = __hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);  // no LDS access below is moved above
    return v;
  };
  auto lds_wait = [&](int32_t *ctr, int32_t want) __attribute__((always_inline)) {
    bounded_wait([&] { return __hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) >= want; }, false);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
  };
  auto lds_post = [&](int32_t *ctr, int32_t v) __attribute__((always_inline)) {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this wavefront's LDS accesses are done
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __hip_atomic_store(ctr, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  auto slot_of = [](int w, int a) __attribute__((always_inline)) {
    return w == 0 ? (NW - 1) * RING + a % RING_IN : (w - 1) * RING + a % RING;
  };
  // a tile's first column in sweep order and its width
  auto xs_of = [&](int a, int &cnt0) __attribute__((always_inline)) {
    const int lo0 = (s[0] > 0 ? a : ntile0 - 1 - a) * tile0;
    cnt0 = min(tile0, n0 - lo0);
    return s[0] > 0 ? lo0 : lo0 + cnt0 - 1;
  };
  // a tile row's first voxel row in sweep order and its height
  auto ys_of = [&](int row, int &cnt1) __attribute__((always_inline)) {
    const int lo1 = (s[1] > 0 ? row : ntile1 - 1 - row) * tile1;
    cnt1 = min(tile1, n1 - lo1);
    return s[1] > 0 ? lo1 : lo1 + cnt1 - 1;
  };

  __builtin_amdgcn_s_setprio(2);
  if (w == NW) {  // the importer
    int cnt1;
    const int ys = ys_of(band * NW, cnt1);
    const gptr<int32_t> wait_on = progress + (band > 0 ? counter_at(band - 1, nchains, c, pad) : 0);
    const uint32_t base = seq * (uint32_t)ntile0;
    // the band below's progress in tiles, as last seen: a look at it before each
    // tile's loads (LOCAL) mostly saves the next tile its poll. The look is waited for
    // before the loads are issued (`base` is subtracted at once): two round trips a tile
    auto look = [&]() __attribute__((always_inline)) {
      return (int32_t)((uint32_t)__hip_atomic_load(wait_on, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - base);
    };
    int32_t got = 0;
    // the two voxel rows below and this lane's slot in them: of the current
    // sweep, or (first band) the images of the previous iterate
    __amdgpu_buffer_rsrc_t below[2];
    uint32_t vk[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int y = ys - (r + 1) * s[1];
      const bool in = y >= 0 && y < n1;
      const Img im = image_of(1, y, n1, dm.latp);
      below[r] = __builtin_amdgcn_make_buffer_rsrc(
          (void *)((gptr<char>)(in ? hc : (gptr<T>)(T *)G_.hprev) + (uint64_t)(uint32_t)((in ? y : im.r) * n0) * colb),
          (short)0, (int)(colb * (uint32_t)n0), kBufferFlags);
      vk[r] = (uint32_t)(!in && im.mir ? kmir[1] : kofs) * (uint32_t)sizeof(T);
    }
    for (int a = 0; a < ntile0; ++a) {
      if (band > 0 && got < a + 1) {
        bounded_wait(
            [&] {
              got = look();
              return got >= a + 1;
            },
            false);
        if (!LOCAL) __atomic_thread_fence(__ATOMIC_ACQUIRE);  // agent scope: the producer's stores are visible
      }
      __atomic_signal_fence(__ATOMIC_SEQ_CST);  // no load below is moved above the poll
      int cnt0;
      const int xs = xs_of(a, cnt0);
      T b[2][TT];
      const int32_t ahead = LOCAL && band > 0 ? look() : 0;
      const uint32_t at = (uint32_t)xs * colb;
#pragma unroll
      for (int k = 0; k < TT; ++k) {
        // columns past the tile re-read its last one: only voxels outside the
        // tile, never stored, see them
        const uint32_t vo = at + (uint32_t)min(k, cnt0 - 1) * dcol;
        b[0][k] = buffer_load<T>(below[0], vk[0] + vo);
        b[1][k] = buffer_load<T>(below[1], vk[1] + vo);
      }
      lds_wait(&used[0], a + 1 - RING_IN);
      T(*const to)[kWave] = ring[slot_of(0, a)];
#pragma unroll
      for (int k = 0; k < TT; ++k) {
        to[k][lane] = b[0][k];
        to[TT + k][lane] = b[1][k];
      }
      lds_post(&made[0], a + 1);
      if (LOCAL) got = max(got, ahead);
    }
    return;
  }
  if (j >= ntile1) return;  // the last band may be partial

  int cnt1;
  const int ys = ys_of(j, cnt1);
  const bool lmake = w < NW - 1 && j + 1 < ntile1;   // top rows to the wavefront above (LDS)
  const bool gmake = w == NW - 1 && j + 1 < ntile1;  // progress to the band above
  // tiles one voxel high: the band above reads the rows of the top two wavefronts
  const bool thin = tile1 == 1, second = thin && lmake && w == NW - 2;
  const gptr<int32_t> publish = progress + counter_at(band, nchains, c, pad);
  // one resource per voxel row (below 1 GiB, checked by the host); rows past a
  // ragged tile repeat its last one and store nothing
  __amdgpu_buffer_rsrc_t rowrs[TT];
#pragma unroll
  for (int k = 0; k < TT; ++k)
    rowrs[k] = __builtin_amdgcn_make_buffer_rsrc(
        (void *)((gptr<char>)hc + (uint64_t)(uint32_t)((ys + min(k, cnt1 - 1) * s[1]) * n0) * colb), (short)0,
        (int)(colb * (uint32_t)n0), kBufferFlags);
  const uint32_t kst = (uint32_t)kofs * (uint32_t)sizeof(T);
  using lds_ptr = __attribute__((address_space(3))) const T *;
  const uint32_t rd_addr = (uint32_t)(uintptr_t)(lds_ptr)(rd_lds + lane);

  // the record data of voxel lane % 16 of tile a (in sweep order: column
  // lane % 4, row lane / 4 % 4). Unconditional loads: lanes outside the tile
  // read one of its voxels, and `build` takes theirs as solid.
  struct Raw {
    uint32_t f;
    T sv[3], svt, wv[2], sq[2];
  };
  const int vi = lane & 3, vr = (lane >> 2) & 3;
  // 32-bit offsets from the tile row's lowest-addressed voxel row
  const int ylo = s[1] > 0 ? ys : ys - (cnt1 - 1);
  const uint64_t rowc = (uint64_t)(uint32_t)(ylo * n0);
  const gptr<const char> flags_r = (gptr<const char>)(flags + rowc), src_r = (gptr<const char>)(src + rowc * kSrcStride),
                         srct_r = (gptr<const char>)(srct + rowc), srcq_r = (gptr<const char>)(srcq + rowc * 4),
                         wall_r0 = (gptr<const char>)(wall + rowc * 6 + pin[0]),
                         wall_r1 = (gptr<const char>)(wall + rowc * 6 + 2 + pin[1]);
  const bool vrow = vr < cnt1;
  const uint32_t vrc = vrow ? (uint32_t)((s[1] > 0 ? vr : cnt1 - 1 - vr) * n0) : 0u;
  auto fetch = [&](int a, Raw &R) __attribute__((always_inline)) {
    int cnt0;
    const int xs = xs_of(a, cnt0);
    const uint32_t m = (uint32_t)min(vi, cnt0 - 1);
    const uint32_t cc = s[0] > 0 ? vrc + (uint32_t)xs + m : vrc + (uint32_t)xs - m;
    R.f = *(gptr<const uint32_t>)(flags_r + cc * 4u);
    const gptr<const T> sp = (gptr<const T>)(src_r + cc * (uint32_t)(kSrcStride * sizeof(T)));
#pragma unroll
    for (int k = 0; k < 3; ++k) R.sv[k] = sp[k];
    if (TAU) R.svt = *(gptr<const T>)(srct_r + cc * (uint32_t)sizeof(T));
    const uint32_t wo = ((cc << 1) + cc) * (uint32_t)(2 * sizeof(T));
    R.wv[0] = *(gptr<const T>)(wall_r0 + wo);
    R.wv[1] = *(gptr<const T>)(wall_r1 + wo);
    if (SH) {
      const gptr<const T> qp = (gptr<const T>)(srcq_r + cc * (uint32_t)(4 * sizeof(T)));
      R.sq[0] = qp[0];
      R.sq[1] = qp[1];
    }
  };
  // this lane's voxel's record: sources, per axis (c1, c2, w), the feedback
  // source and the heat flux; the LDS offset of its reciprocal denominators;
  // what its store offset adds (0, or past the row's range). A solid voxel (or
  // one outside the tile) takes no upstream values: it computes something finite
  // that nothing reads and that is not stored.
  T rs[3], rc1[2], rc2[2], rw[2], rt = T(0), rq[2] = {T(0), T(0)};
  uint32_t rdo, rdrop;
  // MW: per axis, 0 for a voxel whose stencil meets a wall, else past the row's range
  uint32_t rm[2] = {kDrop, kDrop};
  bool walls = false;  // MW: some voxel's does
  bool live = true;  // the tile holds fluid (or is one row thick: it hands on the row below)
  auto build = [&](const Raw &R, int a) __attribute__((always_inline)) {
    int cnt0;
    xs_of(a, cnt0);
    const bool fl = vi < cnt0 && vrow && !(R.f & F_SOLID);
    uint32_t code = 0;
    walls = false;
#pragma unroll
    for (int k = 0; k < 3; ++k) rs[k] = reg_copy(R.sv[k]);
    if (TAU) rt = reg_copy(R.svt);
    if (SH) {
      rq[0] = reg_copy(R.sq[0]);
      rq[1] = reg_copy(R.sq[1]);
    }
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
      const uint32_t fj = R.f >> fbit(k, sidx[k]);
      const bool first = fj & 1u, y1s = fj & 2u;
      rc1[k] = fl ? (first ? (y1s ? T(0) : T(1)) : T(2)) : T(0);
      rc2[k] = fl && !first ? T(-0.5) : T(0);
      const bool at_wall = fl && first && y1s;
      rw[k] = at_wall ? (MW ? alpha * R.wv[k] : R.wv[k]) : T(0);
      if (MW) {
        rm[k] = at_wall ? 0u : kDrop;
        walls = walls || __ballot(at_wall) != 0;
      }
      code |= (first ? 1u : 0u) << k;
    }
    rdo = fl ? code * (uint32_t)(kWave * sizeof(T)) : 0u;
    rdrop = fl ? 0u : kDrop;
    live = __ballot(fl) != 0 || cnt1 == 1;
    // a DPP operand may be read two instructions after its write at the earliest
    // ("+v": the values are those of this point, not formed again after it)
    asm volatile("s_nop 1"
                 : "+v"(rs[0]), "+v"(rs[1]), "+v"(rs[2]), "+v"(rc1[0]), "+v"(rc1[1]), "+v"(rc2[0]), "+v"(rc2[1]),
                   "+v"(rw[0]), "+v"(rw[1]), "+v"(rdo), "+v"(rdrop));
    if (TAU) asm volatile("s_nop 1" : "+v"(rt));
    if (SH) asm volatile("s_nop 1" : "+v"(rq[0]), "+v"(rq[1]));
    if (MW) asm volatile("s_nop 1" : "+v"(rm[0]), "+v"(rm[1]));
  };
  T L1[TT], L2[TT];  // left halo: previous tile's last two columns, or images across the x1 wrap
#pragma unroll
  for (int k = 0; k < TT; ++k) L1[k] = L2[k] = T(0);
  Raw nxt;
  fetch(0, nxt);
  {
    int cnt0;
    const int xs = xs_of(0, cnt0);
#pragma unroll
    for (int k = 0; k < TT; ++k)
      if (k < cnt1) {
        const int y = ys + k * s[1];
        L1[k] = upstream_fluid(dv, hc, hp, 0, xs - s[0], y, 0, kofs, kmir[0]);
        L2[k] = upstream_fluid(dv, hc, hp, 0, xs - 2 * s[0], y, 0, kofs, kmir[0]);
      }
  }
  build(nxt, 0);
  fetch(min(1, ntile0 - 1), nxt);
  // nothing is in flight when the loop is entered, so that the waits inside it
  // are counted from its own loads and stores alone
  __builtin_amdgcn_s_waitcnt(0);

  // the fewest loads that `fetch` can become: the flags, the sources (one, if they
  // are merged) and two wall values, all from addresses of their own. The fence before
  // the loop's fetch and the one in the wait keep them between the stores and it.
  constexpr int kRecordLoads = 4;
  // by one lane, when the stores of tiles below a are in the L2; the release of the
  // agent-scope protocol also writes back what other wavefronts of the block stored
  auto post_progress = [&](int a) __attribute__((always_inline)) {
    __hip_atomic_store(publish, (int32_t)(seq * (uint32_t)ntile0 + (uint32_t)a),
                       LOCAL ? __ATOMIC_RELAXED : __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
  };
  for (int a = 0; a < ntile0; ++a) {
    int cnt0;
    const int xs = xs_of(a, cnt0);
    auto publish_last = [&]() __attribute__((always_inline)) {
      if (a == 0 || !(second || (gmake && (LOCAL || thin)))) return;
      // tile a - 1's stores were followed by the loads of a record: with at most
      // as many operations outstanding they are in the L2
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kRecordLoads) : "memory");
      if (second) return;  // the hand-over of tile a says so
      if (lane == 0) post_progress(a);
    };
    T N[NC], B1[TT];
    const int32_t room = lmake ? lds_get(&used[w + 1]) : 0;  // looked at after the walk
    if (live) {
      // --- what does not depend on the halo: the sources and the denominators ----
      T num[NC], rdv[NC];
      auto read_rd = [&]() __attribute__((always_inline)) {
        static_for<NC>([&](auto V) __attribute__((always_inline)) {
          constexpr int v = V;
          rdv[v] = *(lds_ptr)(uintptr_t)add_bcast<v>(rdo, rd_addr);
        });
      };
      if (!MW) read_rd();
      static_for<NC>([&](auto V) __attribute__((always_inline)) {
        constexpr int v = V;
        T x = bcast<v>(rs[0]);
        if (TAU) x = x * ph;
        fmac_bcast<v>(x, rs[1], vv[0]);
        fmac_bcast<v>(x, rs[2], vv[1]);
        if (TAU) fmac_bcast<v>(x, rt, vsqm);
        if (SH) {
          fmac_bcast<v>(x, rq[0], cq[0]);
          fmac_bcast<v>(x, rq[1], cq[1]);
        }
        num[v] = x;
      });
      if constexpr (MW) {
        // a voxel at a wall along axis k: a_k (1 - alpha) times its own previous
        // iterate at the velocity mirrored in e_k. The loads of the tile's voxels go
        // together (those of voxels at no wall are dropped and give 0), one
        // round trip per axis of a tile that meets walls
        if (walls) {
          const gptr<char> hpb = (gptr<char>)(gptr<T>)(T *)G_.hprev;
          static_for<2>([&](auto K) __attribute__((always_inline)) {
            constexpr int k = K;
            const uint32_t at = (uint32_t)kmir[k] * (uint32_t)sizeof(T) + (uint32_t)xs * colb;
            T hm[NC];
            static_for<NC>([&](auto V) __attribute__((always_inline)) {
              constexpr int v = V;
              hm[v] = buffer_load<T>(
                  __builtin_amdgcn_make_buffer_rsrc(
                      (void *)(hpb + (uint64_t)(uint32_t)((ys + min(v / TT, cnt1 - 1) * s[1]) * n0) * colb), (short)0,
                      (int)(colb * (uint32_t)n0), kBufferFlags),
                  add_bcast<v>(rm[k], at + (uint32_t)(v % TT) * dcol));
            });
            static_for<NC>([&](auto V) __attribute__((always_inline)) {
              constexpr int v = V;
              num[v] = fma(am[k], hm[v], num[v]);
            });
          });
        }
      }
      if (MW) read_rd();  // registers: after the walls' loads
      // --- bottom halo ------------------------------------------------------------
      T B2[TT];
      {
        T(*const from)[kWave] = ring[slot_of(w, a)];
        auto read = [&]() __attribute__((always_inline)) {
#pragma unroll
          for (int k = 0; k < TT; ++k) {
            B1[k] = from[k][lane];
            B2[k] = from[TT + k][lane];
          }
        };
        const int32_t there = lds_get(&made[w]);
        read();
        if (there < a + 1) {
          lds_wait(&made[w], a + 1);
          read();
        }
        lds_post(&used[w], a + 1);
      }
      publish_last();
      // --- the tile's anti-diagonals ------------------------------------------------
      static_for<2 * TT - 1>([&](auto Dg) __attribute__((always_inline)) {
        constexpr int d = Dg;
        // the anti-diagonal's voxels are independent: operation by operation, so
        // that no FMA waits for the one before it
        T y1[TT], y2[TT];
        auto each = [&](auto f) __attribute__((always_inline)) {
          static_for<TT>([&](auto R) __attribute__((always_inline)) {
            constexpr int r = R, i = d - r;
            if constexpr (i >= 0 && i < TT) f(std::integral_constant<int, r>{}, std::integral_constant<int, i>{});
          });
        };
        each([&](auto R, auto I) __attribute__((always_inline)) {
          constexpr int r = R, v = I + TT * r;
          y1[r] = bcast<v>(rw[0]);
          if (TAU) y1[r] = y1[r] * ph;
        });
        each([&](auto R, auto I) __attribute__((always_inline)) {
          constexpr int r = R, v = I + TT * r;
          y2[r] = bcast<v>(rw[1]);
          if (TAU) y2[r] = y2[r] * ph;
        });
        each([&](auto R, auto I) __attribute__((always_inline)) {
          constexpr int r = R, i = I, v = i + TT * r;
          fmac_bcast<v>(y1[r], rc2[0], i >= 2 ? N[i >= 2 ? v - 2 : 0] : (i == 1 ? L1[r] : L2[r]));
        });
        each([&](auto R, auto I) __attribute__((always_inline)) {
          constexpr int r = R, i = I, v = i + TT * r;
          fmac_bcast<v>(y2[r], rc2[1], r >= 2 ? N[r >= 2 ? v - 2 * TT : 0] : (r == 1 ? B1[i] : B2[i]));
        });
        each([&](auto R, auto I) __attribute__((always_inline)) {
          constexpr int r = R, i = I, v = i + TT * r;
          fmac_bcast<v>(y1[r], rc1[0], i >= 1 ? N[i >= 1 ? v - 1 : 0] : L1[r]);
        });
        each([&](auto R, auto I) __attribute__((always_inline)) {
          constexpr int r = R, i = I, v = i + TT * r;
          fmac_bcast<v>(y2[r], rc1[1], r >= 1 ? N[r >= 1 ? v - TT : 0] : B1[i]);
        });
        each([&](auto R, auto I) __attribute__((always_inline)) {
          constexpr int r = R, v = I + TT * r;
          num[v] = fma(aa[0], y1[r], num[v]);
        });
        each([&](auto R, auto I) __attribute__((always_inline)) {
          constexpr int r = R, v = I + TT * r;
          num[v] = fma(aa[1], y2[r], num[v]);
        });
        each([&](auto R, auto I) __attribute__((always_inline)) {
          constexpr int r = R, v = I + TT * r;
          N[v] = num[v] * rdv[v];
        });
      });
    } else {
      __hip_atomic_store(&used[w], a + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      publish_last();
#pragma unroll
      for (int k = 0; k < NC; ++k) N[k] = T(0);
#pragma unroll
      for (int k = 0; k < TT; ++k) B1[k] = T(0);
    }
    // --- hand the tile on ---------------------------------------------------------
    // its top two rows; a tile one voxel thick passes on its own and the one below
    if (lmake) {
      if (room < a + 1 - RING) lds_wait(&used[w + 1], a + 1 - RING);  // the slot's previous tile has been read
      T(*const to)[kWave] = ring[slot_of(w + 1, a)];
      if (cnt1 == TT) {
#pragma unroll
        for (int k = 0; k < TT; ++k) {
          to[k][lane] = N[3 * TT + k];
          to[TT + k][lane] = N[2 * TT + k];
        }
      } else {
#pragma unroll
        for (int k = 0; k < TT; ++k) {
          to[k][lane] = cnt1 == 3 ? N[2 * TT + k] : (cnt1 == 2 ? N[TT + k] : N[k]);
          to[TT + k][lane] = cnt1 == 3 ? N[TT + k] : (cnt1 == 2 ? N[k] : B1[k]);
        }
      }
      lds_post(&made[w + 1], a + 1);
    }
    // --- its stores (after the hand-over, which the rows above wait for) --------------
    uint32_t vx[TT];  // this lane's byte offset of column k in a row
#pragma unroll
    for (int k = 0; k < TT; ++k) vx[k] = kst + (uint32_t)xs * colb + (uint32_t)k * dcol;
    static_for<NC>([&](auto V) __attribute__((always_inline)) {
      constexpr int v = V;
      buffer_store(N[v], rowrs[v / TT], add_bcast<v>(rdrop, vx[v % TT]), 0u);
    });
    // the next tile's left halo: this tile's last two columns (a tile one voxel
    // wide passes on its own and the one before it)
    if (cnt0 == TT) {
#pragma unroll
      for (int k = 0; k < TT; ++k) {
        L1[k] = N[TT * k + 3];
        L2[k] = N[TT * k + 2];
      }
    } else {
#pragma unroll
      for (int k = 0; k < TT; ++k) {
        L2[k] = cnt0 == 3 ? N[TT * k + 1] : (cnt0 == 2 ? N[TT * k] : L1[k]);
        L1[k] = cnt0 == 3 ? N[TT * k + 2] : (cnt0 == 2 ? N[TT * k + 1] : N[TT * k]);
      }
    }
    // --- the next tile's records, and the data of the one after it ------------------
    build(nxt, min(a + 1, ntile0 - 1));
    if (!LOCAL && gmake && !thin && lane == 0) post_progress(a + 1);
    asm volatile("" ::: "memory");
    fetch(min(a + 2, ntile0 - 1), nxt);
  }
  if (second || (gmake && (LOCAL || thin))) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (second) {
      lds_post(&made[w + 1], ntile0 + 1);
    } else {
      if (thin) lds_wait(&made[w], ntile0 + 1);
      if (lane == 0) post_progress(ntile0);
    }
  }
}

}  // namespace
}  // namespace pdvm
