// Step (i) of the iteration (Sec. 3.1, Algorithm 1) on gfx950: the upwind sweep
// (Eq. numerical stencil, Eq. Discretised_linearised_Boltzmann_equations) of one
// tile by one wavefront, for 2D and 3D problems and batches. Included by the
// sources of the queue sweep and of the per-diagonal sweep, one per precision
// (four, so that they compile side by side).
#pragma once
#include "dvm_device.h"

namespace pdvm {
namespace {

// Step (i) for one diagonal of tiles. One wavefront = one tile x 64 discrete
// velocities of one sign octant (lanes = velocities), so every per-voxel
// decision is wavefront-uniform and each voxel's 64 values are one contiguous
// store. The tile is TT x TT voxels in (x1, x2), any depth along x3, walked
// plane by plane in the octant's order. Per plane, each lane first decodes one
// voxel of the plane into an LDS record (source coefficients and, per axis,
// the stencil weights on the two upstream values and the wall term); the
// wavefront then walks the plane's 2 TT - 1 anti-diagonals, whose voxels are
// independent of each other, so their loads and FMA chains overlap. The two
// previous anti-diagonals stay in registers; values outside the tile come
// from the current sweep of upstream tiles (earlier launches) or from the
// lagged images outside the domain.
// EXT bit 0 (PSI, 2D): slots of h and of psi; bit 1 (SH): the Shakhov
// heat-flux source, whose per-voxel values nu (4/5)(1 - Pr) q_j end the record;
// bit 2 (MW): Maxwell walls. A voxel whose axis-j stencil meets a wall (code
// bit 4 + j) adds a_j (1 - alpha) times its own previous-iteration value of
// the velocity mirrored in e_j; the record's wall term is alpha rho_w.
// h at an upstream node (x, y, z) along axis j, as upstream_fluid but without
// the jump across the x1 wrap (the caller adds it where the value is used, so
// nothing waits for the load early) and with no branch: the buffer, the node
// and the velocity slot are selected (uniform values), so the load is issued
// whatever the case and many can be in flight before the first wait.
// The node's offset is formed in 32 bits (a problem has under 2^31 / 6
// voxels) and scaled by the voxel's bytes colb in one 32 x 32 -> 64 bit
// product: these are scalar instructions, a dozen per halo value fewer than
// with 64-bit index arithmetic.
template <typename T>
__device__ __forceinline__ T upstream_sel(const Dom<T> &g, gptr<const T> hc, gptr<const T> hp, int j, int x, int y,
                                          int z, int kofs, int kmir, uint32_t colb) {
  int c[3] = {x, y, z};
  const bool in = c[j] >= 0 && c[j] < g.n[j];
  const Img im = image_of(j, c[j], g.n[j], g.latp);
  c[j] = in ? c[j] : im.r;
  const int k = (!in && im.mir) ? kmir : kofs;
  const uint32_t cell = (uint32_t)(c[0] + g.n[0] * (c[1] + g.n[1] * c[2]));
  const gptr<const char> b = (gptr<const char>)(in ? hc : hp) + (uint64_t)cell * colb;
  return ((gptr<const T>)b)[k];
}
// The jump that upstream_sel leaves out at x1 = x (images across the wrap).
template <typename T>
__device__ __forceinline__ T wrap_jump(const Dom<T> &g, int x) {
  return (x < 0 ? T(1) : (x >= g.n[0] ? T(-1) : T(0))) * g.jump;
}

// LDS of one tile wavefront: the reciprocal denominators of its 64
// velocities and the records of up to PZ planes (128 voxels in 3D).
template <typename T, int DIM, int TT, int EXT>
struct TileLds {
  static constexpr int NC = TT * TT;
  // a record: src (4), nu tau, per axis (c1, c2, w), [q]; its stride RW is
  // padded to 16 bytes, so that a voxel's record is read with 16-byte loads
  static constexpr int RW0 = 5 + 3 * DIM + ((EXT & 2) ? DIM : 0);
  static constexpr int RW = (RW0 * (int)sizeof(T) + 15) / 16 * 16 / (int)sizeof(T);
  static constexpr int PZ = DIM == 3 ? 128 / NC : 1;
  // 3D with 4 x 4 tiles: the two x3-upstream planes of the tile's voxels are
  // carried in registers, ZN values each (one unused value otherwise)
  static constexpr bool ZREG = DIM == 3 && TT == 4;
  static constexpr int ZN = ZREG ? NC : 1;
  T rd[8 * kWave];
  alignas(16) T rec[PZ * NC * RW];
  uint32_t rcode[PZ * NC];
};

// The sweep of one tile (physical tile coordinates tpos) for the 64 velocities
// of group grp in sign octant o; every value it reads outside the tile is final.
// `before` runs once the tile's first records are being loaded and before any
// value outside the tile is read (the queue sweep waits for its upstream tiles
// there). CARRY (3D, 4 x 4 tiles): zc holds the tile's x3-upstream planes
// one and two back (zc[0 .. ZN), zc[ZN .. 2 ZN)) as the caller carries them
// over from the tile below in the same column, unless zload asks for them to
// be loaded from h; it leaves holding the tile's last two planes.
template <typename T, int DIM, int TT, bool Y2WALL, int EXT, bool CARRY = false, typename Before>
__device__ __forceinline__ void sweep_tile(const Geo<T> &G_, int o, int grp, const int (&tpos)[3],
                                           TileLds<T, DIM, TT, EXT> &L, Before &&before, T *zc = nullptr,
                                           bool zload = true) {
  constexpr bool PSI = (EXT & 1) != 0, SH = (EXT & 2) != 0, MW = (EXT & 4) != 0;
  static_assert(!(MW && Y2WALL), "Maxwell walls need stencil rule 1");
  constexpr int NC = TT * TT;
  constexpr int RW = TileLds<T, DIM, TT, EXT>::RW;
  // 3D: the records of PZ planes (128 voxels) are staged at once, before any
  // store of them; KV voxels per lane
  constexpr int PZ = TileLds<T, DIM, TT, EXT>::PZ, KV = (PZ * NC + kWave - 1) / kWave;
  T *const rd_lds = L.rd;
  T *const rec = L.rec;
  uint32_t *const rcode = L.rcode;
  // every per-problem value is read once here; the loops below see registers
  const Dom<T> dm = dom_of(G_);
  const int Ko = G_.Ko, Ko_pad = G_.Ko_pad, tau_fb = G_.tau_fb;
  const int tile[3] = {G_.tile[0], G_.tile[1], G_.tile[2]};
  const gptr<const T> absv = as_global(G_.absv), avv = as_global(G_.av), rden = as_global(G_.rden),
                      vsq = as_global(G_.vsqm);
  const gptr<T> hc = as_global(G_.hcur);
  const gptr<const T> hcc = hc;
  const gptr<const T> hp = as_global(G_.hprev);
  const gptr<const T> src = as_global(G_.srccur);
  const gptr<const T> srct = as_global(G_.srctcur);
  const gptr<const T> srcq = as_global(G_.srcqcur);
  const gptr<const T> wall = as_global(G_.wallcur);
  const gptr<const uint32_t> flags = as_global(G_.flags);
  const int n0 = dm.n[0], n1 = dm.n[1];
  const int lane = threadIdx.x;
  const int q = grp * kWave + lane;
  const bool active = q < Ko;
  // a lane past the octant (last group only) reads the octant's last slot,
  // which its own wavefront owns: it touches no other wavefront's lines
  const int qq = active ? q : Ko - 1;
  const uint32_t colb = (uint32_t)(G_.Kpad * (int64_t)sizeof(T));  // bytes per voxel
  constexpr uint32_t kDrop = 0x40000000u;  // past any row's range; two of them do not wrap
  int s[3], sidx[3], pin[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    sidx[j] = (o >> j) & 1;
    s[j] = sidx[j] ? -1 : 1;
    pin[j] = 1 - sidx[j];  // incoming half at a wall emitting along s e_j has sign -s
  }
  // PSI: the lane's slot holds h (ph = 1) or psi (ph = 0), which has no
  // rho, u or wall term and no jump at the x1 wrap
  const T ph = PSI ? as_global(G_.phm)[qq] : T(1);
  Dom<T> dv = dm;  // as dm, with the jump this lane's values take
  if (PSI) dv.jump = dm.jump * ph;
  T vv[3] = {T(0), T(0), T(0)}, aa[3] = {T(0), T(0), T(0)}, cq[3] = {T(0), T(0), T(0)}, am[3] = {T(0), T(0), T(0)};
  const T qs = SH ? as_global(G_.qsf)[qq] : T(0);  // the Shakhov source's q.v factor
  const T spec = G_.spec, alpha = G_.alpha;
#pragma unroll
  for (int j = 0; j < DIM; ++j) {
    const T a = absv[j * Ko_pad + qq];
    const T av = a * ph;
    vv[j] = s[j] > 0 ? av : -av;
    aa[j] = avv[j * Ko_pad + qq];
    if (SH) cq[j] = (s[j] > 0 ? a : -a) * qs;
    if (MW) am[j] = aa[j] * spec;
  }
  T rdv[1 << DIM];  // written to LDS after the first records' loads are issued
#pragma unroll
  for (int c = 0; c < (1 << DIM); ++c) rdv[c] = rden[c * Ko_pad + qq];
  const T vsqm = tau_fb ? vsq[qq] : T(0);
  const int kofs = o * Ko_pad + qq;
  const uint32_t kst = active ? (uint32_t)kofs * (uint32_t)sizeof(T) : kDrop;  // the lane's byte offset in a voxel
  int kmir[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) kmir[j] = (o ^ (1 << j)) * Ko_pad + qq;

  int lo[3] = {0, 0, 0}, cnt[3] = {1, 1, 1};
#pragma unroll
  for (int j = 0; j < DIM; ++j) {
    lo[j] = tpos[j] * tile[j];
    cnt[j] = min(tile[j], dm.n[j] - lo[j]);
  }
  const int xs = s[0] > 0 ? lo[0] : lo[0] + cnt[0] - 1;
  const int ys = s[1] > 0 ? lo[1] : lo[1] + cnt[1] - 1;
  // 3D with 4 x 4 tiles: the two planes upstream along x3 of every voxel of
  // the tile's plane, ZA one plane back, ZB two, are loaded from h (or the
  // images) for the tile's first plane (or come with the column) and then
  // carried in registers from plane to plane (each voxel's new value replaces
  // ZA, whose value moves to ZB). 8 x 8 tiles read them from h per
  // anti-diagonal (128 more registers would cost them their occupancy).
  constexpr bool ZREG = TileLds<T, DIM, TT, EXT>::ZREG;
  constexpr int ZN = TileLds<T, DIM, TT, EXT>::ZN;
  T ZAl[ZN], ZBl[ZN];
  T *const ZA = CARRY ? zc : ZAl;
  T *const ZB = CARRY ? zc + ZN : ZBl;
  const int64_t Kp = dm.Kpad;
  const uint32_t dcol = s[0] > 0 ? colb : 0u - colb;  // bytes from one column to the next
  using lds_ptr = __attribute__((address_space(3))) const T *;
  const uint32_t rd_addr = (uint32_t)(uintptr_t)(lds_ptr)(rd_lds + lane);
  auto zof = [&](int c3) { return s[2] > 0 ? lo[2] + c3 : lo[2] + cnt[2] - 1 - c3; };
  // the halos of plane z (the current sweep, or the images of the previous
  // iterate outside the domain). Rows and columns past a ragged tile re-read
  // its last one: only voxels outside the tile, which are never stored, see them.
  auto load_halo = [&](int z, T(&L1)[TT], T(&L2)[TT], T(&B1)[TT], T(&B2)[TT]) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < TT; ++k) {
      const int y = ys + min(k, cnt[1] - 1) * s[1], x = xs + min(k, cnt[0] - 1) * s[0];
      L1[k] = upstream_sel(dv, hcc, hp, 0, xs - s[0], y, z, kofs, kmir[0], colb);
      L2[k] = upstream_sel(dv, hcc, hp, 0, xs - 2 * s[0], y, z, kofs, kmir[0], colb);
      B1[k] = upstream_sel(dv, hcc, hp, 1, x, ys - s[1], z, kofs, kmir[1], colb);
      B2[k] = upstream_sel(dv, hcc, hp, 1, x, ys - 2 * s[1], z, kofs, kmir[1], colb);
    }
  };
  // records of the voxels of planes c0 .. c0 + np - 1 (lane l takes voxels
  // l, l + 64, ...). The voxel's sources and wall values are loaded together
  // with its flags (valid addresses whatever the flags say) and every record
  // value is selected, not branched on, so one round trip serves them all.
  // `before` runs between the loads and the LDS writes (the queue sweep polls
  // its upstream tiles there, so the polls and these loads share a round trip)
  auto stage = [&](int c0, int np, auto &&before) __attribute__((always_inline)) {
    uint32_t f[KV];
    T sv[KV][5], wv[KV][DIM], qv[KV][DIM];
    int xy[KV][3];
#pragma unroll
    for (int kv = 0; kv < KV; ++kv) {
      const int v = lane + kv * kWave;
      const int pz = min(v / NC, np - 1), i = v % TT, r = (v / TT) % TT;
      const int x = xs + min(i, cnt[0] - 1) * s[0], y = ys + min(r, cnt[1] - 1) * s[1];
      const int z = zof(c0 + pz);
      xy[kv][0] = x;
      xy[kv][1] = y;
      xy[kv][2] = z;
      const int c = (y + n1 * z) * n0 + x;
      f[kv] = flags[c];
      const gptr<const T> sp = src + c * kSrcStride;
      sv[kv][0] = sp[0];
      sv[kv][1] = sp[1];
      sv[kv][2] = sp[2];
      sv[kv][3] = DIM == 3 ? sp[3] : T(0);
      sv[kv][4] = tau_fb ? srct[c] : T(0);
#pragma unroll
      for (int j = 0; j < DIM; ++j) {
        wv[kv][j] = wall[c * 6 + 2 * j + pin[j]];
        qv[kv][j] = SH ? srcq[c * 4 + j] : T(0);
      }
    }
    before();
#pragma unroll
    for (int kv = 0; kv < KV; ++kv) {
      const int v = lane + kv * kWave;
      if (KV * kWave > PZ * NC && v >= PZ * NC) break;
      const int pz = v / NC, i = v % TT, r = (v / TT) % TT;
      const bool in = pz < np && i < cnt[0] && r < cnt[1];
      const bool fl = in && !(f[kv] & F_SOLID);
      T *rp = rec + v * RW;
#pragma unroll
      for (int k = 0; k < 5; ++k) rp[k] = fl ? sv[kv][k] : T(0);  // a skipped voxel's record is 0: it computes 0
      if (SH) {
#pragma unroll
        for (int j = 0; j < DIM; ++j) rp[5 + 3 * DIM + j] = fl ? qv[kv][j] : T(0);
      }
      uint32_t code = 0;
#pragma unroll
      for (int j = 0; j < DIM; ++j) {
        const uint32_t fj = f[kv] >> fbit(j, sidx[j]);
        const bool first = fj & 1u, y1s = fj & 2u, y2s = fj & 4u;
        T c1 = first ? (y1s ? T(0) : T(1)) : T(2);
        T c2 = first ? T(0) : T(-0.5);
        T w = (first && y1s) ? (MW ? alpha * wv[kv][j] : wv[kv][j]) : T(0);
        if (Y2WALL && fl && !first && y2s) {
          c2 = T(0);
          w = T(-0.5) * wall_at_y1(dm, wall, j, s[j], pin[j], xy[kv][0], xy[kv][1], xy[kv][2]);
        }
        rp[5 + 3 * j] = fl ? c1 : T(0);
        rp[6 + 3 * j] = fl ? c2 : T(0);
        rp[7 + 3 * j] = fl ? w : T(0);
        code |= (first ? 1u : 0u) << j;
        if (MW && first && y1s) code |= 16u << j;
      }
      rcode[v] = fl ? code : R_SKIP;
    }
  };

  const T jx1 = wrap_jump(dv, xs - s[0]), jx2 = wrap_jump(dv, xs - 2 * s[0]);  // the same for every plane
  // the tile's first plane: records, halos and (4 x 4 tiles in 3D) the two
  // planes below, all issued before any wait
  T L1[TT], L2[TT], B1[TT], B2[TT];
  stage(0, min(PZ, cnt[2]), before);
#pragma unroll
  for (int c = 0; c < (1 << DIM); ++c) rd_lds[c * kWave + lane] = rdv[c];
  load_halo(zof(0), L1, L2, B1, B2);
  if (ZREG && (!CARRY || zload)) {
    const int z = zof(0);
#pragma unroll
    for (int v = 0; v < (ZREG ? NC : 0); ++v) {
      const int x = xs + min(v % TT, cnt[0] - 1) * s[0], y = ys + min(v / TT, cnt[1] - 1) * s[1];
      ZA[v] = upstream_sel(dv, hcc, hp, 2, x, y, z - s[2], kofs, kmir[2], colb);
      ZB[v] = upstream_sel(dv, hcc, hp, 2, x, y, z - 2 * s[2], kofs, kmir[2], colb);
    }
  }
  __syncthreads();
  // One 4 x 4 quadrant (qx, qy) of the tile's plane: its voxels' records go from LDS
  // to registers, lane l taking voxel l % 16, and reach the lanes of all 64
  // velocities as row_newbcast operands. Read from LDS by every lane of every
  // voxel, the 14 values of a 3D voxel were 4 KB of LDS return traffic, 32 clocks
  // of the CU per voxel and wavefront. A sweep took, before and after:
  // 667 and 528 us (101 x 50 x 47, 512 velocities, FP64), 3.58 and 3.48 ms (96^3, 4096
  // velocities, FP32, bound by HBM traffic), 2.42 and 2.31 ms (64 problems of
  // 128 - 384 a side, 576 velocities, FP32). La, Lb: the columns one
  // and two to the left; Ba, Bb: the rows one and two below; N: its values.
  constexpr int NV = 16;
  auto quadrant = [&](auto QX, auto QY, int pz, int z, const T(&La)[4], const T(&Lb)[4], const T(&Ba)[4], const T(&Bb)[4],
                      const __amdgpu_buffer_rsrc_t(&rowrs)[TT], const uint32_t(&vx)[TT], T(&N)[NV])
                  __attribute__((always_inline)) {
    constexpr int qx = QX, qy = QY;
    const int mine = pz * NC + (4 * qy + ((lane >> 2) & 3)) * TT + 4 * qx + (lane & 3);
    T rp[RW];
#pragma unroll
    for (int k = 0; k < RW; ++k) rp[k] = rec[mine * RW + k];
    const uint32_t code = rcode[mine];
    uint32_t rdo = (code & 7u) * (uint32_t)(kWave * sizeof(T)), rdrop = (code & R_SKIP) ? kDrop : 0u;
    // a DPP operand may be read two instructions after its write at the earliest
    // ("+v": the values are those of this point, not formed again after it)
    asm volatile("s_nop 1" : "+v"(rdo), "+v"(rdrop));
    T Za[ZREG || DIM == 2 ? 1 : NV], Zb[ZREG || DIM == 2 ? 1 : NV];  // 8 x 8 tiles in 3D: the x3-upstream values from h
    if constexpr (DIM == 3 && !ZREG) {
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int x = xs + min(4 * qx + v % 4, cnt[0] - 1) * s[0], y = ys + min(4 * qy + v / 4, cnt[1] - 1) * s[1];
        Za[v] = upstream_sel(dv, hcc, hp, 2, x, y, z - s[2], kofs, kmir[2], colb);
        Zb[v] = upstream_sel(dv, hcc, hp, 2, x, y, z - 2 * s[2], kofs, kmir[2], colb);
      }
    }
    T num[NV], rdv[NV];
    static_for<NV>([&](auto V) __attribute__((always_inline)) {
      constexpr int v = V;
      rdv[v] = *(lds_ptr)(uintptr_t)add_bcast<v>(rdo, rd_addr);
    });
    static_for<NV>([&](auto V) __attribute__((always_inline)) {
      constexpr int v = V;
      T x = bcast<v>(rp[0]);
      if (PSI) x = x * ph;
      fmac_bcast<v>(x, rp[1], vv[0]);
      fmac_bcast<v>(x, rp[2], vv[1]);
      if constexpr (DIM == 3) fmac_bcast<v>(x, rp[3], vv[2]);
      if constexpr (DIM == 3 || PSI) fmac_bcast<v>(x, rp[4], vsqm);  // 0 without the feedback
      if constexpr (SH) {
#pragma unroll
        for (int j = 0; j < DIM; ++j) fmac_bcast<v>(x, rp[5 + 3 * DIM + j], cq[j]);
      }
      if constexpr (MW) {
        // the voxel's own previous iterate at the mirrored velocity (a uniform branch)
        const uint32_t cv = __builtin_amdgcn_readlane(code, v);
        const gptr<const T> hv_prev =
            hp + (int64_t)((n1 * z + ys + (4 * qy + v / 4) * s[1]) * n0 + xs + (4 * qx + v % 4) * s[0]) * Kp;
#pragma unroll
        for (int j = 0; j < DIM; ++j)
          if (cv & (16u << j)) x = fma(am[j], hv_prev[kmir[j]], x);
      }
      num[v] = x;
    });
    static_for<7>([&](auto Dg) __attribute__((always_inline)) {
      constexpr int d = Dg;
      // the anti-diagonal's voxels are independent: operation by operation
      auto each = [&](auto f) __attribute__((always_inline)) {
        static_for<4>([&](auto R) __attribute__((always_inline)) {
          constexpr int r = R, i = d - r;
          if constexpr (i >= 0 && i < 4) f(std::integral_constant<int, r>{}, std::integral_constant<int, i>{});
        });
      };
      T y1[4], y2[4];
      each([&](auto R, auto I) __attribute__((always_inline)) {
        constexpr int r = R, v = I + 4 * r;
        y1[r] = bcast<v>(rp[7]);
        y2[r] = bcast<v>(rp[10]);
        if (PSI) {
          y1[r] = y1[r] * ph;
          y2[r] = y2[r] * ph;
        }
      });
      each([&](auto R, auto I) __attribute__((always_inline)) {
        constexpr int r = R, i = I, v = i + 4 * r;
        fmac_bcast<v>(y1[r], rp[6], i >= 2 ? N[i >= 2 ? v - 2 : 0] : (i == 1 ? La[r] : Lb[r]));
        fmac_bcast<v>(y2[r], rp[9], r >= 2 ? N[r >= 2 ? v - 8 : 0] : (r == 1 ? Ba[i] : Bb[i]));
      });
      each([&](auto R, auto I) __attribute__((always_inline)) {
        constexpr int r = R, i = I, v = i + 4 * r;
        fmac_bcast<v>(y1[r], rp[5], i >= 1 ? N[i >= 1 ? v - 1 : 0] : La[r]);
        fmac_bcast<v>(y2[r], rp[8], r >= 1 ? N[r >= 1 ? v - 4 : 0] : Ba[i]);
      });
      each([&](auto R, auto I) __attribute__((always_inline)) {
        constexpr int r = R, v = I + 4 * r;
        num[v] = fma(aa[0], y1[r], num[v]);
        if constexpr (DIM == 3) y1[r] = bcast<v>(rp[13]);
      });
      each([&](auto R, auto I) __attribute__((always_inline)) {
        constexpr int r = R, v = I + 4 * r;
        num[v] = fma(aa[1], y2[r], num[v]);
        if constexpr (DIM == 3) fmac_bcast<v>(y1[r], rp[12], ZREG ? ZB[ZREG ? v : 0] : Zb[ZREG ? 0 : v]);
      });
      if constexpr (DIM == 3) {
        each([&](auto R, auto I) __attribute__((always_inline)) {
          constexpr int r = R, v = I + 4 * r;
          fmac_bcast<v>(y1[r], rp[11], ZREG ? ZA[ZREG ? v : 0] : Za[ZREG ? 0 : v]);
        });
        each([&](auto R, auto I) __attribute__((always_inline)) {
          constexpr int r = R, v = I + 4 * r;
          num[v] = fma(aa[2], y1[r], num[v]);
        });
      }
      each([&](auto R, auto I) __attribute__((always_inline)) {
        constexpr int r = R, v = I + 4 * r;
        N[v] = num[v] * rdv[v];
      });
      // a voxel that is not stored (solid, past a ragged tile) or a lane past the
      // octant gets an offset past the row's range, which the hardware drops: no
      // branch around the stores, so the wait counts stay exact and a wait for the
      // next plane's halos never waits for this plane's stores
      each([&](auto R, auto I) __attribute__((always_inline)) {
        constexpr int r = R, i = I, v = i + 4 * r;
        buffer_store(N[v], rowrs[4 * qy + r], add_bcast<v>(rdrop, vx[4 * qx + i]), 0u);
        if constexpr (ZREG) {  // this plane's value is the next plane's one-back, its one-back the two-back
          ZB[ZREG ? v : 0] = ZA[ZREG ? v : 0];
          ZA[ZREG ? v : 0] = N[v];
        }
      });
    });
  };

  // one plane; the first is peeled off the loop, so that the loop is entered,
  // as it is re-entered, right after a plane's stores: its waits for the
  // halos loaded ahead then never cover those stores. The last is peeled too:
  // it loads no halos ahead (one-plane tiles, rare, reload their own)
  auto plane = [&](int c3, auto next) __attribute__((always_inline)) {
    constexpr bool NEXT = decltype(next)::value;  // a plane follows in this tile
    const int z = zof(c3);
    const int pz = c3 % PZ;
    if (c3 > 0 && pz == 0) {  // the next chunk of records (only LDS is written here)
      __syncthreads();
      stage(c3, min(PZ, cnt[2] - c3), [] {});
      __syncthreads();
    }
    // the next plane's halos, issued before this plane's stores: waiting for
    // them then does not wait for the stores
    T L1n[TT], L2n[TT], B1n[TT], B2n[TT];
    if (DIM == 3 && NEXT) load_halo(zof(min(c3 + 1, cnt[2] - 1)), L1n, L2n, B1n, B2n);
    // stores: one buffer resource per row of the tile (a row of h spans below
    // 1 GiB, checked by the host)
    __amdgpu_buffer_rsrc_t rowrs[TT];
    uint32_t vx[TT];  // this lane's byte offset of column k in a row
#pragma unroll
    for (int k = 0; k < TT; ++k) {
      rowrs[k] = __builtin_amdgcn_make_buffer_rsrc(
          (void *)((gptr<char>)hc + (uint64_t)(uint32_t)((n1 * z + ys + min(k, cnt[1] - 1) * s[1]) * n0) * colb),
          (short)0, (int)(colb * (uint32_t)n0), kBufferFlags);
      vx[k] = kst + (uint32_t)xs * colb + (uint32_t)k * dcol;
    }
    // the quadrants in sweep order (one for 4 x 4 tiles)
    constexpr int QN = TT / 4;
    T top1[QN > 1 ? TT : 1], top2[QN > 1 ? TT : 1];  // the lower quadrants' top two rows
    static_for<QN>([&](auto QY) __attribute__((always_inline)) {
      T La[4], Lb[4], N[NV];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        La[r] = L1[4 * QY + r] + jx1;
        Lb[r] = L2[4 * QY + r] + jx2;
      }
      static_for<QN>([&](auto QX) __attribute__((always_inline)) {
        T Ba[4], Bb[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          Ba[i] = QY == 0 ? B1[4 * QX + i] : top1[QN > 1 ? 4 * QX + i : 0];
          Bb[i] = QY == 0 ? B2[4 * QX + i] : top2[QN > 1 ? 4 * QX + i : 0];
        }
        quadrant(QX, QY, pz, z, La, Lb, Ba, Bb, rowrs, vx, N);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          La[k] = N[4 * k + 3];
          Lb[k] = N[4 * k + 2];
          if (QN > 1 && QY == 0) {
            top1[QN > 1 ? 4 * QX + k : 0] = N[12 + k];
            top2[QN > 1 ? 4 * QX + k : 0] = N[8 + k];
          }
        }
      });
    });
    if (DIM == 3 && NEXT) {
#pragma unroll
      for (int k = 0; k < TT; ++k) {
        L1[k] = L1n[k];
        L2[k] = L2n[k];
        B1[k] = B1n[k];
        B2[k] = B2n[k];
      }
    }
  };
  plane(0, std::true_type{});
  for (int c3 = 1; c3 < cnt[2] - 1; ++c3) plane(c3, std::true_type{});
  if (cnt[2] > 1) plane(cnt[2] - 1, std::false_type{});
}

}  // namespace
}  // namespace pdvm
