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
// The jump at x1 = x (images across the wrap), added where a value is used, so
// that nothing waits for its load early.
template <typename T>
__device__ __forceinline__ T wrap_jump(const Dom<T> &g, int x) {
  return (x < 0 ? T(1) : (x >= g.n[0] ? T(-1) : T(0))) * g.jump;
}

// Bits of a record's code (from R_USE1 + 2 j, R_USE2 + 2 j): the voxel's stencil along
// axis j uses the first, the second upstream value. Below them: bit j, the first-order
// stencil (the index of the reciprocal denominator); bit 4 + j, a Maxwell wall.
constexpr int R_USE1 = 8, R_USE2 = 9;

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
  using lds_ptr = __attribute__((address_space(3))) const T *;
  const uint32_t rd_addr = (uint32_t)(uintptr_t)(lds_ptr)(rd_lds + lane);
  auto zof = [&](int c3) { return s[2] > 0 ? lo[2] + c3 : lo[2] + cnt[2] - 1 - c3; };
  // Values outside the tile are loaded a voxel row at a time through a buffer
  // resource of the row (below 1 GiB, checked by the host): one scalar base per
  // row, and per value the lane's offset. What no voxel of the plane uses (its
  // own stencil ends at a wall or it is solid: 45 % of the halo values of the 96^3
  // pack) gets an offset past the row's range, for which the hardware reads
  // nothing and gives 0. The 96^3 pack's sweep took 3.48 ms with all halos
  // loaded from 64-bit addresses formed one by one.
  auto row_rsrc = [&](gptr<const char> base, int y, int z) __attribute__((always_inline)) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)(base + (uint64_t)(uint32_t)((n1 * z + y) * n0) * colb), (short)0,
                                             (int)(colb * (uint32_t)n0), kBufferFlags);
  };
  // node c along axis j: the coordinate, the buffer and the lane's offset in a
  // voxel (the current sweep, or the image of the previous iterate outside the
  // domain)
  struct Node {
    gptr<const char> base;
    int c;
    uint32_t k;
  };
  auto node_of = [&](int j, int c) __attribute__((always_inline)) {
    const bool in = c >= 0 && c < dm.n[j];
    const Img im = image_of(j, c, dm.n[j], dm.latp);
    return Node{(gptr<const char>)(in ? hcc : hp), in ? c : im.r,
                (uint32_t)((!in && im.mir) ? kmir[j] : kofs) * (uint32_t)sizeof(T)};
  };
  const Node nx1 = node_of(0, xs - s[0]), nx2 = node_of(0, xs - 2 * s[0]);
  const Node ny1 = node_of(1, ys - s[1]), ny2 = node_of(1, ys - 2 * s[1]);
  const uint32_t ox1 = nx1.k + (uint32_t)nx1.c * colb, ox2 = nx2.k + (uint32_t)nx2.c * colb;
  // rows and columns past a ragged tile repeat its last one (never stored)
  auto row_y = [&](int r) __attribute__((always_inline)) { return ys + min(r, cnt[1] - 1) * s[1]; };
  uint32_t xo[TT];  // byte offset of column i in a row
#pragma unroll
  for (int i = 0; i < TT; ++i) xo[i] = (uint32_t)(xs + min(i, cnt[0] - 1) * s[0]) * colb;
  constexpr int QN = TT / 4;
  // the record codes of a quadrant of plane pz, lane l taking voxel l % 16
  auto code_of = [&](int pz, int qx, int qy) __attribute__((always_inline)) {
    return rcode[pz * NC + (4 * qy + ((lane >> 2) & 3)) * TT + 4 * qx + (lane & 3)];
  };
  // the halos of plane z; pz its plane in the staged records, or -1 if its
  // records are not staged yet (everything is loaded)
  auto load_halo = [&](int z, int pz, T(&L1)[TT], T(&L2)[TT], T(&B1)[TT], T(&B2)[TT]) __attribute__((always_inline)) {
    static_for<QN>([&](auto Q) __attribute__((always_inline)) {
      constexpr int q4 = 4 * Q;
      // lane 4 r: row r's left values; lane i: column i's lower values. The nearer
      // one is also the second upstream value of the next voxel in.
      const uint32_t cl = code_of(max(pz, 0), 0, Q), cb = QN > 1 ? code_of(max(pz, 0), Q, 0) : cl;
      const uint32_t cl1 = __builtin_amdgcn_mov_dpp((int)cl, 0xF5, 0xF, 0xF, true);   // quad_perm: lane + 1
      const uint32_t cb1 = __builtin_amdgcn_mov_dpp((int)cb, 0x104, 0xF, 0xF, true);  // row_shl:4: lane + 4
      const uint32_t all = pz < 0 ? 1u : 0u;
      uint32_t d1 = ((((cl >> R_USE1) | (cl1 >> R_USE2)) | all) & 1u) ? 0u : kDrop;
      uint32_t d2 = (((cl >> R_USE2) | all) & 1u) ? 0u : kDrop;
      uint32_t e1 = ((((cb >> (R_USE1 + 2)) | (cb1 >> (R_USE2 + 2))) | all) & 1u) ? 0u : kDrop;
      uint32_t e2 = (((cb >> (R_USE2 + 2)) | all) & 1u) ? 0u : kDrop;
      asm volatile("s_nop 1" : "+v"(d1), "+v"(d2), "+v"(e1), "+v"(e2));
      static_for<4>([&](auto K) __attribute__((always_inline)) {
        constexpr int k = K;
        const int y = row_y(q4 + k);
        L1[q4 + k] = buffer_load<T>(row_rsrc(nx1.base, y, z), add_bcast<4 * k>(d1, ox1));
        L2[q4 + k] = buffer_load<T>(row_rsrc(nx2.base, y, z), add_bcast<4 * k>(d2, ox2));
        B1[q4 + k] = buffer_load<T>(row_rsrc(ny1.base, ny1.c, z), add_bcast<k>(e1, ny1.k) + xo[q4 + k]);
        B2[q4 + k] = buffer_load<T>(row_rsrc(ny2.base, ny2.c, z), add_bcast<k>(e2, ny2.k) + xo[q4 + k]);
      });
    });
  };
  // the x3-upstream values, one and two planes back, of the 16 voxels of a
  // quadrant of plane z: d1, d2 hold kDrop in the lanes of voxels that use none
  auto load_z = [&](int qx, int qy, int z, uint32_t d1, uint32_t d2, T *za, T *zb) __attribute__((always_inline)) {
    const Node nz1 = node_of(2, z - s[2]), nz2 = node_of(2, z - 2 * s[2]);
    asm volatile("s_nop 1" : "+v"(d1), "+v"(d2));
    static_for<16>([&](auto V) __attribute__((always_inline)) {
      constexpr int v = V;
      const int y = row_y(4 * qy + v / 4);
      za[v] = buffer_load<T>(row_rsrc(nz1.base, y, nz1.c), add_bcast<v>(d1, nz1.k) + xo[4 * qx + v % 4]);
      zb[v] = buffer_load<T>(row_rsrc(nz2.base, y, nz2.c), add_bcast<v>(d2, nz2.k) + xo[4 * qx + v % 4]);
    });
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
        code |= (c1 != T(0) ? 1u : 0u) << (R_USE1 + 2 * j) | (c2 != T(0) ? 1u : 0u) << (R_USE2 + 2 * j);
        if (MW && first && y1s) code |= 16u << j;
      }
      rcode[v] = fl ? code : R_SKIP;
    }
  };

  const T jx1 = wrap_jump(dv, xs - s[0]), jx2 = wrap_jump(dv, xs - 2 * s[0]);  // the same for every plane
  // the tile's first plane: records, halos and (4 x 4 tiles in 3D) the two
  // planes below
  T L1[TT], L2[TT], B1[TT], B2[TT];
  stage(0, min(PZ, cnt[2]), before);
#pragma unroll
  for (int c = 0; c < (1 << DIM); ++c) rd_lds[c * kWave + lane] = rdv[c];
  __syncthreads();
  load_halo(zof(0), 0, L1, L2, B1, B2);
  if constexpr (ZREG) {
    if (!CARRY || zload) {
      // a value one plane back is also two planes back of the next plane's voxel
      // (in a column, possibly the next tile's: then all are loaded)
      const uint32_t c0 = code_of(0, 0, 0), c1 = cnt[2] > 1 ? code_of(1, 0, 0) : (CARRY ? 1u << (R_USE2 + 4) : 0u);
      const uint32_t d1 = (((c0 >> (R_USE1 + 4)) | (c1 >> (R_USE2 + 4))) & 1u) ? 0u : kDrop;
      load_z(0, 0, zof(0), d1, ((c0 >> (R_USE2 + 4)) & 1u) ? 0u : kDrop, ZA, ZB);
    }
  }
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
    const uint32_t code = code_of(pz, qx, qy);
    uint32_t rdo = (code & 7u) * (uint32_t)(kWave * sizeof(T)), rdrop = (code & R_SKIP) ? kDrop : 0u;
    // a DPP operand may be read two instructions after its write at the earliest
    // ("+v": the values are those of this point, not formed again after it)
    asm volatile("s_nop 1" : "+v"(rdo), "+v"(rdrop));
    T Za[ZREG || DIM == 2 ? 1 : NV], Zb[ZREG || DIM == 2 ? 1 : NV];  // 8 x 8 tiles in 3D: the x3-upstream values from h
    if constexpr (DIM == 3 && !ZREG)
      load_z(qx, qy, z, ((code >> (R_USE1 + 4)) & 1u) ? 0u : kDrop, ((code >> (R_USE2 + 4)) & 1u) ? 0u : kDrop, Za, Zb);
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
    if (DIM == 3 && NEXT) load_halo(zof(min(c3 + 1, cnt[2] - 1)), pz + 1 < PZ ? pz + 1 : -1, L1n, L2n, B1n, B2n);
    __amdgpu_buffer_rsrc_t rowrs[TT];  // stores
    uint32_t vx[TT];  // this lane's byte offset of column k in a row
#pragma unroll
    for (int k = 0; k < TT; ++k) {
      rowrs[k] = row_rsrc((gptr<const char>)hcc, row_y(k), z);
      vx[k] = kst + xo[k];
    }
    // the quadrants in sweep order (one for 4 x 4 tiles)
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
