// Kernels of the warm-start network: a U-Net trained on converged fields of the
// iteration that maps a solid mask and Kn to an initial density and velocity
// field (the iteration itself then runs unchanged from that start).
//
// The dense contractions (every 3x3 and 1x1 convolution, forward, backward
// with respect to the input, and the weight gradient) run on the gfx950 matrix
// cores: v_mfma_f32_16x16x32_bf16, bf16 operands, FP32 accumulation. Lane
// layout of that instruction (checked on the device): lane l holds
// A[m = l % 16][k = 8 (l / 16) + i] and B[k = 8 (l / 16) + i][n = l % 16],
// i = 0..7, and receives D[m = 4 (l / 16) + r][n = l % 16], r = 0..3.
#include <algorithm>

#include "unet_internal.h"

namespace pdvm_nn {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);  // NaN stays NaN
  u += 0x7fffu + ((u >> 16) & 1u);                                           // round to nearest even
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// Implicit-GEMM convolution. A block computes a tile of 64 WX pixels (2^pw
// columns) x 32 WN output channels; each of its WX x WN wavefronts 64 pixels x 32
// channels. The input patch with its one-pixel rim is staged in LDS once, with all its
// channels (up to 384 of them in the 160 KB), so an input value is loaded once and not
// once per tap, and the K loop (taps, then channels: the order of the sums) has no
// barrier. Weights come straight from memory (the L1 serves the block's
// wavefronts), four K steps ahead. The channels are the rows of the products and
// the pixels their columns, so a lane ends with four consecutive channels of a
// pixel: 8- or 16-byte stores. C8: 8 input channels, four taps per K step.
// Bound per K step and CU: 16 KB of LDS reads, 8 KB of L1 reads and the matrix
// products take 128 clocks each; and the staging, which nothing overlaps within a
// block. Measured (MI355X): the 14 forward and 14 backward 3x3 convolutions of a
// training step on 8 x 256^2 1.57 -> 1.0 ms, on 2 x 64^2 0.92 -> 0.45 ms, against
// 128-pixel tiles that staged 32 im2col columns at a time behind two barriers.
template <int WX, int WN, int TAPS, bool C8>
__global__ void __launch_bounds__(64 * WX * WN) conv_kernel(ConvArgs a) {
  constexpr int NT = 64 * WX * WN, RIM = TAPS == 9 ? 1 : 0;
  extern __shared__ __attribute__((aligned(16))) unsigned char patch[];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int wx = wv % WX, wn = wv / WX;
  const int PW = 1 << a.pw, PH = (64 * WX) >> a.pw, RW = PW + 2 * RIM, RR = (PH + 2 * RIM) * RW;
  const int Cin = a.Ca + a.Cb, K = TAPS * Cin;
  const int nch = Cin / 8;                          // 16-byte chunks of a pixel
  const uint32_t pitch = (uint32_t)(Cin * 2 + 16);  // padded: the fragment reads of 16 pixels spread over the banks
  const int tx = blockIdx.x % a.npx, tq = blockIdx.x / a.npx;
  const int x0 = tx * PW, y0 = tq % a.npy * PH, b = tq / a.npy;
  const int n0 = (blockIdx.y * WN + wn) * 32;

  // --- weights: rows n0 + 16 f + lane % 16, k = 32 ks + 8 (lane / 16) ..
  constexpr int D = 4;
  const uint16_t *wrow[2];
#pragma unroll
  for (int f = 0; f < 2; ++f) wrow[f] = a.wt + (int64_t)min(n0 + 16 * f + (lane & 15), a.nrows - 1) * K + 8 * (lane >> 4);
  const int nk = C8 ? (K + 31) / 32 : K / 32;
  uint4 wr[D][2];
  auto wload = [&](int ks, uint4(&r)[2]) __attribute__((always_inline)) {
    const int k = min(ks, nk - 1);  // past the end: loaded again, not used
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      r[f] = make_uint4(0, 0, 0, 0);
      if (!C8 || 32 * k + 8 * (lane >> 4) < K) r[f] = *reinterpret_cast<const uint4 *>(wrow[f] + 32 * k);
    }
  };
#pragma unroll
  for (int d = 0; d < D; ++d) wload(d, wr[d]);

  // --- the input patch: zero outside the image along y, circular along x
  {
    const int total = RR * nch;
    constexpr int U = 8;  // loads in flight per lane
    for (int e0 = tid; e0 < total; e0 += NT * U) {
      uint4 v[U];
      uint32_t to[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = e0 + u * NT;
        const int r = C8 ? e : (int)__umulhi((uint32_t)e, a.div_ch), ch = e - r * nch;  // e / nch (e < 2^16)
        const int ry = (int)__umulhi((uint32_t)r, a.div_rw), rx = r - ry * RW;   // r / RW
        const int y = y0 + ry - RIM;
        int x = x0 + rx - RIM;
        const bool in = e < total && y >= 0 && y < a.H && x <= a.W;  // right of a ragged last tile: nothing to read
        x = x < 0 ? x + a.W : (x >= a.W ? x - a.W : x);
        to[u] = e < total ? (uint32_t)r * pitch + 16u * ch : ~0u;
        v[u] = make_uint4(0, 0, 0, 0);
        if (in) {
          const int c = 8 * ch;
          const uint16_t *src;
          if (c < a.Ca)
            src = a.ups ? a.xa + ((int64_t)(b * (a.H >> 1) + (y >> 1)) * (a.W >> 1) + (x >> 1)) * a.Ca + c
                        : a.xa + ((int64_t)(b * a.H + y) * a.W + x) * a.Ca + c;
          else
            src = a.xb + ((int64_t)(b * a.H + y) * a.W + x) * a.Cb + (c - a.Ca);
          v[u] = *reinterpret_cast<const uint4 *>(src);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (to[u] != ~0u) *reinterpret_cast<uint4 *>(patch + to[u]) = v[u];
    }
  }
  __syncthreads();

  // --- pixel fragments: pixel t = 64 wx + 16 f + lane % 16 of the tile
  uint32_t pb[4];
#pragma unroll
  for (int f = 0; f < 4; ++f) {
    const int t = 64 * wx + 16 * f + (lane & 15);
    pb[f] = (uint32_t)((t >> a.pw) * RW + (t & (PW - 1))) * pitch + (C8 ? 0u : 16u * (lane >> 4));
  }
  f32x4 acc[2][4];
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int f = 0; f < 4; ++f) acc[m][f] = f32x4{0.f, 0.f, 0.f, 0.f};
  uint4 pr[2][4];
  // K step ks: tap ks / (Cin / 32) at channels 32 (ks % (Cin / 32)); its offset into the patch advances with ks
  uint32_t ko = 0;
  int kc = 0, kt = 0;
  const int ncs = Cin / 32;
  auto pload = [&](int ks, uint4(&r)[4]) __attribute__((always_inline)) {
    if (C8) {
      const int t = 4 * ks + (lane >> 4);
      const uint32_t o = (uint32_t)(t / 3 * RW + t % 3) * pitch;
#pragma unroll
      for (int f = 0; f < 4; ++f)
        r[f] = t < TAPS ? *reinterpret_cast<const uint4 *>(patch + pb[f] + o) : make_uint4(0, 0, 0, 0);
      return;
    }
#pragma unroll
    for (int f = 0; f < 4; ++f) r[f] = *reinterpret_cast<const uint4 *>(patch + pb[f] + ko);
    ko += 64;
    if (++kc == ncs) {  // the next tap (past the last one: the patch's first pixel, not used)
      kc = 0;
      kt = kt + 1 == TAPS ? 0 : kt + 1;
      ko = (uint32_t)(kt / 3 * RW + kt % 3) * pitch;
    }
  };
  pload(0, pr[0]);
  for (int k0 = 0; k0 < nk; k0 += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      if (k0 + d < nk) {
        pload(k0 + d + 1, pr[(d + 1) & 1]);
        bf16x8 fw[2], fp[4];
#pragma unroll
        for (int m = 0; m < 2; ++m) fw[m] = __builtin_bit_cast(bf16x8, wr[d][m]);
#pragma unroll
        for (int f = 0; f < 4; ++f) fp[f] = __builtin_bit_cast(bf16x8, pr[d & 1][f]);
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
          for (int f = 0; f < 4; ++f)
            acc[m][f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[m], fp[f], acc[m][f], 0, 0, 0);
        wload(k0 + d + D, wr[d]);
      }
    }
  }

  // --- D[m = 4 (lane / 16) + r][n = lane % 16]: channels n0 + 16 m + 4 (lane / 16) + r of pixel 16 f + lane % 16
#pragma unroll
  for (int f = 0; f < 4; ++f) {
    const int t = 64 * wx + 16 * f + (lane & 15);
    const int y = y0 + (t >> a.pw), x = x0 + (t & (PW - 1));
    if (y >= a.H || x >= a.W) continue;
    const int64_t p = (int64_t)(b * a.H + y) * a.W + x;
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const int n = n0 + 16 * m + 4 * (lane >> 4);
      if (n >= a.nstore) continue;
      f32x4 v = acc[m][f];
      if (a.bias) v += *reinterpret_cast<const f32x4 *>(a.bias + n);
      if (a.relu) {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = fmaxf(v[r], 0.f);
      }
      const int64_t at = p * a.ystride + n;
      if (a.gate) {
        const uint2 gw = *reinterpret_cast<const uint2 *>(a.gate + at);
        v[0] = bf2f((uint16_t)gw.x) > 0.f ? v[0] : 0.f;
        v[1] = bf2f((uint16_t)(gw.x >> 16)) > 0.f ? v[1] : 0.f;
        v[2] = bf2f((uint16_t)gw.y) > 0.f ? v[2] : 0.f;
        v[3] = bf2f((uint16_t)(gw.y >> 16)) > 0.f ? v[3] : 0.f;
      }
      if (n + 4 > a.nstore) {  // the head: 3 of 4 channels
        for (int r = 0; r < 4 && n + r < a.nstore; ++r) {
          if (a.yb) a.yb[at + r] = f2bf(v[r]);
          else a.yf[at + r] = v[r];
        }
      } else if (a.yb) {
        *reinterpret_cast<uint2 *>(a.yb + at) = make_uint2((uint32_t)f2bf(v[0]) | ((uint32_t)f2bf(v[1]) << 16),
                                                           (uint32_t)f2bf(v[2]) | ((uint32_t)f2bf(v[3]) << 16));
      } else {
        *reinterpret_cast<f32x4 *>(a.yf + at) = v;
      }
    }
  }
}

// dW partials of kPixPerSplit pixels each. A wavefront owns 32 output channels x
// 16 input channels x the three taps of one row of the stencil; a block is WM
// wavefronts along the output and WC along the input channels, for one stencil
// row (blockIdx.z % 3). Both operands are pixel-major in memory while the matrix
// instruction wants 8 consecutive pixels of one channel per lane: they are staged
// in LDS as they are (rows of pixels) and read with the transposing LDS load
// (ds_read_b64_tr_b16: lane l of 16 gets column l of 4 rows of 16 values).
// kRun pixels are staged at a time, two buffers, the next run's loads in flight.
// Of the input, a run is the contiguous stretch of the image's rows padded by a
// pixel on either side (the wrapped neighbours), so the three taps read it at
// offsets 0, 1 and 2: pixel k of the run, i rows into it, is padded pixel k + 2 i.
// The sums' order (32 pixels per product, products in pixel order, splits in
// order) does not depend on the tiles.
// Bound: the instructions of one wavefront per run (addresses, staging, 20
// transposing loads per 6 matrix products), as the order leaves only P /
// kPixPerSplit runs of work side by side. Measured (MI355X, training step on 8 x
// 256^2): all weight gradients 1.0 ms, against 3.25 ms with 64 x 32 tiles
// transposed by 16-bit LDS writes; 0.67 ms with the patches of a split spread over
// wavefronts in another order of sums, which a few steps of Adam (whose update is
// nearly the sign of a small gradient) turn into differences of 1e-2.
constexpr int kRun = 128;

typedef short v4s __attribute__((ext_vector_type(4)));
__device__ __forceinline__ bf16x8 tr_pair(uint32_t a0, uint32_t a1) {
  using lp = __attribute__((address_space(3))) v4s *;
  const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(uintptr_t)a0);
  const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(uintptr_t)a1);
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// TX: taps per stencil row (3, or 1 for 1x1); XN: 16-byte pieces of a run's input per thread
template <int TX, int WM, int WC, int XN>
__global__ void __launch_bounds__(64 * WM * WC) wgrad_kernel(WgradArgs a) {
  constexpr int NT = 64 * WM * WC, BM = 32 * WM, BC = 16 * WC;
  constexpr int RIM = TX == 3 ? 1 : 0;
  constexpr int XP = BC * 2 + 16, GP = BM * 2 + 16;  // LDS row pitches in bytes
  constexpr int XCH = BC / 8, GCH = BM / 8;          // 16-byte pieces per pixel
  constexpr int GN = kRun * GCH / NT;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const uint32_t l0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int wm = wv % WM, wc = wv / WM;
  const int m0 = blockIdx.x * BM, c0 = blockIdx.y * BC;
  const int dy = TX == 3 ? (int)(blockIdx.z % 3) - 1 : 0, split = TX == 3 ? blockIdx.z / 3 : blockIdx.z;
  const int Cin = a.Ca + a.Cb, H = a.H, W = a.W, WR = W + 2 * RIM;
  const int P = a.B * H * W;
  const int pbeg = split * kPixPerSplit, pend = min(P, pbeg + kPixPerSplit);
  const uint32_t xbytes = (uint32_t)a.xrows * XP, bufbytes = xbytes + kRun * GP;
  // this block's channels come from one of the concatenated inputs
  const bool inA = c0 < a.Ca;
  const uint16_t *const xs = inA ? a.xa : a.xb;
  const int xc = inA ? c0 : c0 - a.Ca, xC = inA ? a.Ca : a.Cb;
  const int ups = inA ? a.ups : 0;

  // a quotient of small numbers (below 2^16), or of ones below 2 d
  auto quot = [](int v, int d, uint32_t magic) {
    return d == 1 ? v : (magic ? (int)__umulhi((uint32_t)v, magic) : (v >= d ? 1 : 0));
  };
  constexpr int AHEAD = 2;  // runs whose loads are in flight
  struct Run {
    uint4 x[XN], g[GN];
  } runs[AHEAD];
  // the next run to load: its first pixel, and that pixel's column, row and image
  int lp = pbeg, lx = pbeg % W, ly = pbeg / W % H, lb = pbeg / W / H;
  const char *const xbase = reinterpret_cast<const char *>(xs + xc), *const gbase = reinterpret_cast<const char *>(a.g + m0);
  // byte offsets fit in 32 bits (a tensor has under 2^31 values)
  auto load = [&](Run &R) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < XN; ++i) {
      const int e = tid + NT * i, l = e / XCH, ch = e % XCH;
      R.x[i] = make_uint4(0, 0, 0, 0);
      const int u = l + lx, row = quot(u, WR, a.div_wr);
      int x = u - row * WR - RIM, y = ly + row, b = lb;
      if (y >= H) {  // past this image
        const int q = y >= 2 * H ? y / H : 1;
        b += q;
        y -= q * H;
      }
      y += dy;
      x = x < 0 ? x + W : (x >= W ? x - W : x);
      if (l < a.xrows && b < a.B && y >= 0 && y < H && xc + 8 * ch < xC) {
        const uint32_t p = ups ? (uint32_t)((b * (H >> 1) + (y >> 1)) * (W >> 1) + (x >> 1)) : (uint32_t)((b * H + y) * W + x);
        R.x[i] = *reinterpret_cast<const uint4 *>(xbase + (uint32_t)(p * (uint32_t)(2 * xC) + 16u * ch));
      }
    }
#pragma unroll
    for (int i = 0; i < GN; ++i) {
      const int e = tid + NT * i, k = e / GCH, ch = e % GCH;
      R.g[i] = make_uint4(0, 0, 0, 0);
      if (lp + k < pend) R.g[i] = *reinterpret_cast<const uint4 *>(gbase + (uint32_t)((uint32_t)(lp + k) * (uint32_t)(2 * a.M) + 16u * ch));
    }
    if (lp + kRun >= pend) return;  // the last run: loaded again, not used
    const int t = lx + kRun, rows = quot(t, W, a.div_w);
    lp += kRun;
    lx = t - rows * W;
    ly += rows;
    while (ly >= H) {
      ly -= H;
      ++lb;
    }
  };
  auto store = [&](uint32_t buf, const Run &R) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < XN; ++i) {
      const int e = tid + NT * i;
      if (e < a.xrows * XCH) *reinterpret_cast<uint4 *>(lds + buf + e / XCH * XP + e % XCH * 16) = R.x[i];
    }
#pragma unroll
    for (int i = 0; i < GN; ++i) {
      const int e = tid + NT * i;
      *reinterpret_cast<uint4 *>(lds + buf + xbytes + e / GCH * GP + e % GCH * 16) = R.g[i];
    }
  };
  f32x4 acc[2][TX];
#pragma unroll
  for (int ms = 0; ms < 2; ++ms)
#pragma unroll
    for (int t = 0; t < TX; ++t) acc[ms][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  // fragments: pixel k = 32 c + 8 (lane / 16) + 4 h + (lane % 16) / 4, columns 4 (lane % 4) ..
  const int kr = 8 * (lane >> 4) + ((lane & 15) >> 2), cq = 4 * (lane & 3);
  const uint32_t gcol = (uint32_t)(wm * 32 + cq) * 2, xcol = (uint32_t)(wc * 16 + cq) * 2;

  auto products = [&](int x0, uint32_t buf) __attribute__((always_inline)) {
    const uint32_t xb = l0 + buf + xcol, gb = l0 + buf + xbytes + gcol;
#pragma unroll
    for (int c = 0; c < kRun / 32; ++c) {
      uint32_t xa[2], ga[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int k = 32 * c + kr + 4 * h;
        xa[h] = xb + (uint32_t)(k + 2 * RIM * quot(x0 + k, W, a.div_w)) * XP;
        ga[h] = gb + (uint32_t)k * GP;
      }
      bf16x8 fa[2];
#pragma unroll
      for (int ms = 0; ms < 2; ++ms) fa[ms] = tr_pair(ga[0] + ms * 32, ga[1] + ms * 32);
#pragma unroll
      for (int t = 0; t < TX; ++t) {
        const bf16x8 fb = tr_pair(xa[0] + t * XP, xa[1] + t * XP);
#pragma unroll
        for (int ms = 0; ms < 2; ++ms) acc[ms][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[ms], fb, acc[ms][t], 0, 0, 0);
      }
    }
  };
#pragma unroll
  for (int i = 0; i < AHEAD; ++i) load(runs[i]);
  uint32_t buf = 0;
  int x0 = pbeg % W;  // the column of the run's first pixel
  for (int p0 = pbeg; p0 < pend; p0 += AHEAD * kRun) {
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) {
      const int p = p0 + i * kRun;
      if (p < pend) {
        store(buf, runs[i]);
        __syncthreads();  // this run is staged, and the other buffer's reads are done
        load(runs[i]);
        products(x0, buf);
        x0 += kRun;
        x0 -= quot(x0, W, a.div_w) * W;
        buf = buf ? 0 : bufbytes;
      }
    }
  }
  // D[m = 4 (lane / 16) + r][n = lane % 16]
  const int K = (TX == 3 ? 9 : 1) * Cin, c = c0 + wc * 16 + (lane & 15);
  if (c >= Cin) return;
  float *const out = a.part + (int64_t)split * a.M * K + c;
#pragma unroll
  for (int ms = 0; ms < 2; ++ms)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = m0 + wm * 32 + ms * 16 + 4 * (lane >> 4) + r;
#pragma unroll
      for (int t = 0; t < TX; ++t) out[(int64_t)m * K + (TX == 3 ? 3 * (dy + 1) + t : 0) * Cin] = acc[ms][t][r];
    }
}

// Column sums of a bf16 matrix [P][C] (C divides 256) per kColsumPix rows: row
// lane j of 256 / C sums rows j, j + 256 / C, ... in order, then the row lanes are
// added in order. A lane takes two columns; two partials per block. The sums are
// chains of up to 1024 additions, so the loads run 32 ahead of them and rows that every
// row lane has take no test (9 us per layer on 8 x 256^2; 25 with a test per row, 94
// with one load per addition).
__global__ void __launch_bounds__(256) colsum_kernel(const uint16_t *g, int64_t P, int C, float *part) {
  __shared__ float red[2][256];
  const int t = threadIdx.x & 127, w = threadIdx.x >> 7, G = C / 2, lanes = 256 / C;
  const int c = t % G * 2, j0 = t / G;
  const int64_t blk = (int64_t)blockIdx.x * 2 + w, beg = blk * kColsumPix;
  const int rows = (int)max((int64_t)0, min((int64_t)kColsumPix, P - beg));
  const uint32_t *const src = reinterpret_cast<const uint32_t *>(g + beg * C + c);
  const int step = lanes * C / 2;  // words from one of this lane's rows to the next
  const int n = rows > j0 ? (rows - j0 + lanes - 1) / lanes : 0;
  constexpr int U = 32;
  uint32_t v[U], vn[U];
  auto load = [&](int i0, uint32_t(&r)[U]) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) r[u] = i0 + u < n ? src[(int64_t)j0 * G + (int64_t)(i0 + u) * step] : 0u;
  };
  float lo = 0.f, hi = 0.f;
  auto load_all = [&](int i0, uint32_t(&r)[U]) __attribute__((always_inline)) {
    const uint32_t *const p = src + (int64_t)j0 * G + (int64_t)i0 * step;
#pragma unroll
    for (int u = 0; u < U; ++u) r[u] = p[u * step];
  };
  auto add_all = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      lo += bf2f((uint16_t)v[u]);
      hi += bf2f((uint16_t)(v[u] >> 16));
    }
  };
  // U rows at a time that every row lane has: no test per row
  int i0 = 0;
  const int full = rows / lanes / U * U;
  if (full > 0) {
    load_all(0, v);
    for (; i0 + U < full; i0 += U) {
      load_all(i0 + U, vn);
      add_all();
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = vn[u];
    }
    add_all();
    i0 += U;
  }
  if (i0 < n) load(i0, v);
  for (; i0 < n; i0 += U) {
    load(i0 + U, vn);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (i0 + u < n) {
        lo += bf2f((uint16_t)v[u]);
        hi += bf2f((uint16_t)(v[u] >> 16));
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = vn[u];
  }
  red[w][j0 * C + c] = lo;
  red[w][j0 * C + c + 1] = hi;
  __syncthreads();
  if (rows > 0 && j0 == 0) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      float a = 0.f;
      for (int j = 0; j < lanes; ++j) a += red[w][j * C + c + k];
      part[blk * C + c + k] = a;
    }
  }
}

// The weight gradients out[i] = sum over the splits, in order, of part[split][i]
// (four values per lane), and in the last blocks the bias gradients outb[c] =
// the sum in order of bsplits partials, staged in LDS 256 partials of 32 columns at a
// time (one lane adding from memory would wait for each load).
__global__ void __launch_bounds__(256) sum_splits_kernel(const float *part, int splits, int64_t n, float *out,
                                                         const float *bpart, int bsplits, int nb, float *outb) {
  __shared__ float tile[256 * 32];
  const int64_t wblocks = (n / 4 + 255) / 256;
  const int t = threadIdx.x;
  if (blockIdx.x < wblocks) {
    const int64_t i = ((int64_t)blockIdx.x * 256 + t) * 4;
    if (i >= n) return;
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 16
    for (int j = 0; j < splits; ++j) s += *reinterpret_cast<const f32x4 *>(part + (int64_t)j * n + i);
    *reinterpret_cast<f32x4 *>(out + i) = s;
    return;
  }
  const int c0 = (int)(blockIdx.x - wblocks) * 32;
  float s = 0.f;
  for (int j0 = 0; j0 < bsplits; j0 += 256) {
    const int m = min(256, bsplits - j0);
    __syncthreads();
    for (int e = t; e < m * 32; e += 256) tile[e] = bpart[(int64_t)(j0 + e / 32) * nb + c0 + e % 32];
    __syncthreads();
    if (t < 32) {
#pragma unroll 16
      for (int j = 0; j < m; ++j) s += tile[j * 32 + t];
    }
  }
  if (t < 32) outb[c0 + t] = s;
}

// Input tensor [B][H][W][8]: solid (0/1), the scaled log Kn feature, zeros.
__global__ void build_input_kernel(const uint8_t *solid_set, const float *feat_set, Slots sl, int B, int H, int W,
                                   uint16_t *x) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t HW = (int64_t)H * W;
  if (i >= B * HW) return;
  const int b = (int)(i / HW);
  const int64_t c = i - b * HW;
  const int s = sl.s[b];
  uint4 v = make_uint4(0, 0, 0, 0);
  v.x = (uint32_t)f2bf(solid_set[s * HW + c] ? 1.f : 0.f) | ((uint32_t)f2bf(feat_set[s]) << 16);
  reinterpret_cast<uint4 *>(x)[i] = v;  // kInC = 8 bf16 = 16 bytes per voxel
}

// 2x2 max pooling (first maximum in the order (0,0), (0,1), (1,0), (1,1)).
__global__ void maxpool_kernel(const uint16_t *x, int B, int H, int W, int C, uint16_t *y, uint8_t *idx) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int Ho = H / 2, Wo = W / 2;
  if (i >= (int64_t)B * Ho * Wo * C) return;
  const int c = (int)(i % C);
  int64_t t = i / C;
  const int xo = (int)(t % Wo);
  t /= Wo;
  const int yo = (int)(t % Ho);
  const int b = (int)(t / Ho);
  float best = 0.f;
  int bi = 0;
  for (int j = 0; j < 4; ++j) {
    const int yy = 2 * yo + (j >> 1), xx = 2 * xo + (j & 1);
    const float v = bf2f(x[((int64_t)(b * H + yy) * W + xx) * C + c]);
    if (j == 0 || v > best) {
      best = v;
      bi = j;
    }
  }
  y[i] = f2bf(best);
  idx[i] = (uint8_t)bi;
}

// Eight channels at a time: dy where the activation y is positive, as bfloat16.
__device__ __forceinline__ uint4 gated(const float (&dy)[8], uint4 y) {
  const uint32_t yw[4] = {y.x, y.y, y.z, y.w};
  uint32_t o[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float lo = bf2f((uint16_t)yw[k]) > 0.f ? dy[2 * k] : 0.f;
    const float hi = bf2f((uint16_t)(yw[k] >> 16)) > 0.f ? dy[2 * k + 1] : 0.f;
    o[k] = (uint32_t)f2bf(lo) | ((uint32_t)f2bf(hi) << 16);
  }
  return make_uint4(o[0], o[1], o[2], o[3]);
}
__device__ __forceinline__ void add8(float (&s)[8], const float *p) {
  const f32x4 a = *reinterpret_cast<const f32x4 *>(p), b = *reinterpret_cast<const f32x4 *>(p + 4);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    s[k] += a[k];
    s[4 + k] += b[k];
  }
}

// Gradient at the pre-activation of the deeper input A of a concatenation
// [up(A), skip]: the concatenation's gradient summed over each 2x2 block
// (nearest upsampling), where A is positive. One lane: one pixel of A, 8 channels.
// Memory-bound: dcat read once, one bf16 write (with the kernel below and the
// convolution's gate it replaces separate passes for the upsampling, the skip's
// copy, the pooling and the ReLU: 0.11 instead of 0.45 ms per step on 8 x 256^2).
__global__ void up_grad_kernel(const float *dcat, const uint16_t *y, int B, int H, int W, int Ca, int C, uint16_t *g) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int Ho = H / 2, Wo = W / 2, G = Ca / 8;
  if (i >= (int64_t)B * Ho * Wo * G) return;
  const int c = (int)(i % G) * 8;
  int64_t t = i / G;
  const int xo = (int)(t % Wo);
  t /= Wo;
  const int yo = (int)(t % Ho);
  const int b = (int)(t / Ho);
  float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int j = 0; j < 4; ++j)
    add8(s, dcat + ((int64_t)(b * H + 2 * yo + (j >> 1)) * W + 2 * xo + (j & 1)) * C + c);
  reinterpret_cast<uint4 *>(g)[i] = gated(s, reinterpret_cast<const uint4 *>(y)[i]);
}

// Gradient at the pre-activation of a tensor that is pooled and also skips to
// the decoder: the skip's gradient (channels Ca.. of the concatenation's) plus,
// at each window's maximum, the pooled tensor's. One lane: one 2x2 window, 8 channels.
__global__ void pool_skip_grad_kernel(const float *dcat, int Ca, int C, const float *dp, const uint8_t *idx,
                                      const uint16_t *y, int B, int H, int W, int Cs, uint16_t *g) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int Ho = H / 2, Wo = W / 2, G = Cs / 8;
  if (i >= (int64_t)B * Ho * Wo * G) return;
  const int c = (int)(i % G) * 8;
  int64_t t = i / G;
  const int xo = (int)(t % Wo);
  t /= Wo;
  const int yo = (int)(t % Ho);
  const int b = (int)(t / Ho);
  const uint64_t w = reinterpret_cast<const uint64_t *>(idx)[i];
  float pooled[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  add8(pooled, dp + i * 8);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int64_t p = (int64_t)(b * H + 2 * yo + (j >> 1)) * W + 2 * xo + (j & 1);
    float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    add8(s, dcat + p * C + Ca + c);
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if ((int)((w >> (8 * k)) & 0xFF) == j) s[k] += pooled[k];
    const int64_t e = (p * Cs + c) / 8;
    reinterpret_cast<uint4 *>(g)[e] = gated(s, reinterpret_cast<const uint4 *>(y)[e]);
  }
}

// Masked squared error over the fluid voxels, per sample weight wsamp (1 / (3 nf)),
// averaged over the batch. Writes the bf16 gradient at the head output
// ([p][32], channels >= 3 zero) and per-block partial losses.
__global__ void loss_kernel(const float *pred, const uint8_t *solid_set, const float *target_set, const float *wsamp,
                            Slots sl, int B, int H, int W, uint16_t *g, float *part) {
  __shared__ float red[256];
  const int64_t HW = (int64_t)H * W;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  float l = 0.f;
  if (i < B * HW) {
    const int b = (int)(i / HW);
    const int64_t c = i - b * HW;
    const int s = sl.s[b];
    const bool fluid = solid_set[s * HW + c] == 0;
    const float w = wsamp[s] / (float)B;
    uint16_t o3[3];
    for (int ch = 0; ch < 3; ++ch) {
      const float d = fluid ? pred[i * 4 + ch] - target_set[(s * 3 + ch) * HW + c] : 0.f;
      l += w * d * d;
      o3[ch] = f2bf(2.f * w * d);
    }
    uint4 *dst = reinterpret_cast<uint4 *>(g + i * 32);
    dst[0] = make_uint4((uint32_t)o3[0] | ((uint32_t)o3[1] << 16), (uint32_t)o3[2], 0u, 0u);
    dst[1] = dst[2] = dst[3] = make_uint4(0, 0, 0, 0);
  }
  red[threadIdx.x] = l;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if (threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ void adam_kernel(float *p, const float *g, float *m, float *v, int64_t n, float lr, float b1, float b2,
                            float eps, float c1, float c2) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

__global__ void to_bf16_kernel(const float *src, int64_t n, uint16_t *dst) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = f2bf(src[i]);
}

// Weights of the input-gradient convolution: wb[c][t * Cout + o] = wt[o][(taps-1-t) * Cin + c].
// All layers in one launch (each is a few us of latency, and so was its launch:
// 14 of 4.7 us a step, now one of 11 us).
__global__ void __launch_bounds__(256) wt_back_kernel(WtBackArgs a) {
  int l = 0;
  while (l + 1 < a.layers && (int)blockIdx.x >= a.first[l + 1]) ++l;
  const int Cout = a.Cout[l], Cin = a.Cin[l], taps = a.taps[l];
  const uint16_t *const wt = a.wt + a.off[l];
  uint16_t *const wb = a.wb + a.off[l];
  const int i = ((int)blockIdx.x - a.first[l]) * 256 + (int)threadIdx.x;
  if (i >= Cout * Cin * taps) return;
  const int o = i % Cout, r = i / Cout;
  const int t = r % taps, c = r / taps;
  wb[i] = wt[(int64_t)o * taps * Cin + (int64_t)(taps - 1 - t) * Cin + c];
}

__device__ double block_sum(double v, double *red) {
  red[threadIdx.x] = v;
  __syncthreads();
  for (int off = blockDim.x / 2; off > 0; off >>= 1) {
    if (threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  const double s = red[0];
  __syncthreads();
  return s;
}

__device__ __forceinline__ double usigma(double kn256) {
  const double a = kKnKnee * kn256;
  return a / (1.0 + a);
}

// Normalised targets of one sample (one block of 1024 threads):
// t0 = (rho + J (x1 - 1/2) - mean over fluid) N1 / (256 J),
// t1, t2 = U sigma(Kn256) u_j N1 / (256 J); zero on solid voxels.
__global__ void __launch_bounds__(1024) targets_kernel(const uint8_t *solid, const double *rho, const double *u,
                                                       int H, int W, double jump, double kn256, float *target,
                                                       float *wsamp_one) {
  __shared__ double red[1024];
  const int64_t HW = (int64_t)H * W;
  double s = 0, c = 0;
  for (int64_t i = threadIdx.x; i < HW; i += blockDim.x) {
    if (solid[i]) continue;
    const int x = (int)(i % W);
    s += rho[i] + jump * ((x + 0.5) / W - 0.5);
    c += 1;
  }
  s = block_sum(s, red);
  c = block_sum(c, red);
  const double mean = c > 0 ? s / c : 0.0;
  const double gscale = W / (kRefLen * jump);
  const double us = kUScale * usigma(kn256) * gscale;
  for (int64_t i = threadIdx.x; i < HW; i += blockDim.x) {
    const int x = (int)(i % W);
    const bool f = !solid[i];
    target[i] = f ? (float)((rho[i] + jump * ((x + 0.5) / W - 0.5) - mean) * gscale) : 0.f;
    target[HW + i] = f ? (float)(u[i] * us) : 0.f;
    target[2 * HW + i] = f ? (float)(u[HW + i] * us) : 0.f;
  }
  if (threadIdx.x == 0) *wsamp_one = c > 0 ? (float)(1.0 / (3.0 * c)) : 0.f;
}

// Physical fields from the network output of one sample (the inverse of the
// target normalisation, mean density 0); solid voxels read 0.
__global__ void fields_kernel(const float *pred, const uint8_t *solid, int H, int W, double jump, double kn256,
                              double *rho, double *u) {
  const int64_t HW = (int64_t)H * W;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= HW) return;
  const int x = (int)(i % W);
  const bool f = !solid[i];
  const double gscale = W / (kRefLen * jump);
  const double us = kUScale * usigma(kn256) * gscale;
  rho[i] = f ? pred[i * 4] / gscale - jump * ((x + 0.5) / W - 0.5) : 0.0;
  u[i] = f ? pred[i * 4 + 1] / us : 0.0;
  u[HW + i] = f ? pred[i * 4 + 2] / us : 0.0;
}

inline unsigned nblocks(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

namespace {
template <int WX, int WN, int TAPS, bool C8>
hipError_t conv_as(ConvArgs a, hipStream_t st) {
  // the widest tile up to 16 (8 for 64 pixels) columns that the image has use for
  a.pw = 0;
  while ((1 << a.pw) < std::min(a.W, WX == 1 ? 8 : 16)) ++a.pw;
  const int PW = 1 << a.pw, PH = (64 * WX) >> a.pw, RIM = TAPS == 9 ? 1 : 0;
  a.npx = (a.W + PW - 1) / PW;
  a.npy = (a.H + PH - 1) / PH;
  const int Cin = a.Ca + a.Cb, RW = PW + 2 * RIM, RR = (PH + 2 * RIM) * RW;
  a.div_ch = (uint32_t)(((uint64_t(1) << 32) + Cin / 8 - 1) / (Cin / 8));
  a.div_rw = (uint32_t)(((uint64_t(1) << 32) + RW - 1) / RW);
  const size_t lds = (size_t)RR * (Cin * 2 + 16);
  const dim3 grid((unsigned)(a.B * a.npx * a.npy), (unsigned)((a.nstore + 32 * WN - 1) / (32 * WN)));
  conv_kernel<WX, WN, TAPS, C8><<<grid, 64 * WX * WN, lds, st>>>(a);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_conv(const ConvArgs &a, hipStream_t st) {
  const int Cin = a.Ca + a.Cb;
  if (a.taps == 1) return conv_as<4, 1, 1, false>(a, st);  // the head: 32 rows either way
  if (Cin == 8) return conv_as<4, 1, 9, true>(a, st);
  // 128 output channels of 64 pixels, 64 of 128, 32 of 256: the fewest wavefronts read the same weights or pixels
  if (a.nrows % 128 == 0) return conv_as<1, 4, 9, false>(a, st);
  if (a.nrows % 64 == 0) return conv_as<2, 2, 9, false>(a, st);
  return conv_as<4, 1, 9, false>(a, st);
}

namespace {
template <int TX, int WM, int WC, int XN>
void wgrad_as(const WgradArgs &a, hipStream_t st) {
  constexpr int BM = 32 * WM, BC = 16 * WC;
  const int splits = (a.B * a.H * a.W + kPixPerSplit - 1) / kPixPerSplit;
  const dim3 grid((unsigned)(a.M / BM), (unsigned)((a.Ca + a.Cb + BC - 1) / BC), (unsigned)(splits * TX));
  const size_t lds = 2 * ((size_t)a.xrows * (BC * 2 + 16) + kRun * (BM * 2 + 16));
  wgrad_kernel<TX, WM, WC, XN><<<grid, 64 * WM * WC, lds, st>>>(a);
}
// a magic reciprocal for quotients of numbers below 2^16, or 0 where they stay below 2 d
uint32_t small_div(int d) { return d >= 512 || d == 1 ? 0u : (uint32_t)(((uint64_t(1) << 32) + d - 1) / d); }
}  // namespace

hipError_t launch_wgrad(WgradArgs a, hipStream_t st) {
  const int rim = a.taps == 9 ? 2 : 0, W = a.W;
  // padded pixels of a run: it spans at most (W + kRun - 2) / W + 1 rows
  a.xrows = kRun + rim * ((W + kRun - 2) / W + 1);
  a.div_w = small_div(W);
  a.div_wr = small_div(W + rim);
  // 32 input channels per block (16 where there are only 8), and 64 output channels where there are as many
  const bool c32 = a.Ca % 32 == 0 && a.Cb % 32 == 0, wide = a.M % 64 == 0;
  // pieces per thread: a run of a wide image, or of any (every pixel a row of its own)
#define PDVM_WG(T, M, C)                                                                            \
  if (a.xrows * (2 * C) <= 64 * M * C * ((140 * 2 + 64 * M - 1) / (64 * M)))                        \
    wgrad_as<T, M, C, (140 * 2 + 64 * M - 1) / (64 * M)>(a, st);                                    \
  else                                                                                              \
    wgrad_as<T, M, C, (386 * 2 + 64 * M - 1) / (64 * M)>(a, st)
  if (a.taps == 1) {
    PDVM_WG(1, 1, 2);  // the head: 32 input channels
  } else if (!c32) {
    PDVM_WG(3, 1, 1);
  } else if (wide) {
    PDVM_WG(3, 2, 2);
  } else {
    PDVM_WG(3, 1, 2);
  }
#undef PDVM_WG
  return hipGetLastError();
}

hipError_t launch_colsum(const uint16_t *g, int64_t P, int C, float *part, hipStream_t st) {
  colsum_kernel<<<nblocks(P, 2 * kColsumPix), 256, 0, st>>>(g, P, C, part);
  return hipGetLastError();
}

hipError_t launch_sum_splits(const float *part, int splits, int64_t n, float *out, const float *bpart, int bsplits, int nb,
                             float *outb, hipStream_t st) {
  sum_splits_kernel<<<nblocks(n / 4, 256) + nblocks(nb, 32), 256, 0, st>>>(part, splits, n, out, bpart, bsplits, nb, outb);
  return hipGetLastError();
}

hipError_t launch_build_input(const uint8_t *solid_set, const float *feat_set, Slots sl, int B, int H, int W,
                              uint16_t *x, hipStream_t st) {
  build_input_kernel<<<nblocks((int64_t)B * H * W, 256), 256, 0, st>>>(solid_set, feat_set, sl, B, H, W, x);
  return hipGetLastError();
}

hipError_t launch_maxpool(const uint16_t *x, int B, int H, int W, int C, uint16_t *y, uint8_t *idx, hipStream_t st) {
  maxpool_kernel<<<nblocks((int64_t)B * (H / 2) * (W / 2) * C, 256), 256, 0, st>>>(x, B, H, W, C, y, idx);
  return hipGetLastError();
}

hipError_t launch_up_grad(const float *dcat, const uint16_t *y, int B, int H, int W, int Ca, int C, uint16_t *g,
                          hipStream_t st) {
  up_grad_kernel<<<nblocks((int64_t)B * (H / 2) * (W / 2) * (Ca / 8), 256), 256, 0, st>>>(dcat, y, B, H, W, Ca, C, g);
  return hipGetLastError();
}

hipError_t launch_pool_skip_grad(const float *dcat, int Ca, int C, const float *dp, const uint8_t *idx, const uint16_t *y,
                                 int B, int H, int W, int Cs, uint16_t *g, hipStream_t st) {
  pool_skip_grad_kernel<<<nblocks((int64_t)B * (H / 2) * (W / 2) * (Cs / 8), 256), 256, 0, st>>>(dcat, Ca, C, dp, idx, y,
                                                                                                B, H, W, Cs, g);
  return hipGetLastError();
}

hipError_t launch_loss(const float *pred, const uint8_t *solid_set, const float *target_set, const float *wsamp,
                       Slots sl, int B, int H, int W, uint16_t *g, float *part, int nblk, hipStream_t st) {
  loss_kernel<<<(unsigned)nblk, 256, 0, st>>>(pred, solid_set, target_set, wsamp, sl, B, H, W, g, part);
  return hipGetLastError();
}

hipError_t launch_adam(float *p, const float *g, float *m, float *v, int64_t n, float lr, float b1, float b2,
                       float eps, float c1, float c2, hipStream_t st) {
  adam_kernel<<<nblocks(n, 256), 256, 0, st>>>(p, g, m, v, n, lr, b1, b2, eps, c1, c2);
  return hipGetLastError();
}

hipError_t launch_to_bf16(const float *src, int64_t n, uint16_t *dst, hipStream_t st) {
  to_bf16_kernel<<<nblocks(n, 256), 256, 0, st>>>(src, n, dst);
  return hipGetLastError();
}

hipError_t launch_wt_back(WtBackArgs a, hipStream_t st) {
  if (a.layers < 1 || a.layers > WtBackArgs::kMax) return hipErrorInvalidValue;
  a.first[0] = 0;
  for (int l = 0; l < a.layers; ++l)
    a.first[l + 1] = a.first[l] + (int)(((int64_t)a.Cout[l] * a.Cin[l] * a.taps[l] + 255) / 256);
  wt_back_kernel<<<a.first[a.layers], 256, 0, st>>>(a);
  return hipGetLastError();
}

hipError_t launch_targets(const uint8_t *solid, const double *rho, const double *u, int H, int W, double jump,
                          double kn256, float *target, float *wsamp_one, hipStream_t st) {
  targets_kernel<<<1, 1024, 0, st>>>(solid, rho, u, H, W, jump, kn256, target, wsamp_one);
  return hipGetLastError();
}

hipError_t launch_fields(const float *pred, const uint8_t *solid, int H, int W, double jump, double kn256,
                         double *rho, double *u, hipStream_t st) {
  fields_kernel<<<nblocks((int64_t)H * W, 256), 256, 0, st>>>(pred, solid, H, W, jump, kn256, rho, u);
  return hipGetLastError();
}

}  // namespace pdvm_nn
