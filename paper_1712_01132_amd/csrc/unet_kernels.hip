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

constexpr int kPitch = 40;  // LDS row pitch in bf16: 32 k values + 8 pad (conflict-free 16-byte reads)

// One 8-channel group of the im2col matrix: row = output pixel (b, y, x),
// columns k .. k+7 (k a multiple of 8). Zero outside the image along y (zero
// padding), circular along x (the periodic flow axis), zero beyond K.
struct Im2col {
  const uint16_t *xa, *xb;
  int Ca, Cb, ups, taps, H, W, K, Cin;
  __device__ __forceinline__ uint4 load(int b, int y, int x, int k) const {
    uint4 v = make_uint4(0, 0, 0, 0);
    if (k >= K) return v;
    const int tap = k / Cin;
    const int c = k - tap * Cin;
    const int dy = taps == 9 ? tap / 3 - 1 : 0;
    const int dx = taps == 9 ? tap % 3 - 1 : 0;
    const int yy = y + dy;
    if (yy < 0 || yy >= H) return v;
    int xx = x + dx;
    xx = xx < 0 ? xx + W : (xx >= W ? xx - W : xx);
    const uint16_t *src;
    if (c < Ca) {
      src = ups ? xa + ((int64_t)((b * (H >> 1) + (yy >> 1)) * (W >> 1) + (xx >> 1))) * Ca + c
                : xa + ((int64_t)((b * H + yy) * W + xx)) * Ca + c;
    } else {
      src = xb + ((int64_t)((b * H + yy) * W + xx)) * Cb + (c - Ca);
    }
    return *reinterpret_cast<const uint4 *>(src);
  }
};

// out tile: 128 pixels x BN output channels, 4 wavefronts of 32 pixels each.
template <int BN>
__global__ void __launch_bounds__(256) conv_kernel(ConvArgs a) {
  __shared__ uint4 As[128 * kPitch / 8];
  __shared__ uint4 Bs[BN * kPitch / 8];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int P = a.B * a.H * a.W;
  const int p0 = blockIdx.x * 128;
  const int n0 = blockIdx.y * BN;
  const int Cin = a.Ca + a.Cb;
  const int K = a.taps * Cin;
  const int nk = (K + 31) / 32;
  const Im2col im{a.xa, a.xb, a.Ca, a.Cb, a.ups, a.taps, a.H, a.W, K, Cin};

  int pb[2], py[2], px[2];
  bool pv[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int p = p0 + (tid >> 2) + 64 * i;
    pv[i] = p < P;
    const int q = pv[i] ? p : 0;
    px[i] = q % a.W;
    const int t = q / a.W;
    py[i] = t % a.H;
    pb[i] = t / a.H;
  }
  const int kg = (tid & 3) * 8;
  const int brow = tid >> 2;
  const bool bload = brow < BN && n0 + brow < a.nrows;

  uint4 ra[2], rb = make_uint4(0, 0, 0, 0);
  auto gload = [&](int kt) {
    const int k = kt * 32 + kg;
#pragma unroll
    for (int i = 0; i < 2; ++i) ra[i] = pv[i] ? im.load(pb[i], py[i], px[i], k) : make_uint4(0, 0, 0, 0);
    rb = make_uint4(0, 0, 0, 0);
    if (bload && k < K) rb = *reinterpret_cast<const uint4 *>(a.wt + (int64_t)(n0 + brow) * K + k);
  };

  f32x4 acc[2][BN / 16];
#pragma unroll
  for (int ms = 0; ms < 2; ++ms)
#pragma unroll
    for (int ns = 0; ns < BN / 16; ++ns) acc[ms][ns] = f32x4{0.f, 0.f, 0.f, 0.f};

  gload(0);
  for (int kt = 0; kt < nk; ++kt) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) As[((tid >> 2) + 64 * i) * (kPitch / 8) + (tid & 3)] = ra[i];
    if (brow < BN) Bs[brow * (kPitch / 8) + (tid & 3)] = rb;
    __syncthreads();
    if (kt + 1 < nk) gload(kt + 1);
    bf16x8 fa[2], fb[BN / 16];
#pragma unroll
    for (int ms = 0; ms < 2; ++ms)
      fa[ms] = __builtin_bit_cast(bf16x8, As[(32 * wv + 16 * ms + (lane & 15)) * (kPitch / 8) + (lane >> 4)]);
#pragma unroll
    for (int ns = 0; ns < BN / 16; ++ns)
      fb[ns] = __builtin_bit_cast(bf16x8, Bs[(16 * ns + (lane & 15)) * (kPitch / 8) + (lane >> 4)]);
#pragma unroll
    for (int ms = 0; ms < 2; ++ms)
#pragma unroll
      for (int ns = 0; ns < BN / 16; ++ns)
        acc[ms][ns] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[ms], fb[ns], acc[ms][ns], 0, 0, 0);
  }

#pragma unroll
  for (int ns = 0; ns < BN / 16; ++ns) {
    const int n = n0 + 16 * ns + (lane & 15);
    if (n >= a.nstore) continue;
    const float bias = a.bias ? a.bias[n] : 0.f;
#pragma unroll
    for (int ms = 0; ms < 2; ++ms)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int p = p0 + 32 * wv + 16 * ms + 4 * (lane >> 4) + r;
        if (p >= P) continue;
        float v = acc[ms][ns][r] + bias;
        if (a.relu) v = fmaxf(v, 0.f);
        if (a.gate) v = bf2f(a.gate[(int64_t)p * a.ystride + n]) > 0.f ? v : 0.f;
        if (a.yb) a.yb[(int64_t)p * a.ystride + n] = f2bf(v);
        else a.yf[(int64_t)p * a.ystride + n] = v;
      }
  }
}

// dW partials. A wavefront owns 32 output channels x (all taps x 16 CB input
// channels), reduced over patches of 32 pixels (2^pw columns x 32 / 2^pw rows of
// one image); a block is WM wavefronts along the output channels x 4 / WM along
// the patches. Both operands are pixel-major in memory while the matrix
// instruction wants 8 consecutive pixels of one channel per lane: they are
// staged in LDS as they are (rows of pixels) and read with the transposing LDS
// load (ds_read_b64_tr_b16: lane l of 16 gets column l of 4 rows of 16 values).
// The input patch is staged once with its one-pixel rim, and each tap reads it
// at a shifted pixel; so a block reads the output gradient once per 16 CB input
// channels (not once per 32 im2col columns) and the input once (not per tap).
// The bias gradient is one more product, with a matrix of ones, in the blocks
// of the first input channels. With WM < 4 the wavefronts of one channel range add
// their sums through LDS at the end.
// Bound: the LDS reads (40 transposing loads per 36 matrix products of a patch).
// Measured (MI355X, training step on 8 x 256^2): all weight and bias gradients
// 0.67 ms, against 3.25 ms with 64 x 32 tiles transposed by 16-bit LDS writes and
// 1.4 ms of column sums; adding up the splits 0.17 ms, against 0.97.
constexpr int kPatch = 32;

typedef short v4s __attribute__((ext_vector_type(4)));
typedef short v8s __attribute__((ext_vector_type(8)));
__device__ __forceinline__ v4s tr_read(uint32_t addr) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s *)addr);
}
__device__ __forceinline__ bf16x8 tr_pair(uint32_t a0, uint32_t a1) {
  const v4s lo = tr_read(a0), hi = tr_read(a1);
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

template <int TAPS, int WM, int CB>
__global__ void __launch_bounds__(256) wgrad_kernel(WgradArgs a) {
  constexpr int WP = 4 / WM, BM = 32 * WM, BC = 16 * CB;
  constexpr int RIM = TAPS == 9 ? 1 : 0;
  constexpr int XROWS = TAPS == 9 ? 102 : 32;           // pixels of a patch with its rim, at most (32 x 1)
  constexpr int XP = BC * 2 + 16, GP = BM * 2 + 16;     // LDS row pitches in bytes
  constexpr int XCH = BC / 8, GCH = BM / 8;             // 16-byte chunks per pixel
  constexpr int XN = (WP * XROWS * XCH + 255) / 256, GN = WP * kPatch * GCH / 256;
  constexpr int XBYTES = WP * XROWS * XP, GBYTES = WP * kPatch * GP;
  constexpr int REDUCE = WP > 1 ? WM * TAPS * CB * 256 * 4 : 0;  // bytes of one 16-row half of the sums
  __shared__ __attribute__((aligned(16))) unsigned char lds[XBYTES + GBYTES > REDUCE ? XBYTES + GBYTES : REDUCE];
  __shared__ int4 base[2][WP];
  const uint32_t l0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int wm = wv % WM, wp = wv / WM;
  const int PW = 1 << a.pw, PH = kPatch >> a.pw, RW = PW + 2 * RIM, RR = (PH + 2 * RIM) * RW;
  const int m0 = blockIdx.x * BM, c0 = blockIdx.y * BC;
  const int qbeg = blockIdx.z * a.per_split, qend = min(a.patches, qbeg + a.per_split);
  const int Cin = a.Ca + a.Cb;
  // this block's channels come from one of the concatenated inputs
  const bool inA = c0 < a.Ca;
  const uint16_t *const xs = inA ? a.xa : a.xb;
  const int xc = inA ? c0 : c0 - a.Ca, xC = inA ? a.Ca : a.Cb;
  const int ups = inA ? a.ups : 0;

  // the pixel within a patch and the 16-byte chunk of each staged piece
  int xslot[XN], xry[XN], xrx[XN], xch[XN];
  uint32_t xto[XN];
#pragma unroll
  for (int i = 0; i < XN; ++i) {
    const int e = tid + 256 * i, px = e / XCH;
    xch[i] = e % XCH;
    const int sl = px / XROWS, r = px % XROWS;
    const bool ok = sl < WP && r < RR && xc + xch[i] * 8 < xC;
    xslot[i] = ok ? sl : -1;
    xry[i] = r / RW - RIM;
    xrx[i] = r % RW - RIM;
    xto[i] = sl < WP ? (uint32_t)((sl * XROWS + r) * XP + xch[i] * 16) : ~0u;
  }
  int gslot[GN], gpy[GN], gpx[GN], gch[GN];
#pragma unroll
  for (int i = 0; i < GN; ++i) {
    const int e = tid + 256 * i, px = e / GCH;
    gch[i] = e % GCH;
    gslot[i] = px / kPatch;
    gpy[i] = (px % kPatch) >> a.pw;
    gpx[i] = (px % kPatch) & (PW - 1);
  }
  // first pixel of patch q (its image, row and column; image -1 past the end)
  auto locate = [&](int q, int buf) {
    if (tid < WP) {
      const int qq = q + tid;
      const int x = qq % a.npx, t = qq / a.npx;
      base[buf][tid] = qq < qend ? make_int4(t / a.npy, t % a.npy * PH, x * PW, 0) : make_int4(-1, 0, 0, 0);
    }
  };
  uint4 rx[XN], rg[GN];
  auto load = [&](int buf) {
#pragma unroll
    for (int i = 0; i < XN; ++i) {
      rx[i] = make_uint4(0, 0, 0, 0);
      const int4 b = base[buf][max(xslot[i], 0)];
      const int y = b.y + xry[i];
      int x = b.z + xrx[i];
      // circular along x; past the right rim of a ragged last patch there is nothing to read
      const bool in = xslot[i] >= 0 && b.x >= 0 && y >= 0 && y < a.H && x <= a.W;
      x = x < 0 ? x + a.W : (x >= a.W ? x - a.W : x);
      if (in) {
        const int64_t p = ups ? (int64_t)(b.x * (a.H >> 1) + (y >> 1)) * (a.W >> 1) + (x >> 1)
                              : (int64_t)(b.x * a.H + y) * a.W + x;
        rx[i] = *reinterpret_cast<const uint4 *>(xs + p * xC + xc + xch[i] * 8);
      }
    }
#pragma unroll
    for (int i = 0; i < GN; ++i) {
      rg[i] = make_uint4(0, 0, 0, 0);
      const int4 b = base[buf][gslot[i]];
      const int y = b.y + gpy[i], x = b.z + gpx[i];
      if (b.x >= 0 && y < a.H && x < a.W)
        rg[i] = *reinterpret_cast<const uint4 *>(a.g + ((int64_t)(b.x * a.H + y) * a.W + x) * a.M + m0 + gch[i] * 8);
    }
  };
  // fragment addresses: pixel k = 8 (lane / 16) + 4 h + (lane % 16) / 4, columns 4 (lane % 4) ..
  const int kr = 8 * (lane >> 4) + ((lane & 15) >> 2), cq = 4 * (lane & 3);
  uint32_t ga[2], xa[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int k = kr + 4 * h;
    ga[h] = l0 + XBYTES + (uint32_t)((wp * kPatch + k) * GP + (wm * 32 + cq) * 2);
    xa[h] = l0 + (uint32_t)((wp * XROWS + (k >> a.pw) * RW + (k & (PW - 1))) * XP + cq * 2);
  }
  uint32_t toff[TAPS];
#pragma unroll
  for (int t = 0; t < TAPS; ++t) toff[t] = (uint32_t)((t / 3 * RW + t % 3) * XP);

  f32x4 acc[2][TAPS][CB], accb[2];
#pragma unroll
  for (int ms = 0; ms < 2; ++ms) {
    accb[ms] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < TAPS; ++t)
#pragma unroll
      for (int cs = 0; cs < CB; ++cs) acc[ms][t][cs] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const bool bias = blockIdx.y == 0;
  const bf16x8 ones = {(__bf16)1.f, (__bf16)1.f, (__bf16)1.f, (__bf16)1.f, (__bf16)1.f, (__bf16)1.f, (__bf16)1.f, (__bf16)1.f};

  locate(qbeg, 0);
  __syncthreads();
  load(0);
  locate(qbeg + WP, 1);
  int buf = 1;
  for (int q = qbeg; q < qend; q += WP) {
    __syncthreads();  // the last patch's reads are done; the next patch is located
#pragma unroll
    for (int i = 0; i < XN; ++i)
      if (xto[i] != ~0u) *reinterpret_cast<uint4 *>(lds + xto[i]) = rx[i];
#pragma unroll
    for (int i = 0; i < GN; ++i)
      *reinterpret_cast<uint4 *>(lds + XBYTES + (gslot[i] * kPatch + (tid + 256 * i) / GCH % kPatch) * GP + gch[i] * 16) = rg[i];
    __syncthreads();
    if (q + WP < qend) {
      load(buf);
      buf ^= 1;
      locate(q + 2 * WP, buf);
    }
    bf16x8 fa[2];
#pragma unroll
    for (int ms = 0; ms < 2; ++ms) fa[ms] = tr_pair(ga[0] + ms * 32, ga[1] + ms * 32);
    if (bias) {
#pragma unroll
      for (int ms = 0; ms < 2; ++ms) accb[ms] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[ms], ones, accb[ms], 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < TAPS; ++t)
#pragma unroll
      for (int cs = 0; cs < CB; ++cs) {
        const bf16x8 fb = tr_pair(xa[0] + toff[t] + cs * 32, xa[1] + toff[t] + cs * 32);
#pragma unroll
        for (int ms = 0; ms < 2; ++ms)
          acc[ms][t][cs] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[ms], fb, acc[ms][t][cs], 0, 0, 0);
      }
  }
  if (WP > 1) {  // the wavefronts of one channel range: their sums into wavefront wp = 0's
    f32x4 *const red = reinterpret_cast<f32x4 *>(lds) + wm * TAPS * CB * 64 + lane;
    for (int w = 1; w < WP; ++w) {
#pragma unroll
      for (int ms = 0; ms < 2; ++ms) {
        __syncthreads();
        if (wp == w) {
#pragma unroll
          for (int t = 0; t < TAPS; ++t)
#pragma unroll
            for (int cs = 0; cs < CB; ++cs) red[(t * CB + cs) * 64] = acc[ms][t][cs];
        }
        __syncthreads();
        if (wp == 0) {
#pragma unroll
          for (int t = 0; t < TAPS; ++t)
#pragma unroll
            for (int cs = 0; cs < CB; ++cs) acc[ms][t][cs] += red[(t * CB + cs) * 64];
        }
        __syncthreads();
        if (wp == w) red[0] = accb[ms];
        __syncthreads();
        if (wp == 0) accb[ms] += red[0];
      }
    }
    if (wp != 0) return;
  }
  // D[m = 4 (lane / 16) + r][n = lane % 16]; a split's partials are [M][taps * Cin] and then the M bias sums
  const int K = TAPS * Cin;
  float *const out = a.part + (int64_t)blockIdx.z * (a.M * (int64_t)(K + 1));
#pragma unroll
  for (int ms = 0; ms < 2; ++ms)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = m0 + wm * 32 + ms * 16 + 4 * (lane >> 4) + r;
#pragma unroll
      for (int t = 0; t < TAPS; ++t)
#pragma unroll
        for (int cs = 0; cs < CB; ++cs) {
          const int c = c0 + cs * 16 + (lane & 15);
          if (c < Cin) out[(int64_t)m * K + t * Cin + c] = acc[ms][t][cs][r];
        }
      if (bias && (lane & 15) == 0) out[(int64_t)a.M * K + m] = accb[ms][r];
    }
}

// out[i] = sum over the splits of part[split][i], four values per lane: 16
// wavefronts take every 16th split each, then add through LDS (a few hundred
// splits of a small layer read one after the other left most of the GPU idle).
__global__ void __launch_bounds__(1024) sum_splits_kernel(const float *part, int splits, int64_t n, float *out) {
  __shared__ f32x4 red[16][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t i = ((int64_t)blockIdx.x * 64 + lane) * 4;
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
  if (i < n)
    for (int j = w; j < splits; j += 16) s += *reinterpret_cast<const f32x4 *>(part + (int64_t)j * n + i);
  red[w][lane] = s;
  __syncthreads();
  if (w == 0 && i < n) {
#pragma unroll
    for (int k = 1; k < 16; ++k) s += red[k][lane];
    *reinterpret_cast<f32x4 *>(out + i) = s;
  }
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
__global__ void wt_back_kernel(const uint16_t *wt, int Cout, int Cin, int taps, uint16_t *wb) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)Cout * Cin * taps) return;
  const int o = (int)(i % Cout);
  int64_t r = i / Cout;
  const int t = (int)(r % taps);
  const int c = (int)(r / taps);
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

hipError_t launch_conv(const ConvArgs &a, hipStream_t st) {
  const int P = a.B * a.H * a.W;
  const bool wide = a.nstore > 32 && a.nrows % 64 == 0;
  if (wide) {
    dim3 grid(nblocks(P, 128), (unsigned)((a.nstore + 63) / 64));
    conv_kernel<64><<<grid, 256, 0, st>>>(a);
  } else {
    dim3 grid(nblocks(P, 128), (unsigned)((a.nstore + 31) / 32));
    conv_kernel<32><<<grid, 256, 0, st>>>(a);
  }
  return hipGetLastError();
}

namespace {
template <int TAPS, int WM, int CB>
void wgrad_as(const WgradArgs &a, int ctiles, hipStream_t st) {
  const dim3 grid((unsigned)(a.M / (32 * WM)), (unsigned)ctiles, (unsigned)((a.patches + a.per_split - 1) / a.per_split));
  wgrad_kernel<TAPS, WM, CB><<<grid, 256, 0, st>>>(a);
}
}  // namespace

WgradPlan wgrad_plan(int M, int Ca, int Cb, int taps, int B, int H, int W) {
  WgradPlan p;
  // wavefronts along the output channels: as many as there are 32-channel
  // ranges (the others split the patches); a power of two that divides M / 32
  p.wm = M % 128 == 0 ? 4 : (M % 64 == 0 ? 2 : 1);
  const int Cin = Ca + Cb;
  p.cb = Ca % 32 == 0 && Cb % 32 == 0 ? 2 : 1;  // 32 input channels a block; 16 where a part has an odd 16 or 8
  const int tiles = M / (32 * p.wm) * ((Cin + 16 * p.cb - 1) / (16 * p.cb));
  p.max_splits = std::max(1, kWgradBlocks / tiles);
  // patches as wide as the image up to 32 pixels (rounded up to a power of two)
  p.pw = 0;
  while ((1 << p.pw) < std::min(W, kPatch)) ++p.pw;
  const int PW = 1 << p.pw, PH = kPatch >> p.pw;
  p.npx = (W + PW - 1) / PW;
  p.npy = (H + PH - 1) / PH;
  p.patches = B * p.npx * p.npy;
  const int wp = 4 / p.wm;
  p.per_split = (p.patches + p.max_splits - 1) / p.max_splits;
  p.per_split = (p.per_split + wp - 1) / wp * wp;
  p.splits = (p.patches + p.per_split - 1) / p.per_split;
  (void)taps;
  return p;
}

hipError_t launch_wgrad(const WgradArgs &a, const WgradPlan &p, hipStream_t st) {
  const int ct = (a.Ca + a.Cb + 16 * p.cb - 1) / (16 * p.cb);
#define PDVM_WG(T, C)                          \
  if (p.wm == 4) wgrad_as<T, 4, C>(a, ct, st); \
  else if (p.wm == 2) wgrad_as<T, 2, C>(a, ct, st); \
  else wgrad_as<T, 1, C>(a, ct, st)
  if (a.taps == 9 && p.cb == 2) { PDVM_WG(9, 2); }
  else if (a.taps == 9) { PDVM_WG(9, 1); }
  else if (p.cb == 2) { PDVM_WG(1, 2); }
  else { PDVM_WG(1, 1); }
#undef PDVM_WG
  return hipGetLastError();
}

hipError_t launch_sum_splits(const float *part, int splits, int64_t n, float *out, hipStream_t st) {
  sum_splits_kernel<<<nblocks(n, 256), 1024, 0, st>>>(part, splits, n, out);
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

hipError_t launch_wt_back(const uint16_t *wt, int Cout, int Cin, int taps, uint16_t *wb, hipStream_t st) {
  wt_back_kernel<<<nblocks((int64_t)Cout * Cin * taps, 256), 256, 0, st>>>(wt, Cout, Cin, taps, wb);
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
