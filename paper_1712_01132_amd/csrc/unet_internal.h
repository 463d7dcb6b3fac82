// Internal declarations of the warm-start network kernels (unet_kernels.hip)
// used by its host runtime (unet_host.cpp). Not part of the public C ABI.
//
// Tensors are NHWC: element (b, y, x, c) at ((b * H + y) * W + x) * C + c,
// x = the flow axis x1 (periodic: circular padding), y = x2 (zero padding).
// Activations and MFMA operands are bfloat16 (stored as raw 16-bit words,
// rounded to nearest even); accumulation, biases, gradients of activations and
// master weights are FP32.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace pdvm_nn {

constexpr int kMaxBatch = 32;
constexpr int kInC = 8;  // input channels: solid, scaled log Kn, six zero pads
constexpr int kColsumPix = 1024;    // rows per partial of the bias gradients
constexpr int kPixPerSplit = 4096;  // pixels per partial of the weight gradients

struct Slots {
  int32_t s[kMaxBatch];
};

// Convolution as an implicit GEMM: out[p][n] = sum_k A[p][k] Wt[n][k] (+ bias,
// ReLU), k = tap * Cin + c over `taps` (9: 3x3, or 1: 1x1) and the
// concatenated input channels [A (Ca, optionally read at (y/2, x/2)), B (Cb)].
struct ConvArgs {
  const uint16_t *xa;
  const uint16_t *xb;
  int Ca, Cb, ups;
  const uint16_t *wt;  // [nrows][taps * (Ca + Cb)]
  int nrows;           // weight rows allocated (>= every stored n)
  const float *bias;   // [nrows] or null
  int taps;
  int B, H, W;
  int relu;
  uint16_t *yb;        // bf16 output or null
  float *yf;           // fp32 output or null
  int nstore, ystride; // channels stored, channel stride of the output
  const uint16_t *gate;  // null, or laid out as the output: where it is not positive, 0 is stored
  // set by launch_conv: tiles of 2^pw columns, npx x npy per image; reciprocals of
  // the chunks per pixel and of the patch's columns
  int pw, npx, npy;
  uint32_t div_ch, div_rw;
};

// Weight gradient partials: part[split][m][k] = sum over the split's pixels of
// G[p][m] * A[p][k], with G the bf16 gradient at the conv output ([p][M]) and A the
// im2col matrix of the conv input.
struct WgradArgs {
  const uint16_t *g;
  int M;               // output channels (a multiple of 32)
  const uint16_t *xa;
  const uint16_t *xb;
  int Ca, Cb, ups, taps;
  int B, H, W;
  float *part;
  int xrows;               // set by launch_wgrad: padded pixels staged per run,
  uint32_t div_w, div_wr;  // reciprocals of the image's width and padded width
};

hipError_t launch_conv(const ConvArgs &a, hipStream_t st);
hipError_t launch_wgrad(WgradArgs a, hipStream_t st);
// ceil(P / kColsumPix) partials: part[.][C]
hipError_t launch_colsum(const uint16_t *g, int64_t P, int C, float *part, hipStream_t st);
// weight gradients from `splits` partials of n values, bias gradients from bsplits of nb
hipError_t launch_sum_splits(const float *part, int splits, int64_t n, float *out, const float *bpart, int bsplits, int nb,
                             float *outb, hipStream_t st);
hipError_t launch_build_input(const uint8_t *solid_set, const float *feat_set, Slots sl, int B, int H, int W,
                              uint16_t *x, hipStream_t st);
hipError_t launch_maxpool(const uint16_t *x, int B, int H, int W, int C, uint16_t *y, uint8_t *idx, hipStream_t st);
hipError_t launch_up_grad(const float *dcat, const uint16_t *y, int B, int H, int W, int Ca, int C, uint16_t *g,
                          hipStream_t st);
hipError_t launch_pool_skip_grad(const float *dcat, int Ca, int C, const float *dp, const uint8_t *idx, const uint16_t *y,
                                 int B, int H, int W, int Cs, uint16_t *g, hipStream_t st);
hipError_t launch_loss(const float *pred, const uint8_t *solid_set, const float *target_set, const float *wsamp,
                       Slots sl, int B, int H, int W, uint16_t *g, float *part, int nblk, hipStream_t st);
hipError_t launch_adam(float *p, const float *g, float *m, float *v, int64_t n, float lr, float b1, float b2,
                       float eps, float c1, float c2, hipStream_t st);
hipError_t launch_to_bf16(const float *src, int64_t n, uint16_t *dst, hipStream_t st);
// The weights of every input-gradient convolution (nothing for layer 0's), one
// launch: layer l's from wt + off[l] to wb + off[l].
struct WtBackArgs {
  static constexpr int kMax = 16;
  const uint16_t *wt;
  uint16_t *wb;
  int layers;
  int64_t off[kMax];
  int Cout[kMax], Cin[kMax], taps[kMax];
  int first[kMax + 1];  // set by the launch: each layer's first block
};
hipError_t launch_wt_back(WtBackArgs a, hipStream_t st);
hipError_t launch_targets(const uint8_t *solid, const double *rho, const double *u, int H, int W, double jump,
                          double kn256, float *target, float *wsamp_one, hipStream_t st);
hipError_t launch_fields(const float *pred, const uint8_t *solid, int H, int W, double jump, double kn256,
                         double *rho, double *u, hipStream_t st);

// Normalisation shared by training targets and predictions.
constexpr double kUScale = 10.0;   // U
constexpr double kKnKnee = 10.0;   // a in sigma(K) = a K / (1 + a K)
constexpr double kRefLen = 256.0;  // voxels of the reference length of Kn and of the gradient

}  // namespace pdvm_nn
