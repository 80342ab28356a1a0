// Warm-start network: kernel arguments and launchers (internal).
//
// Activations are NHWC bfloat16 (stored as raw 16-bit words, round to nearest
// even); accumulation is FP32 on the matrix cores.  A view of a tensor is a
// base pointer, a channel count and the element stride between pixels, so a
// layer can read or write a channel slice of a wider buffer (the skip
// concatenation needs no copies).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fft_engine.hpp"

namespace lshom {
namespace cnn {

using bf16_t = uint16_t;

// Pixel maps of the implicit GEMM (output pixel (b, i, j) on an Ho x Wo grid).
enum ConvMode : int {
  CM_CONV3 = 0,    // 9 taps, input ((i + p - 1) mod Ho) / up, ((j + q - 1) mod Wo) / up
  CM_DOWN3 = 1,    // 9 taps, input (3 i + p, 3 j + q)
  CM_POINT = 2,    // 1 tap, input (i, j)
  CM_DOWN3_T = 3,  // 1 tap per launch slice z = 3 p + q: input (i, j), output (3 i + p, 3 j + q)
};

struct ConvArgs {
  const bf16_t* in0;     // channels [0, C0)
  int C0, ld0;           // channel count and pixel stride (multiples of 8)
  int B, Hi, Wi, Ho, Wo;
  int mode, up;
  const bf16_t* w;       // weights in fragment order (WeightTiles): wblocks blocks of 32
  int wsteps, wblocks;   // output channels, wsteps steps of 32 of the reduction
  int N, Np;             // output channels, padded to a multiple of 8
  const float* bias;     // [N] or null
  int relu;
  bf16_t* out_b;         // bf16 output (or null): pixel stride ldb
  int ldb;
  float* out_f;          // FP32 output (or null): pixel stride ldf
  int ldf;
  // Input gradients (mask given): channels below n_b leave as the next layer's
  // operand, bf16((value + add) where mask > 0, else 0) in out_b; the others
  // in FP32 as channels 0, 1, .. of out_f.
  const bf16_t* mask;    // activation whose ReLU the gradient passes, or null: pixel stride ldm
  int ldm;
  const float* add;      // second gradient of the activation, or null: pixel stride lda
  int lda;
  int n_b;               // a multiple of 8
  int wide_b, wide_f, wide_m;  // 16-byte accesses fit the base and stride (set by the launcher)
  FastDiv fd_chunks;     // C0 / 8 (set by the launcher)
};

struct WgradArgs {
  const bf16_t* in0;
  int C0, ld0;           // input channels (a multiple of 8) and pixel stride
  int B, Hi, Wi, Ho, Wo;
  int mode, up;          // CM_CONV3, CM_DOWN3 or CM_POINT
  const bf16_t* gy;      // [B Ho Wo][ldg], Np channels used
  int ldg, Np;
  int taps;
  int rows;              // taps C0 + 1: the last row sums gy (bias gradient)
  long long pix_per_split;
  float* partial;        // [splits][rows][Np]
};

constexpr int kWgradRows = 32;  // rows of the im2col matrix per wave
constexpr int kWgradWaves = 4;  // waves per block: row tiles of one split, which read the same pixels
// Pixel splits of a layer's weight gradient; each holds a multiple of 32
// pixels (one step of the kernel).
inline int wgrad_splits(long long pixels) {
  const long long s = (pixels + 8191) / 8192;
  return (int)(s < 64 ? s : 64);
}

// The kernel of a launch, by its shape.  Convolutions: the LDS patch of th
// rows with the four waves in cw channel halves, or (th 0) wave tiles of 16 mt
// pixels x 32 np channels straight from global memory.  Weight gradients:
// columns per wave, and whether an image row is shorter than a lane's step.
struct ConvVariant {
  int th, cw, mt, np;
};
struct WgradVariant {
  int columns;
  bool small;
};
ConvVariant conv_variant(const ConvArgs& a);
WgradVariant wgrad_variant(const WgradArgs& a, int splits);
hipError_t launch_conv(const ConvArgs& a, hipStream_t s);
hipError_t launch_wgrad(const WgradArgs& a, int splits, hipStream_t s);
// grad[r][n] = sum_s partial[s][r][n] for r < rows (fixed order); row r = t cin
// + c goes to grad_w[(t cin_real + c) cout + n] where c < cin_real and n < cout,
// the last row to grad_b[n].
hipError_t launch_wgrad_reduce(const float* partial, int splits, int rows, int Np, int cin, int cin_real, int cout,
                               float* grad_w, float* grad_b, hipStream_t s);

// gpre[p][c] = bf16(g[p * ld + c]), c < C, zero for C <= c < Cp.
hipError_t launch_grad_prep(long long P, int C, int Cp, const float* g, int ld, bf16_t* gpre, hipStream_t s);
// coarse[b, I, J, c] = sum over the 3 x 3 fine pixels of fine[b, 3I+p, 3J+q, c];
// with act [B, Hc, Wc, C] the sum where act > 0, else 0, as bf16 in coarse_b.
hipError_t launch_pool3_sum(int B, int Hc, int Wc, int C, const float* fine, float* coarse, const bf16_t* act,
                            bf16_t* coarse_b, hipStream_t s);
// Network input [B, N, N, 8]: phase indicator (phase != 0), log10(rho) / 4, zeros.
// transpose: read the image transposed (load case E = e2).  scale 3: the
// image is 3N x 3N and pixel (i, j) is the majority of block (3i.., 3j..).
hipError_t launch_make_input(int B, int N, const uint8_t* phase, const float* log10_rho, int transpose, int scale,
                             bf16_t* x, hipStream_t s);
// Relative MSE of pred [B, N, N, 2] (FP32, pixel stride 2) against the
// fluctuation of FP64 planar fields e [B][2][N][N] for E = e1; writes the
// loss (device scalar) and the FP32 gradient [B, N, N, 2].  part: 2 B * 256
// doubles of scratch.
hipError_t launch_rel_mse(int B, int N, const float* pred, const double* e, double* part, double* loss,
                          float* grad, hipStream_t s);
// Predicted field (FP64 planar [B][2][N][N]): E + prediction; transpose maps
// the prediction for the transposed image to the load case E = e2.
// scale 3: the field is 3N x 3N, pixel (i, j) takes prediction (i / 3, j / 3).
hipError_t launch_make_field(int B, int N, const float* pred, int transpose, int scale, double* e, hipStream_t s);
// A bfloat16 weight operand of the convolutions: `blocks` blocks of 32 rows
// (output channels of the product), `steps` steps of 32 of its reduction, each
// step of a half block 1 KB in the matrix cores' fragment order.
struct WeightTiles {
  int blocks, steps;
  long long elements() const { return (long long)blocks * 2 * steps * 512; }
};
inline WeightTiles weight_tiles_fwd(int taps, int cin, int np) { return {(np + 31) / 32, (taps * cin + 31) / 32}; }
// tap_pad: the reduction of every tap padded to whole steps (the input
// gradient of a stride-3 layer takes one tap per launch slice)
inline WeightTiles weight_tiles_grad(int taps, int cin, int np, int tap_pad) {
  return {(cin + 31) / 32, tap_pad ? taps * ((np + 31) / 32) : (taps * np + 31) / 32};
}
// Both copies of every layer's master weights w[t][c][o] (taps x cin_real x
// cout, zeros up to cin and np): w16 for the forward convolution, wt16 for the
// input gradient (conv3 flips the taps, t' = 8 - t; down3 and 1x1 keep them).
constexpr int kCastLayers = 24;
struct CastLayer {
  long long w_off, f_off, t_off;  // elements into w, w16, wt16
  int taps, cin, cin_real, cout, np, flip, tap_pad;
  int steps_f, steps_t;           // set by the launcher, as the following
  long long n_f, n_t;
  unsigned first;                 // first block of the layer
};
struct CastArgs {
  const float* w;
  bf16_t *w16, *wt16;
  int layers;
  CastLayer layer[kCastLayers];
};
hipError_t launch_cast_weights(const CastArgs& a, hipStream_t s);
hipError_t launch_adam(long long n, float* w, const float* g, float* m, float* v, float lr, float b1, float b2,
                       float eps, float c1, float c2, hipStream_t s);
hipError_t launch_fill_f32(float* p, long long n, float v, hipStream_t s);

}  // namespace cnn
}  // namespace lshom
