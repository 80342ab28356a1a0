// Warm-start network kernels for gfx950: implicit-GEMM convolutions on the
// matrix cores (bfloat16 inputs, FP32 accumulation), the weight gradient as
// a split-K GEMM with a fixed-order reduction, and the elementwise steps.
#include <type_traits>

#include "cnn.hpp"

namespace lshom {
namespace cnn {

typedef float float4_t __attribute__((ext_vector_type(4)));

// Round to nearest even (finite inputs).
__device__ __forceinline__ bf16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(bf16_t h) { return __uint_as_float((uint32_t)h << 16); }

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

// Implicit-GEMM convolution on the matrix cores (16x16x32 bfloat16 MFMA, FP32
// accumulation): out[pixel][n] = sum_k im2col(in)[pixel][k] w[n][k], the
// reduction 32 at a time in the order (tap, channel).
//
// A lane's fragment is eight consecutive k of one row of each operand.  The
// weights are stored in fragment order (1 KB per 16 channels and step, a
// lane's 16 bytes at 16 lane): read row by row, the 16 lanes of a quarter
// wave would touch 16 lines a load, and the vector cache's port, not the
// matrix cores, would set the pace (256 -> 256 channels on 9^2: 27 us by rows).
// The weights are the first operand: an accumulator then holds channels of
// one pixel, and the rows of a tile pair are dealt so that a lane ends with
// eight consecutive channels of its pixel (one 16-byte store).

// The lane's part of step 0 of the weight tile that holds half nt of the
// channels 32 cb .. 32 cb + 31 (steps 512 elements apart; see cast_weights_kernel).
__device__ __forceinline__ const bf16_t* conv_weight_tile(const ConvArgs& a, int cb, int nt, int lane) {
  return a.w + ((long long)(2 * cb + nt) * a.wsteps * 64 + lane) * 8;
}

// Store channels n .. n + 7 (below a.N) of output pixel op: bias, ReLU, rounding.
__device__ __forceinline__ void conv_store(const ConvArgs& a, long long op, int n, const float4_t& lo,
                                           const float4_t& hi, const float (&bias)[8]) {
  float v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    v[e] = (e < 4 ? lo[e & 3] : hi[e & 3]) + bias[e];
    if (a.relu) v[e] = fmaxf(v[e], 0.f);
  }
  bool to_b = a.out_b != nullptr, to_f = a.out_f != nullptr;
  int nf = n;
  if (a.mask) {
    to_b = n < a.n_b;
    to_f = !to_b;
    nf = n - a.n_b;
    if (to_b) {
      const long long om = op * a.ldm + n, oa = op * a.lda + n;
      const bool all = n + 8 <= a.N;
      bf16_t m[8];
      float w[8];
      if (all && a.wide_m) {
        const uint4 q = *reinterpret_cast<const uint4*>(a.mask + om);
        const uint32_t qw[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) m[e] = (bf16_t)(qw[e >> 1] >> (16 * (e & 1)));
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) m[e] = n + e < a.N ? a.mask[om + e] : (bf16_t)0;
      }
      if (a.add) {
#pragma unroll
        for (int e = 0; e < 8; ++e) w[e] = n + e < a.N ? a.add[oa + e] : 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += w[e];
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = bf2f(m[e]) > 0.f ? v[e] : 0.f;
    }
  }
  if (to_b) {
    bf16_t* o = a.out_b + op * a.ldb + n;
    if (n + 8 <= a.N && a.wide_b) {
      uint4 w;
      w.x = f2bf(v[0]) | ((uint32_t)f2bf(v[1]) << 16);
      w.y = f2bf(v[2]) | ((uint32_t)f2bf(v[3]) << 16);
      w.z = f2bf(v[4]) | ((uint32_t)f2bf(v[5]) << 16);
      w.w = f2bf(v[6]) | ((uint32_t)f2bf(v[7]) << 16);
      *reinterpret_cast<uint4*>(o) = w;
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (n + e < a.N) o[e] = f2bf(v[e]);
    }
  }
  if (to_f) {
    float* o = a.out_f + op * a.ldf + nf;
    if (n + 8 <= a.N && a.wide_f) {
      *reinterpret_cast<float4_t*>(o) = float4_t{v[0], v[1], v[2], v[3]};
      *reinterpret_cast<float4_t*>(o + 4) = float4_t{v[4], v[5], v[6], v[7]};
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (n + e < a.N) o[e] = v[e];
    }
  }
}

// The bias of channels n .. n + 7.
__device__ __forceinline__ void conv_bias(const ConvArgs& a, int n, float (&bias)[8]) {
#pragma unroll
  for (int e = 0; e < 8; ++e) bias[e] = (a.bias && n + e < a.N) ? a.bias[n + e] : 0.f;
}

// Neighbouring blocks share input rows: one contiguous run of blocks per XCD.
__device__ __forceinline__ unsigned conv_xcd_block() {
  const unsigned total = gridDim.x, xcd = blockIdx.x & 7u, slot = blockIdx.x >> 3;
  const unsigned q = total >> 3, rem = total & 7u;
  return xcd * q + (xcd < rem ? xcd : rem) + slot;
}

// Circular 3x3 convolution (CM_CONV3) with the input patch in LDS: a block
// computes TH x 32 pixels of one image, its (TH + 2) x 34 input pixels staged
// once with every channel (the nearest-neighbour upsampling of an up layer
// applied on the way), so that the nine taps read LDS and global memory sees
// each value about once; read per tap from the vector cache the layer is
// bound by it (243^2, 32 -> 32 channels: 107 us, whatever the number of loads
// in flight).  A pixel's row in LDS is its channels and 16 bytes more, which
// spreads eight consecutive pixels over all banks.  The weights' fragments
// come straight from global memory, three steps ahead.  A wave owns MT tiles
// of 16 pixels x 32 channels; with CW = 2 the four waves split 64 channels
// two ways, so that each weight fragment feeds twice the pixels (81^2, 128 ->
// 64 channels: 76 -> 50 us).
// 16 images, the layer alone with both outputs, against two LDS buffers of
// im2col rows with a block barrier per step: 243^2, 32 -> 32 channels 110 ->
// 51 us (the FP32 output is 121 MB of its 242); 81^2, 128 -> 64 63 -> 39 us;
// 27^2, 256 -> 128 54 -> 25 us.  Inference of 16 images 1.40 -> 0.70 ms.
template <int TH, int CW, bool UNI>
__global__ __launch_bounds__(256) void conv3_tile_kernel(ConvArgs a) {
  constexpr int TW = 32, PW = TW + 2, MT = TH * CW / 2, D = 3;
  extern __shared__ __align__(16) unsigned char patch[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, g = lane >> 4;
  const int W = a.Wo, H = a.Ho;
  const int Cin = a.C0, K = 9 * Cin;
  const int n0 = (int)(blockIdx.y * CW + (CW == 1 ? 0 : wave % CW)) * 32;
  const unsigned tw = (unsigned)((W + TW - 1) / TW), th = (unsigned)((H + TH - 1) / TH);
  const unsigned bx = conv_xcd_block();
  const int b = (int)(bx / (tw * th));
  const unsigned rem = bx - (unsigned)b * tw * th;
  const int i0 = (int)(rem / tw) * TH, j0 = (int)(rem % tw) * TW;

  // the weights' first steps, then the patch
  const bf16_t* wt[2];
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) wt[nt] = conv_weight_tile(a, n0 / 32 < a.wblocks ? n0 / 32 : 0, nt, lane);
  uint4 pw[D][2];
  const int steps = (K + 31) / 32;
  auto fetch = [&](int s, int d) {
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) pw[d][nt] = *reinterpret_cast<const uint4*>(wt[nt] + 512ll * s);
  };
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (d < steps) fetch(d, d);

  const int pitch = 2 * Cin + 16;  // bytes of a pixel in the patch
  {
    const uint32_t chunks = (uint32_t)Cin / 8u, total = (uint32_t)((TH + 2) * PW) * chunks;
    const bf16_t* img = a.in0 + (long long)b * a.Hi * a.Wi * a.ld0;
    constexpr int kIn = 6;  // loads in flight per thread
    for (uint32_t e0 = tid; e0 < total; e0 += 256 * kIn) {
      uint4 v[kIn];
      uint32_t at[kIn];
#pragma unroll
      for (int u = 0; u < kIn; ++u) {
        const uint32_t e = e0 + 256u * u;
        const uint32_t px = fdiv(e, a.fd_chunks), c = e - px * chunks;
        const int hy = (int)(px / PW), hx = (int)(px - (px / PW) * PW);
        // circular; beyond the image's end any pixel serves (not stored)
        int ii = i0 + hy - 1, jj = j0 + hx - 1;
        ii += ii < 0 ? H : 0;
        ii -= ii >= H ? H : 0;
        jj += jj < 0 ? W : 0;
        jj -= jj >= W ? W : 0;
        if (a.up == 3) {
          ii = (int)((uint32_t)ii / 3u);
          jj = (int)((uint32_t)jj / 3u);
        }
        at[u] = px * (uint32_t)pitch + c * 16u;
        v[u] = uint4{0u, 0u, 0u, 0u};
        if (e < total) v[u] = *reinterpret_cast<const uint4*>(img + ((long long)ii * a.Wi + jj) * a.ld0 + 8 * c);
      }
#pragma unroll
      for (int u = 0; u < kIn; ++u)
        if (e0 + 256u * u < total) *reinterpret_cast<uint4*>(patch + at[u]) = v[u];
    }
  }
  __syncthreads();

  // tile T = (wave / CW) MT + mt: row T / 2, columns 16 (T % 2) ..
  const unsigned char* px0[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int T = (wave / CW) * MT + mt;
    px0[mt] = patch + ((T >> 1) * PW + 16 * (T & 1) + li) * pitch + (UNI ? 16 * g : 0);
  }
  float4_t acc[MT][2];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) acc[mt][nt] = float4_t{0.f, 0.f, 0.f, 0.f};
  int tap = 0, off = 0, cc = 0;  // UNI: byte offset of the step's tap and channels
  for (int s0 = 0; s0 < steps; s0 += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int s = s0 + d;
      if (s >= steps) break;
      bf16x8_t fa[MT];
      if constexpr (UNI) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) fa[mt] = *reinterpret_cast<const bf16x8_t*>(px0[mt] + off + 2 * cc);
        cc += 32;
        if (cc == Cin) {
          cc = 0;
          ++tap;
          off = ((tap / 3) * PW + tap % 3) * pitch;
        }
      } else {
        const int k = 32 * s + 8 * g;
        const bool in = k < K;
        const int t = in ? k / Cin : 0, c = in ? k - t * Cin : 0;
        const int o = ((t / 3) * PW + t % 3) * pitch + 2 * c;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          const uint4 v = *reinterpret_cast<const uint4*>(px0[mt] + o);
          fa[mt] = __builtin_bit_cast(bf16x8_t, in ? v : uint4{0u, 0u, 0u, 0u});
        }
      }
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
          acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, pw[d][nt]), fa[mt],
                                                                acc[mt][nt], 0, 0, 0);
      if (s + D < steps) fetch(s + D, d);
    }
  }

  const int n = n0 + 8 * g;
  if (n >= a.N) return;
  float bias[8];
  conv_bias(a, n, bias);
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int T = (wave / CW) * MT + mt;
    const int i = i0 + (T >> 1), j = j0 + 16 * (T & 1) + li;
    if (i >= H || j >= W) continue;
    conv_store(a, ((long long)b * H + i) * W + j, n, acc[mt][0], acc[mt][1], bias);
  }
}

// The other convolutions (stride-3, its transpose, 1x1: every input value is
// used by one tap) and the 3x3 ones of small images: every fragment straight
// from global memory, no LDS and no barrier.  A wave computes 16 MT pixels x
// 32 NP channels; the loads of the next D steps are in flight while a step
// multiplies.
//
// UNI: the input channels are a multiple of 32, so a step lies in one tap for
// all lanes; otherwise each lane finds the tap of its eight k.
template <int MT, int NP, int TAPS, bool UNI, int D>
__global__ __launch_bounds__(256) void conv_kernel(ConvArgs a) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int li = lane & 15, g = lane >> 4;
  const unsigned bx = conv_xcd_block();
  const int W = a.Wo, H = a.Ho;
  const int hw = H * W;
  const int M = a.B * hw;  // below 2^25
  const int m0 = (int)(bx * 4 + wave) * (16 * MT);
  if (m0 >= M) return;
  const int n0 = blockIdx.y * (32 * NP);
  const int z = blockIdx.z;
  const int Cin = a.C0;
  const int K = TAPS * Cin;
  const uint32_t ld8 = (uint32_t)a.ld0 / 8u;

  // first pixel (in units of 8 elements) of the input rows, and the input
  // columns, of the taps of the lane's pixel in each tile
  uint32_t rowoff[MT][TAPS == 9 ? 3 : 1], coloff[MT][TAPS == 9 ? 3 : 1];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    int m = m0 + 16 * mt + li;
    m = m < M ? m : M - 1;  // rows past the end are computed and not stored
    const int b = m / hw, rem = m - b * hw;
    const int i = rem / W, j = rem - i * W;
    if constexpr (TAPS == 9) {
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        int ii = 3 * i + t, jj = 3 * j + t;
        if (a.mode == CM_CONV3) {
          ii = i + t - 1;
          ii += ii < 0 ? H : 0;
          ii -= ii >= H ? H : 0;
          jj = j + t - 1;
          jj += jj < 0 ? W : 0;
          jj -= jj >= W ? W : 0;
          if (a.up == 3) {
            ii = (int)((uint32_t)ii / 3u);
            jj = (int)((uint32_t)jj / 3u);
          }
        }
        rowoff[mt][t] = (uint32_t)(b * a.Hi + ii) * (uint32_t)a.Wi * ld8;
        coloff[mt][t] = (uint32_t)jj * ld8;
      }
    } else {
      rowoff[mt][0] = (uint32_t)(b * a.Hi + i) * (uint32_t)a.Wi * ld8;
      coloff[mt][0] = (uint32_t)j * ld8;
    }
  }
  const bf16_t* wt[2 * NP];
#pragma unroll
  for (int nt = 0; nt < 2 * NP; ++nt) {
    const int cb = n0 / 32 + (nt >> 1);
    wt[nt] = conv_weight_tile(a, cb < a.wblocks ? cb : 0, nt & 1, lane) +
             (a.mode == CM_DOWN3_T ? (long long)z * ((Cin + 31) / 32) * 512 : 0);
  }

  // (values first: a conditional on the array elements themselves would index the arrays in scratch memory)
  auto tap_pixel = [&](int mt, int p, int q) -> uint32_t {
    if constexpr (TAPS == 9) {
      const uint32_t r0 = rowoff[mt][0], r1 = rowoff[mt][1], r2 = rowoff[mt][2];
      const uint32_t c0 = coloff[mt][0], c1 = coloff[mt][1], c2 = coloff[mt][2];
      return (p == 0 ? r0 : (p == 1 ? r1 : r2)) + (q == 0 ? c0 : (q == 1 ? c1 : c2));
    } else {
      return rowoff[mt][0] + coloff[mt][0];
    }
  };
  uint4 pa[D][MT], pw[D][2 * NP];
  const bf16_t* src[MT];  // the lane's eight channels of the fetch position (UNI)
  int fp = 0, fq = 0, fc = 0;
  auto tap_source = [&]() {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      src[mt] = a.in0 + 8ull * tap_pixel(mt, fp, fq) + 8 * g;
    }
  };
  if constexpr (UNI) tap_source();
  auto fetch = [&](int s, int d) {
    if constexpr (UNI) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) pa[d][mt] = *reinterpret_cast<const uint4*>(src[mt] + fc);
#pragma unroll
      for (int nt = 0; nt < 2 * NP; ++nt) pw[d][nt] = *reinterpret_cast<const uint4*>(wt[nt] + 512ll * s);
      fc += 32;
      if (fc == Cin) {
        fc = 0;
        if (++fq == 3) {
          fq = 0;
          ++fp;
        }
        if (fp < 3) tap_source();
      }
    } else {
      const int k = 32 * s + 8 * g;
      const bool in = k < K;
      const int t = in ? k / Cin : 0, c = in ? k - t * Cin : 0;
      const int p = TAPS == 9 ? t / 3 : 0, q = TAPS == 9 ? t - 3 * p : 0;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const uint4 v = *reinterpret_cast<const uint4*>(a.in0 + 8ull * tap_pixel(mt, p, q) + c);
        pa[d][mt] = in ? v : uint4{0u, 0u, 0u, 0u};
      }
#pragma unroll
      for (int nt = 0; nt < 2 * NP; ++nt) pw[d][nt] = *reinterpret_cast<const uint4*>(wt[nt] + 512ll * s);
    }
  };

  float4_t acc[MT][2 * NP];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < 2 * NP; ++nt) acc[mt][nt] = float4_t{0.f, 0.f, 0.f, 0.f};
  const int steps = (K + 31) / 32;
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (d < steps) fetch(d, d);
  for (int s0 = 0; s0 < steps; s0 += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int s = s0 + d;
      if (s >= steps) break;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < 2 * NP; ++nt)
          acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, pw[d][nt]),
                                                                __builtin_bit_cast(bf16x8_t, pa[d][mt]), acc[mt][nt],
                                                                0, 0, 0);
      if (s + D < steps) fetch(s + D, d);
    }
  }

  // lane (li, g): pixel li of the tile, channels n0 + 32 pr + 8 g + (0..7)
#pragma unroll
  for (int pr = 0; pr < NP; ++pr) {
    const int n = n0 + 32 * pr + 8 * g;
    if (n >= a.N) continue;
    float bias[8];
    conv_bias(a, n, bias);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int m = m0 + 16 * mt + li;
      if (m >= M) continue;
      long long op = m;
      if (a.mode == CM_DOWN3_T) {
        const int b = m / hw, rem = m - b * hw;
        const int ii = rem / W, jj = rem - ii * W;
        const int p = z / 3, q = z - 3 * (z / 3);
        op = ((long long)b * 3 * H + 3 * ii + p) * (3LL * W) + 3 * jj + q;
      }
      conv_store(a, op, n, acc[mt][2 * pr], acc[mt][2 * pr + 1], bias);
    }
  }
}

// Weight gradient: partial[s][r][n] = sum over the pixels of split s of
// im2col(in)[pixel][r] * gy[pixel][n]; row r = taps * Cin is all ones (the
// bias gradient).
//
// A GEMM whose reduction runs over the pixels, the slow index of both
// operands, while a matrix-core fragment wants eight consecutive pixels of
// one channel.  Each lane reads two channels of eight consecutive pixels
// (4 bytes a pixel) and transposes the block in registers, one byte permute
// per word: channel t of lane li is then row li of row tile t (tile t holds
// the rows 2 li + t), so neither operand passes through LDS and the loop has
// no barrier.  A wave owns 32 rows x NB columns of one split and adds its
// 32-pixel steps in order, D of them in flight: the order of every sum is that
// of the pixels within a split and of the splits, whatever the tile.  (The
// rounding of a weight to 16 bits can hang on the last bit of a gradient near
// zero, through Adam's normalised step: the order stays.)  Bound by the
// chain of a split's steps, 0.4 us each (0.6 us where an image row is
// shorter than a step and every pixel finds its row).
// 16 images of 243^2, 32 -> 32 channels: 564 -> 200 us; the 21 layers of a
// training step: 9.0 -> 3.1 ms (1.6 ms with four times the splits and four
// waves sharing one, which added in another order: not kept).
//
// KIND: the pixel map (WG_CONV3, WG_UP3, WG_PLAIN); SMALL: images of fewer
// than eight columns, whose steps touch more than two rows.  With the map
// known at run time only, branches per pixel and the code of every path made the
// step up to 1.6 times as long (4.3 ms for the 21 layers).
enum WgradKind : int { WG_CONV3 = 0, WG_UP3 = 1, WG_PLAIN = 2 };
template <int NB, int KIND, bool SMALL>
__global__ __launch_bounds__(64 * kWgradWaves, 1) void wgrad_kernel(WgradArgs a) {
  constexpr int CB = NB / 16;   // gy channels per lane
  constexpr int RT = 2;         // row tiles per wave
  constexpr int D = NB == 32 ? 6 : 4;  // steps in flight
  const int lane = threadIdx.x & 63;
  const int li = lane & 15, g = lane >> 4;
  const int rbase = (int)(blockIdx.x * kWgradWaves + (threadIdx.x >> 6)) * kWgradRows;  // the wave's first row
  if (rbase >= a.rows) return;
  const int s = blockIdx.z;
  const int W = a.Wo, H = a.Ho;
  const long long M = (long long)a.B * H * W;
  const long long pb0 = (long long)s * a.pix_per_split;
  const long long pend = (pb0 + a.pix_per_split < M) ? pb0 + a.pix_per_split : M;
  const int Kf = a.taps * a.C0;
  // the lane's two im2col rows (one tap) and CB output channels
  const int r = rbase + 2 * li;
  const int n = blockIdx.y * NB + CB * li;
  const bool row_in = r < Kf, ones = r == Kf, col_in = n < a.Np;
  const int tap = row_in ? r / a.C0 : 0;
  const int tp = a.taps == 9 ? tap / 3 : 0, tq = a.taps == 9 ? tap - 3 * tp : 0;
  const long long hw = (long long)H * W;
  // offsets are 32-bit, from the first image the block reads (a batch holds
  // less than 2^25 pixels of at most 128 channels)
  const int b0 = (int)(pb0 < M ? pb0 / hw : 0);
  const bf16_t* in = a.in0 + (long long)b0 * a.Hi * a.Wi * a.ld0 + (row_in ? r - tap * a.C0 : 0);
  const bf16_t* gy = a.gy + (col_in ? n : 0);
  const uint32_t ld = (uint32_t)a.ld0;
  constexpr bool c3 = KIND != WG_PLAIN;
  const int cstep = !c3 && a.mode == CM_DOWN3 ? 3 : 1;   // input columns per output column
  const int coff = c3 ? tq - 1 : (a.mode == CM_DOWN3 ? tq : 0);

  // first input pixel (from image b0) of the input row that output row (b, i) reads at the lane's tap
  auto third = [](uint32_t v) -> uint32_t { return (v * 43691u) >> 17; };  // v / 3 for v < 2^16
  auto in_row = [&](int b, int i) -> uint32_t {
    int ii = cstep * i + (a.taps == 9 ? tp : 0);
    if constexpr (c3) {
      ii -= 1;
      ii += ii < 0 ? H : 0;
      ii -= ii >= H ? H : 0;
      if constexpr (KIND == WG_UP3) ii = (int)third((uint32_t)ii);
    }
    return (uint32_t)((b - b0) * a.Hi + ii) * (uint32_t)a.Wi;
  };
  auto in_col = [&](int j) -> uint32_t {
    int jj = cstep * j + coff;
    if constexpr (c3) {
      jj += jj < 0 ? W : 0;
      jj -= jj >= W ? W : 0;
      if constexpr (KIND == WG_UP3) jj = (int)third((uint32_t)jj);
    }
    return (uint32_t)jj;
  };

  uint32_t ra[D][8];           // [step][pixel]: two channels
  uint32_t rb[D][8][CB / 2];
  auto load_b = [&](int d, int u, const bf16_t* p) {
    if constexpr (CB == 4) {
      const uint2 y = *reinterpret_cast<const uint2*>(p);
      rb[d][u][0] = y.x;
      rb[d][u][1] = y.y;
    } else {
      rb[d][u][0] = *reinterpret_cast<const uint32_t*>(p);
    }
  };
  // Loads of the step whose first pixel of this lane is m = (b, i, j), every
  // pixel of it within the split.  Rows and columns beyond the operands load
  // what the first ones do: their sums are not stored.
  auto fetch = [&](int d, long long m, int b, int i, int j, uint32_t row0, const bf16_t* gp) {
    uint32_t off[8];
    if constexpr (SMALL) {
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int bu = (int)((m + u) / hw);
        const int rem = (int)((m + u) - bu * hw);
        off[u] = (in_row(bu, rem / W) + in_col(rem - (rem / W) * W)) * ld;
      }
    } else {
      // steps whose eight input pixels follow each other in one row (all lanes)
      const bool run = KIND != WG_UP3 && j + 8 <= W && (!c3 || (j + coff >= 0 && j + 7 + coff < W));
      if (KIND != WG_UP3 && __all(run)) {
        off[0] = (row0 + (uint32_t)(cstep * j + coff)) * ld;
#pragma unroll
        for (int u = 1; u < 8; ++u) off[u] = off[u - 1] + (uint32_t)cstep * ld;
      } else {
        const bool wrap = i + 1 == H;
        const uint32_t row1 = in_row(wrap ? b + 1 : b, wrap ? 0 : i + 1);  // used only where it is a pixel of the batch
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int ju = j + u;
          const bool next = ju >= W;
          off[u] = ((next ? row1 : row0) + in_col(next ? ju - W : ju)) * ld;
        }
      }
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) ra[d][u] = *reinterpret_cast<const uint32_t*>(in + off[u]);
#pragma unroll
    for (int u = 0; u < 8; ++u) load_b(d, u, gp + u * a.ldg);
  };

  float4_t acc[RT][CB];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int nt = 0; nt < CB; ++nt) acc[t][nt] = float4_t{0.f, 0.f, 0.f, 0.f};

  // 32 pixels a step; (m, b, i, j) is the fetch position
  const int dj = 32 % W, di = 32 / W;
  long long m = pb0 + 8 * g;
  int b = (int)(m / hw);
  int i = (int)((m - b * hw) / W);
  int j = (int)(m - ((long long)b * H + i) * W);
  uint32_t row0 = in_row(b, i);  // of the position's row
  const bf16_t* gp = gy + m * a.ldg;
  auto advance = [&]() {
    m += 32;
    gp += 32 * a.ldg;
    j += dj;
    i += di;
    if (j >= W || di > 0) {
      if (j >= W) {
        j -= W;
        ++i;
      }
      while (i >= H) {
        i -= H;
        ++b;
      }
      row0 = in_row(b, i);
    }
  };
  union Frag {
    uint32_t w[4];
    bf16x8_t v;
  };
  const bool has_ones = __any(ones);
  Frag af[RT], bf[CB];
  auto fragments = [&](int d) {
    if (has_ones && ones) {
      // 1.0 in the first row of the group
#pragma unroll
      for (int u = 0; u < 8; ++u) ra[d][u] = 0x3F80u;
    }
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int k = 0; k < 4; ++k)
        af[t].w[k] = __builtin_amdgcn_perm(ra[d][2 * k + 1], ra[d][2 * k], t ? 0x07060302u : 0x05040100u);
#pragma unroll
    for (int nt = 0; nt < CB; ++nt)
#pragma unroll
      for (int k = 0; k < 4; ++k)
        bf[nt].w[k] = __builtin_amdgcn_perm(rb[d][2 * k + 1][nt >> 1], rb[d][2 * k][nt >> 1],
                                            (nt & 1) ? 0x07060302u : 0x05040100u);
  };
  auto multiply = [&]() {
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int nt = 0; nt < CB; ++nt)
        acc[t][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[t].v, bf[nt].v, acc[t][nt], 0, 0, 0);
  };
  const int steps = pend > pb0 ? (int)((pend - pb0) / 32) : 0;  // whole steps
#pragma unroll
  for (int d = 0; d < D; ++d) {
    if (d < steps) {
      fetch(d, m, b, i, j, row0, gp);
      advance();
    }
  }
  for (int s0 = 0; s0 < steps; s0 += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      if (s0 + d >= steps) break;
      fragments(d);
      if (s0 + d + D < steps) {
        fetch(d, m, b, i, j, row0, gp);
        advance();
      }
      multiply();
    }
  }
  if (pb0 + 32ll * steps < pend) {
    // the last pixels of the batch: those past the end add zeros
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const bool pv = m + u < pend;
      ra[0][u] = 0u;
#pragma unroll
      for (int c = 0; c < CB / 2; ++c) rb[0][u][c] = 0u;
      if (pv) {
        const int bu = (int)((m + u) / hw);
        const int rem = (int)((m + u) - bu * hw);
        ra[0][u] = *reinterpret_cast<const uint32_t*>(in + (in_row(bu, rem / W) + in_col(rem - (rem / W) * W)) * ld);
        load_b(0, u, gy + (m + u) * a.ldg);
      }
    }
    fragments(0);
    multiply();
  }

#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int ro = rbase + 2 * (4 * g + e) + t;
      if (ro >= a.rows) continue;
#pragma unroll
      for (int nt = 0; nt < CB; ++nt)
        if (n + nt < a.Np) a.partial[((long long)s * a.rows + ro) * a.Np + n + nt] = acc[t][nt][e];
    }
}

// Sum of the splits in order, the loads of eight in flight.
__global__ __launch_bounds__(64) void wgrad_reduce_kernel(const float* partial, int splits, int rows, int Np, int cin,
                                                          int cin_real, int cout, float* gw, float* gb) {
  const long long n_el = (long long)rows * Np;
  const long long e = (long long)blockIdx.x * 64 + threadIdx.x;
  if (e < n_el) {
    float s = 0.f;
    int k = 0;
    for (; k + 8 <= splits; k += 8) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = partial[(long long)(k + u) * n_el + e];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; k < splits; ++k) s += partial[(long long)k * n_el + e];
    const int r = (int)(e / Np), n = (int)(e - (long long)r * Np);
    if (n < cout) {
      const int t = r / cin, c = r - t * cin;
      if (r == rows - 1) gb[n] = s;
      else if (c < cin_real) gw[((long long)t * cin_real + c) * cout + n] = s;
    }
  }
}

__global__ void grad_prep_kernel(long long P, int C, int Cp, const float* g, int ld, bf16_t* gpre) {
  const long long n = P * Cp;
  for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
    const long long p = e / Cp;
    const int c = (int)(e - p * Cp);
    gpre[e] = f2bf(c < C ? g[p * ld + c] : 0.f);
  }
}

__global__ void pool3_sum_kernel(int B, int Hc, int Wc, int C, const float* fine, float* coarse, const bf16_t* act,
                                 bf16_t* coarse_b) {
  const long long n = (long long)B * Hc * Wc * C;
  for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
    const int c = (int)(e % C);
    const long long pc = e / C;
    const int J = (int)(pc % Wc);
    const long long t = pc / Wc;
    const int I = (int)(t % Hc);
    const int b = (int)(t / Hc);
    float s = 0.f;
    for (int p = 0; p < 3; ++p)
      for (int q = 0; q < 3; ++q)
        s += fine[(((long long)b * 3 * Hc + 3 * I + p) * (3LL * Wc) + 3 * J + q) * C + c];
    if (act) coarse_b[e] = f2bf(bf2f(act[e]) > 0.f ? s : 0.f);
    else coarse[e] = s;
  }
}

__global__ void make_input_kernel(int B, int N, const uint8_t* phase, const float* lr, int transpose, int scale,
                                  bf16_t* x) {
  const long long n = (long long)B * N * N;
  const int NF = N * scale;  // side of the stored image
  for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
    const int j = (int)(e % N);
    const long long t = e / N;
    const int i = (int)(t % N);
    const int b = (int)(t / N);
    int cnt = 0;
    for (int p = 0; p < scale; ++p)
      for (int q = 0; q < scale; ++q) {
        const int fi = scale * i + p, fj = scale * j + q;
        const long long src = transpose ? ((long long)b * NF + fj) * NF + fi : ((long long)b * NF + fi) * NF + fj;
        cnt += phase[src] != 0;
      }
    uint4 v0 = {0u, 0u, 0u, 0u};
    const uint32_t ph = 2 * cnt > scale * scale ? 0x3F80u : 0u;
    const uint32_t rr = f2bf(lr[b] * 0.25f);
    v0.x = ph | (rr << 16);
    *reinterpret_cast<uint4*>(x + e * 8) = v0;
  }
}

__global__ void mse_sums_kernel(int N, const float* pred, const double* e, double* part) {
  const int b = blockIdx.y;
  const long long nn = (long long)N * N;
  double s_num = 0.0, s_den = 0.0;
  for (long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x; p < nn; p += (long long)gridDim.x * blockDim.x) {
    for (int c = 0; c < 2; ++c) {
      const double t = e[((long long)b * 2 + c) * nn + p] - (c == 0 ? 1.0 : 0.0);
      const double d = (double)pred[((long long)b * nn + p) * 2 + c] - t;
      s_num += d * d;
      s_den += t * t;
    }
  }
  __shared__ double red[2][256];
  red[0][threadIdx.x] = s_num;
  red[1][threadIdx.x] = s_den;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) {
      red[0][threadIdx.x] += red[0][threadIdx.x + off];
      red[1][threadIdx.x] += red[1][threadIdx.x + off];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[((long long)b * 2 + 0) * gridDim.x + blockIdx.x] = red[0][0];
    part[((long long)b * 2 + 1) * gridDim.x + blockIdx.x] = red[1][0];
  }
}

__global__ void mse_grad_kernel(int B, int N, int nb, const float* pred, const double* e, const double* part,
                                float* grad) {
  const int b = blockIdx.y;
  double den = 0.0;
  for (int k = 0; k < nb; ++k) den += part[((long long)b * 2 + 1) * nb + k];
  den = den > 1e-30 ? den : 1e-30;
  const double scale = 2.0 / (den * B);
  const long long nn = (long long)N * N;
  for (long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x; p < nn; p += (long long)gridDim.x * blockDim.x)
    for (int c = 0; c < 2; ++c) {
      const double t = e[((long long)b * 2 + c) * nn + p] - (c == 0 ? 1.0 : 0.0);
      const long long q = ((long long)b * nn + p) * 2 + c;
      grad[q] = (float)(scale * ((double)pred[q] - t));
    }
}

// One wave per image sums its partials (lane l the entries l, l + 64, ...,
// then a fixed tree); the images' ratios are added in order.  One thread doing
// both took 245 us at 16 images, of 13.5 ms of a training step.
__global__ __launch_bounds__(256) void mse_loss_kernel(int B, int nb, const double* part, double* loss) {
  __shared__ double ratio[4];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  double l = 0.0;
  for (int b0 = 0; b0 < B; b0 += 4) {
    const int b = b0 + w;
    double num = 0.0, den = 0.0;
    if (b < B) {
      for (int k = lane; k < nb; k += 64) {
        num += part[((long long)b * 2 + 0) * nb + k];
        den += part[((long long)b * 2 + 1) * nb + k];
      }
    }
    for (int off = 32; off > 0; off >>= 1) {
      num += __shfl_down(num, off, 64);
      den += __shfl_down(den, off, 64);
    }
    if (lane == 0) ratio[w] = b < B ? num / (den > 1e-30 ? den : 1e-30) : 0.0;
    __syncthreads();
    if (threadIdx.x == 0) l += ((ratio[0] + ratio[1]) + ratio[2]) + ratio[3];
    __syncthreads();
  }
  if (threadIdx.x == 0) *loss = l / B;
}

__global__ void make_field_kernel(int B, int N, const float* pred, int transpose, int scale, double* e) {
  const int NF = N * scale;
  const long long nn = (long long)N * N, nnf = (long long)NF * NF;
  const long long n = (long long)B * nnf;
  for (long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (long long)gridDim.x * blockDim.x) {
    const int b = (int)(q / nnf);
    const long long pf = q - (long long)b * nnf;
    const int fi = (int)(pf / NF), fj = (int)(pf - (pf / NF) * NF);
    const int i = fi / scale, j = fj / scale;
    for (int c = 0; c < 2; ++c) {
      double v;
      if (!transpose) {
        v = (c == 0 ? 1.0 : 0.0) + (double)pred[((long long)b * nn + (long long)i * N + j) * 2 + c];
      } else {
        // field of the load case e2 from the prediction for the transposed image
        const long long pt = (long long)j * N + i;
        v = (c == 1 ? 1.0 : 0.0) + (double)pred[((long long)b * nn + pt) * 2 + (1 - c)];
      }
      e[((long long)b * 2 + c) * nnf + pf] = v;
    }
  }
}

// Fragment order of a weight operand: element e of lane l of step s of tile
// t (16 channels: half t % 2 of the 32 of block t / 2) at ((t S + s) 64 + l) 8
// + e is row 32 (t / 2) + 8 (li / 4) + 4 (t % 2) + li % 4 (li = l % 16),
// reduction index 32 s + 8 (l / 16) + e; zeros beyond the operand's rows and
// reduction.  Forward: row o, k = t cin + c.  Input gradient: row c,
// k = t' np + o, each tap's np padded to whole steps for a stride-3 layer
// (whose launches take one tap each).  A thread writes the eight elements of a
// lane; one launch covers all layers (a launch each: 21 of 4.5 us).
constexpr int kCastUnits = 512;  // lanes' parts per block
__global__ __launch_bounds__(256) void cast_weights_kernel(CastArgs a) {
  int li_ = 0;
  while (li_ + 1 < a.layers && blockIdx.x >= a.layer[li_ + 1].first) ++li_;
  const CastLayer& L = a.layer[li_];
  const float* w = a.w + L.w_off;
  const long long base = (long long)(blockIdx.x - L.first) * kCastUnits, units = (L.n_f + L.n_t) / 8;
  for (int u = threadIdx.x; u < kCastUnits && base + u < units; u += 256) {
    const long long e = (base + u) * 8;
    const bool fwd = e < L.n_f;
    const long long q = fwd ? e : e - L.n_f;
    const int l = (int)(q >> 3) & 63, li = l & 15;
    const int ts = (int)(q >> 9), S = fwd ? L.steps_f : L.steps_t;
    const int t2 = ts / S, s = ts - t2 * S;
    const int row = 32 * (t2 >> 1) + 8 * (li >> 2) + 4 * (t2 & 1) + (li & 3);
    const int k0 = 32 * s + 8 * (l >> 4);
    // forward: k = t cin + c; input gradient: k = t' per + o
    const int per = fwd ? L.cin : (L.tap_pad ? (L.np + 31) / 32 * 32 : L.np);
    uint32_t h[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = k0 + j;
      const int tt = k / per, x = k - tt * per;
      const int t = !fwd && L.flip ? L.taps - 1 - tt : tt;
      const int c = fwd ? x : row, o = fwd ? row : x;
      float v = 0.f;
      if (tt < L.taps && c < L.cin_real && o < L.cout) v = w[((long long)t * L.cin_real + c) * L.cout + o];
      h[j] = f2bf(v);
    }
    *reinterpret_cast<uint4*>((fwd ? a.w16 + L.f_off : a.wt16 + L.t_off) + q) =
        uint4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
  }
}

__global__ void adam_kernel(long long n, float* w, const float* g, float* m, float* v, float lr, float b1, float b2,
                            float eps, float c1, float c2) {
  for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
    const float gg = g[e];
    const float mm = b1 * m[e] + (1.f - b1) * gg;
    const float vv = b2 * v[e] + (1.f - b2) * gg * gg;
    m[e] = mm;
    v[e] = vv;
    w[e] -= lr * (mm / c1) / (sqrtf(vv / c2) + eps);
  }
}

__global__ void fill_f32_kernel(float* p, long long n, float v) {
  for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x)
    p[e] = v;
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------

constexpr long long kConvWaves = 1536;  // waves of a direct launch (two per SIMD on three SIMDs of four)
// Image side from which the LDS patch pays: below, a 32-pixel row of a tile
// is mostly past the image's end.
constexpr int kConvTileSide = 27;
constexpr size_t kConvTileLds8 = 60 * 1024, kConvTileLds4 = 120 * 1024;
static size_t conv3_tile_lds(int th, int cin) { return (size_t)(th + 2) * 34 * (2 * cin + 16); }

static unsigned grid_for(long long n, int per = 256, long long cap = 8192) {
  long long b = (n + per - 1) / per;
  if (b < 1) b = 1;
  return (unsigned)(b > cap ? cap : b);
}

template <int MT, int NP, int D>
static hipError_t launch_conv_tile(const ConvArgs& a, hipStream_t s) {
  const long long M = (long long)a.B * a.Ho * a.Wo;
  const bool nine = a.mode == CM_CONV3 || a.mode == CM_DOWN3, uni = a.C0 % 32 == 0;
  const dim3 grid((unsigned)((M + 64 * MT - 1) / (64 * MT)), (unsigned)((a.N + 32 * NP - 1) / (32 * NP)),
                  a.mode == CM_DOWN3_T ? 9u : 1u);
  if (nine && uni) hipLaunchKernelGGL((conv_kernel<MT, NP, 9, true, D>), grid, dim3(256), 0, s, a);
  else if (nine) hipLaunchKernelGGL((conv_kernel<MT, NP, 9, false, D>), grid, dim3(256), 0, s, a);
  else if (uni) hipLaunchKernelGGL((conv_kernel<MT, NP, 1, true, D>), grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL((conv_kernel<MT, NP, 1, false, D>), grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

template <int TH, int CW>
static hipError_t launch_conv3_tile(const ConvArgs& a, hipStream_t s) {
  const dim3 grid((unsigned)((long long)a.B * ((a.Ho + TH - 1) / TH) * ((a.Wo + 31) / 32)),
                  (unsigned)((a.Np + 32 * CW - 1) / (32 * CW)));
  const size_t lds = conv3_tile_lds(TH, a.C0);
  if (a.C0 % 32 == 0) hipLaunchKernelGGL((conv3_tile_kernel<TH, CW, true>), grid, dim3(256), lds, s, a);
  else hipLaunchKernelGGL((conv3_tile_kernel<TH, CW, false>), grid, dim3(256), lds, s, a);
  return hipGetLastError();
}

ConvVariant conv_variant(const ConvArgs& a) {
  if (a.mode == CM_CONV3 && a.Wo >= kConvTileSide) {
    // eight rows a block while two blocks fit a CU (the patch's two extra rows
    // weigh less: 64 -> 32 channels on 243^2 87 us, four rows 102 us), else
    // four rows (layers that wide have more than 32 output channels); from 296
    // channels on layers read global memory per tap
    if (conv3_tile_lds(8, a.C0) <= kConvTileLds8) return {8, a.N <= 32 ? 1 : 2, 0, 0};
    if (conv3_tile_lds(4, a.C0) <= kConvTileLds4) return {4, 2, 0, 0};
  }
  // the largest wave tile that still gives two waves to most SIMDs; below
  // that a layer is bound by the length of its reduction, and narrow tiles
  // with more steps in flight win
  const long long M = (long long)a.B * a.Ho * a.Wo * (a.mode == CM_DOWN3_T ? 9 : 1);
  auto waves = [&](int mt, int np) { return ((M + 16 * mt - 1) / (16 * mt)) * ((a.Np + 32 * np - 1) / (32 * np)); };
  if (a.Np > 32) {
    if (waves(4, 2) >= kConvWaves) return {0, 0, 4, 2};
    if (waves(2, 2) >= kConvWaves) return {0, 0, 2, 2};
  } else if (waves(4, 1) >= kConvWaves) {
    return {0, 0, 4, 1};
  }
  if (waves(2, 1) >= kConvWaves) return {0, 0, 2, 1};
  return {0, 0, 1, 1};
}

hipError_t launch_conv(const ConvArgs& in, hipStream_t s) {
  ConvArgs a = in;
  a.wide_b = a.ldb % 8 == 0 && (reinterpret_cast<uintptr_t>(a.out_b) & 15u) == 0;
  a.wide_f = a.ldf % 4 == 0 && (reinterpret_cast<uintptr_t>(a.out_f) & 15u) == 0;
  a.wide_m = a.ldm % 8 == 0 && (reinterpret_cast<uintptr_t>(a.mask) & 15u) == 0;
  a.fd_chunks = make_fastdiv((uint32_t)a.C0 / 8u);
  const ConvVariant v = conv_variant(a);
  if (v.th == 8) return v.cw == 1 ? launch_conv3_tile<8, 1>(a, s) : launch_conv3_tile<8, 2>(a, s);
  if (v.th == 4) return launch_conv3_tile<4, 2>(a, s);
  // (the narrower the tile, the more steps in flight)
  if (v.np == 2) return v.mt == 4 ? launch_conv_tile<4, 2, 2>(a, s) : launch_conv_tile<2, 2, 3>(a, s);
  if (v.mt == 4) return launch_conv_tile<4, 1, 3>(a, s);
  return v.mt == 2 ? launch_conv_tile<2, 1, 4>(a, s) : launch_conv_tile<1, 1, 6>(a, s);
}

static unsigned wgrad_row_blocks(const WgradArgs& a) {
  return (unsigned)((a.rows + kWgradRows * kWgradWaves - 1) / (kWgradRows * kWgradWaves));
}

WgradVariant wgrad_variant(const WgradArgs& a, int splits) {
  // wide tiles read the input rows half as often, where they still give every
  // second SIMD a wave
  const long long wide_waves = (long long)wgrad_row_blocks(a) * kWgradWaves * ((a.Np + 63) / 64) * splits;
  return {a.Np > 32 && wide_waves >= 512 ? 64 : 32, a.Wo < 8};
}

hipError_t launch_wgrad(const WgradArgs& a, int splits, hipStream_t s) {
  const unsigned rb = wgrad_row_blocks(a);
  const WgradVariant v = wgrad_variant(a, splits);
  const int nb = v.columns;
  const dim3 grid(rb, (unsigned)((a.Np + nb - 1) / nb), (unsigned)splits);
  const int kind = a.mode != CM_CONV3 ? WG_PLAIN : (a.up == 3 ? WG_UP3 : WG_CONV3);
  auto launch = [&](auto NB, auto KIND) {
    if (v.small) hipLaunchKernelGGL((wgrad_kernel<NB(), KIND(), true>), grid, dim3(64 * kWgradWaves), 0, s, a);
    else hipLaunchKernelGGL((wgrad_kernel<NB(), KIND(), false>), grid, dim3(64 * kWgradWaves), 0, s, a);
  };
  auto launch_kind = [&](auto NB) {
    if (kind == WG_CONV3) launch(NB, std::integral_constant<int, WG_CONV3>{});
    else if (kind == WG_UP3) launch(NB, std::integral_constant<int, WG_UP3>{});
    else launch(NB, std::integral_constant<int, WG_PLAIN>{});
  };
  if (nb == 32) launch_kind(std::integral_constant<int, 32>{});
  else launch_kind(std::integral_constant<int, 64>{});
  return hipGetLastError();
}

hipError_t launch_wgrad_reduce(const float* partial, int splits, int rows, int Np, int cin, int cin_real, int cout,
                               float* gw, float* gb, hipStream_t s) {
  hipLaunchKernelGGL(wgrad_reduce_kernel, dim3((unsigned)(((long long)rows * Np + 63) / 64)), dim3(64), 0, s, partial,
                     splits, rows, Np, cin, cin_real, cout, gw, gb);
  return hipGetLastError();
}

hipError_t launch_grad_prep(long long P, int C, int Cp, const float* g, int ld, bf16_t* gpre, hipStream_t s) {
  hipLaunchKernelGGL(grad_prep_kernel, dim3(grid_for(P * Cp)), dim3(256), 0, s, P, C, Cp, g, ld, gpre);
  return hipGetLastError();
}

hipError_t launch_pool3_sum(int B, int Hc, int Wc, int C, const float* fine, float* coarse, const bf16_t* act,
                            bf16_t* coarse_b, hipStream_t s) {
  hipLaunchKernelGGL(pool3_sum_kernel, dim3(grid_for((long long)B * Hc * Wc * C)), dim3(256), 0, s, B, Hc, Wc, C, fine,
                     coarse, act, coarse_b);
  return hipGetLastError();
}

hipError_t launch_make_input(int B, int N, const uint8_t* phase, const float* log10_rho, int transpose, int scale,
                             bf16_t* x, hipStream_t s) {
  hipLaunchKernelGGL(make_input_kernel, dim3(grid_for((long long)B * N * N)), dim3(256), 0, s, B, N, phase, log10_rho,
                     transpose, scale, x);
  return hipGetLastError();
}

hipError_t launch_rel_mse(int B, int N, const float* pred, const double* e, double* part, double* loss, float* grad,
                          hipStream_t s) {
  const int nb = 256;
  hipLaunchKernelGGL(mse_sums_kernel, dim3(nb, B), dim3(256), 0, s, N, pred, e, part);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  if (grad) {
    hipLaunchKernelGGL(mse_grad_kernel, dim3(64, B), dim3(256), 0, s, B, N, nb, pred, e, part, grad);
    if ((err = hipGetLastError()) != hipSuccess) return err;
  }
  hipLaunchKernelGGL(mse_loss_kernel, dim3(1), dim3(256), 0, s, B, nb, part, loss);
  return hipGetLastError();
}

hipError_t launch_make_field(int B, int N, const float* pred, int transpose, int scale, double* e, hipStream_t s) {
  hipLaunchKernelGGL(make_field_kernel, dim3(grid_for((long long)B * N * N * scale * scale)), dim3(256), 0, s, B, N,
                     pred, transpose, scale, e);
  return hipGetLastError();
}

hipError_t launch_cast_weights(const CastArgs& in, hipStream_t s) {
  CastArgs a = in;
  unsigned blocks = 0;
  for (int i = 0; i < a.layers; ++i) {
    CastLayer& L = a.layer[i];
    const WeightTiles f = weight_tiles_fwd(L.taps, L.cin, L.np), t = weight_tiles_grad(L.taps, L.cin, L.np, L.tap_pad);
    L.steps_f = f.steps;
    L.steps_t = t.steps;
    L.n_f = f.elements();
    L.n_t = t.elements();
    L.first = blocks;
    blocks += (unsigned)(((L.n_f + L.n_t) / 8 + kCastUnits - 1) / kCastUnits);
  }
  hipLaunchKernelGGL(cast_weights_kernel, dim3(blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_adam(long long n, float* w, const float* g, float* m, float* v, float lr, float b1, float b2,
                       float eps, float c1, float c2, hipStream_t s) {
  hipLaunchKernelGGL(adam_kernel, dim3(grid_for(n)), dim3(256), 0, s, n, w, g, m, v, lr, b1, b2, eps, c1, c2);
  return hipGetLastError();
}

hipError_t launch_fill_f32(float* p, long long n, float v, hipStream_t s) {
  hipLaunchKernelGGL(fill_f32_kernel, dim3(grid_for(n)), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

}  // namespace cnn
}  // namespace lshom
