// Passes of 2-D grids along axes of 81, 243 or 729 nodes.
//
// Same algebra, reads and writes as the block passes of passes.hip (spectral
// arrays stored [k1][k0], no padding), with the transforms of wave_fft.hpp:
// lengths and radices known at compile time, nine points per lane, whole
// sequences per wave (81, 243; no block barrier in a transform) or three
// sequences per block (729).  The first stage of a column transform reads its
// points from global memory and the last stage's outputs go from registers to
// global memory, the projection or the polarisation, so that a column pass
// exchanges through LDS only between stages.
//
// Bound by memory for batches (the row pass reads and writes segments of two
// rows per pair of a wave) and by latency for one image (a 729^2 launch has
// about one wave per SIMD).  Measured in us per pass (axis-0 inverse / row /
// axis-0 forward), block passes -> these: one 729^2 image FP64 19.6 / 25.4 /
// 18.5 -> 12.6 / 13.5 / 11.3; ten of them in a batch 79 / 122 / 79 -> 48 / 70 /
// 42; 32 images of 243^2 FP32 15.2 / 23.9 / 13.9 -> 10.1 / 11.9 / 9.3.
#include <hip/hip_runtime.h>

#include "kernels.hpp"
#include "reduce.hpp"
#include "wave_fft.hpp"

namespace lshom {

namespace {

// A block: two waves of whole sequences, or (729) four waves with three
// sequences of 81 lanes.
template <int N>
struct W2 {
  static constexpr int LPS = N / 9;
  static constexpr bool kWide = N > 243;
  static constexpr int NT = kWide ? 256 : 128;
  static constexpr int SPG = kWide ? NT / LPS : 64 / LPS;          // sequences per exchange group (wave or block)
  static constexpr int SPB = kWide ? SPG : (NT / 64) * SPG;        // per block
  static constexpr int GT = kWide ? NT : 64;                       // threads of a group
};

// Sequence of this thread in its block, its lane in the sequence, and
// whether it owns points.
template <int N>
struct W2Lane {
  int group, in_group, j, seq;
  bool act;
  __device__ __forceinline__ W2Lane() {
    using G = W2<N>;
    const int t = G::kWide ? (int)threadIdx.x : (int)(threadIdx.x & 63);
    group = G::kWide ? 0 : (int)(threadIdx.x >> 6);
    in_group = t;
    const int s = t / G::LPS;
    j = t - s * G::LPS;
    act = s < G::SPG;
    seq = group * G::SPG + (act ? s : 0);
  }
};

__device__ __forceinline__ int w2_freq(int m, int n) { return (m <= n / 2) ? m : m - n; }

template <typename T, int N, int NT>
struct W2Twiddles {
  static constexpr int PER = (N + NT - 1) / NT;
  cx<T> v[PER];
  __device__ __forceinline__ void fetch(const cx<T>* __restrict__ src) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int i = (int)threadIdx.x + u * NT;
      v[u] = cx<T>{T(0), T(0)};
      if (i < N) v[u] = src[i];
    }
  }
  __device__ __forceinline__ void put(cx<T>* tw) const {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int i = (int)threadIdx.x + u * NT;
      if (i < N) tw[i] = v[u];
    }
  }
};

// 1 / |xi| at (axis-0 index l, last-axis column c); 0 where the Green operator
// vanishes (k = 0; the Nyquist column of an even last axis; axis 0 is odd).
// k2: |xi|^2 there.
template <typename T, int N>
__device__ __forceinline__ double w2_inv_norm(const ColArgs<T>& a, int l, int c, double* x0, double* k2_out) {
  const int n1 = a.nd[1];
  *x0 = (double)w2_freq(l, N) * a.cinv[0];
  const double x1 = (double)c * a.cinv[1];
  const double k2 = *x0 * *x0 + x1 * x1;
  *k2_out = k2;
  const bool nz = k2 > 0.0 && !((n1 & 1) == 0 && c == n1 / 2);
  return nz ? 1.0 / sqrt(k2) : 0.0;
}

// Two blocks or more read the halves of one cache line: each XCD takes one
// contiguous run of (problem, block) pairs.
__device__ __forceinline__ void w2_xcd_order(unsigned& bx, unsigned& by) {
  const unsigned gx = gridDim.x, total = gx * gridDim.y;
  const unsigned lin = blockIdx.y * gx + blockIdx.x;
  const unsigned xcd = lin & 7u, slot = lin >> 3;
  const unsigned q = total >> 3, rem = total & 7u;
  const unsigned lin2 = xcd * q + (xcd < rem ? xcd : rem) + slot;
  by = lin2 / gx;
  bx = lin2 - by * gx;
}

}  // namespace

int w2_seqs(int n) {
  switch (n) {
    case 729: return W2<729>::SPB;
    case 243: return W2<243>::SPB;
    default: return W2<81>::SPB;
  }
}

// ---------------------------------------------------------------------------
// Axis-0 inverse: c (or the CG direction step p = r + beta p) -> i khat_a c ->
// inverse FFT -> comp[a]
// ---------------------------------------------------------------------------
template <typename T, int N>
__global__ __launch_bounds__(W2<N>::NT) void w2_inv_kernel(ColArgs<T> a) {
  using G = W2<N>;
  constexpr int NT = G::NT, LPS = G::LPS;
  const int pb = batch_prob(a.bt);
  DevState* st = a.st + pb;
  Partials parts = a.parts;
  parts.base += (long long)pb * a.bt.pstride;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* tw = reinterpret_cast<cx<T>*>(smem_raw);
  const W2Lane<N> ln;
  cx<T>* buf = tw + N + ln.seq * N;
  const int c = (int)blockIdx.x * G::SPB + ln.seq;
  const bool ok = ln.act && c < a.inner;
  const long long col = (long long)pb * a.bt.vstride + (long long)(ok ? c : 0) * N + ln.j;
  // the column and the twiddles are requested before the sums are waited for
  cx<T> cv[9], pv[9];
  const cx<T>* src = a.cg_step ? a.r_in : a.c_in;
#pragma unroll
  for (int r = 0; r < 9; ++r) {
    cv[r] = cx<T>{T(0), T(0)};
    pv[r] = cx<T>{T(0), T(0)};
    if (ok) {
      cv[r] = src[col + LPS * r];
      if (a.cg_step) pv[r] = a.p_io[col + LPS * r];
    }
  }
  W2Twiddles<T, N, NT> twv;
  twv.fetch(a.tw);
  if (a.cg_step) {
    double beta = 0.0;
    if (!cg_direction<NT>(st, parts, a.inv_n, &beta, a.gate, a.eq, blockIdx.x == 0)) return;
    const T tb = (T)beta;
    if (ok) {
#pragma unroll
      for (int r = 0; r < 9; ++r) {
        cv[r] = cx<T>{cv[r].re + tb * pv[r].re, cv[r].im + tb * pv[r].im};
        a.p_io[col + LPS * r] = cv[r];
      }
    }
  } else if (a.basic_step) {
    if (!basic_direction<NT>(st, parts, a.inv_n, a.gate, blockIdx.x == 0)) return;
  } else if (gated_out_stable(st, a.gate)) {
    return;
  }
  twv.put(tw);
  double inv[9];
#pragma unroll
  for (int r = 0; r < 9; ++r) {
    double x0, k2;
    inv[r] = w2_inv_norm<T, N>(a, ln.j + LPS * r, c, &x0, &k2);
  }
  const double x1 = (double)c * a.cinv[1];
  __syncthreads();
#pragma unroll 1
  for (int al = 0; al < 2; ++al) {
    cx<T> v[9], out[9];
#pragma unroll
    for (int r = 0; r < 9; ++r) {
      const double xa = al == 0 ? (double)w2_freq(ln.j + LPS * r, N) * a.cinv[0] : x1;
      const T k = (T)(xa * inv[r]);
      v[r] = cx<T>{-k * cv[r].im, k * cv[r].re};  // i khat_a c
    }
    wave_fft_regs<T, N, +1>(v, buf, tw, ln.j, ln.act, out);
    if (ok) {
      cx<T>* dst = (al == 0 ? a.comp[0] : a.comp[1]) + col;
#pragma unroll
      for (int r = 0; r < 9; ++r) dst[LPS * r] = out[r];
    }
  }
}

// ---------------------------------------------------------------------------
// Axis-0 forward + projection: out = coef_base base + coef_s [1 / l0] s,
// s = -i khat . tau_hat, and the dot
// ---------------------------------------------------------------------------
template <typename T, int N>
__global__ __launch_bounds__(W2<N>::NT) void w2_fwd_kernel(ColArgs<T> a) {
  using G = W2<N>;
  constexpr int NT = G::NT, LPS = G::LPS;
  const int pb = batch_prob(a.bt);
  DevState* st = a.st + pb;
  const ProbEntry* pe = a.bt.tab ? a.bt.tab + pb : nullptr;
  Partials parts = a.parts;
  parts.base += (long long)pb * a.bt.pstride;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* tw = reinterpret_cast<cx<T>*>(smem_raw);
  const W2Lane<N> ln;
  cx<T>* buf = tw + N + ln.seq * N;
  const int c = (int)blockIdx.x * G::SPB + ln.seq;
  const bool ok = ln.act && c < a.inner;
  const long long col = (long long)pb * a.bt.vstride + (long long)(ok ? c : 0) * N + ln.j;
  cx<T> v[2][9];
#pragma unroll
  for (int al = 0; al < 2; ++al)
#pragma unroll
    for (int r = 0; r < 9; ++r) v[al][r] = ok ? a.comp[al][col + LPS * r] : cx<T>{T(0), T(0)};
  W2Twiddles<T, N, NT> twv;
  twv.fetch(a.tw);
  if (gated_out_stable(st, a.gate)) return;
  twv.put(tw);
  __syncthreads();
  const double x1 = (double)c * a.cinv[1];
  const bool origin = a.eq && ok && c == 0 && ln.j == 0;
  // k = 0: the cell sum of the transformed field (dL (E + u) or dL u)
  double* sums = a.dot == 1 ? st->taup : st->jx;
  cx<T> t[9], bv[9];
  wave_fft_regs<T, N, -1>(v[0], buf, tw, ln.j, ln.act, t);
  if (origin) sums[0] = (double)t[0].re;
  // base arrives during the second transform
#pragma unroll
  for (int r = 0; r < 9; ++r) bv[r] = (ok && a.base) ? a.base[col + LPS * r] : cx<T>{T(0), T(0)};
  double inv[9];
#pragma unroll
  for (int r = 0; r < 9; ++r) {
    double x0, k2;
    inv[r] = w2_inv_norm<T, N>(a, ln.j + LPS * r, c, &x0, &k2);
    const T k = (T)(x0 * inv[r]);
    t[r] = cx<T>{k * t[r].re, k * t[r].im};
  }
  {
    cx<T> z[9];
    wave_fft_regs<T, N, -1>(v[1], buf, tw, ln.j, ln.act, z);
    if (origin) {
      sums[1] = (double)z[0].re;
      sums[2] = 0.0;
    }
#pragma unroll
    for (int r = 0; r < 9; ++r) {
      const T k = (T)(x1 * inv[r]);
      t[r].re += k * z[r].re;
      t[r].im += k * z[r].im;
    }
  }
  const T cs = a.coef_s * (a.s_inv_l0 ? (T)(1.0 / (pe ? pe->l0 : a.l0)) : T(1));
  const int n1 = a.nd[1];
  const double w = c == 0 || ((n1 & 1) == 0 && c == n1 / 2) ? 1.0 : 2.0;
  double acc[2] = {0.0, 0.0};
  if (ok) {
#pragma unroll
    for (int r = 0; r < 9; ++r) {
      // s = -i khat . tau_hat
      cx<T> val = {cs * t[r].im, -cs * t[r].re};
      val.re += a.coef_base * bv[r].re;
      val.im += a.coef_base * bv[r].im;
      a.out[col + LPS * r] = val;
      if (a.dot == 1) {
        acc[0] += w * ((double)bv[r].re * (double)val.re + (double)bv[r].im * (double)val.im);
      } else if (a.dot) {
        // dot 2: |out|^2; dot 3: the step |out - base|^2 of the basic scheme
        const double dr = a.dot == 3 ? (double)val.re - (double)bv[r].re : (double)val.re;
        const double di = a.dot == 3 ? (double)val.im - (double)bv[r].im : (double)val.im;
        const double m2 = dr * dr + di * di;
        acc[0] += w * m2;
        if (a.eq) {
          const double x0 = (double)w2_freq(ln.j + LPS * r, N) * a.cinv[0];
          // (the weight of k = 0 and of the Nyquist column is immaterial: out is zero there)
          acc[1] += w * (x0 * x0 + x1 * x1) * m2;
        }
      }
    }
  }
  if (a.dot) {
    (void)block_sums_gated<NT, 2>(acc, 0);
    if (threadIdx.x == 0) {
      parts.region(a.dot_region)[blockIdx.x] = acc[0];
      if (a.eq && a.dot != 1) parts.region(a.eq_region)[blockIdx.x] = acc[1];
      if (a.dot_region == PART_RR0 && blockIdx.x == 0) st->nparts[0] = (int)gridDim.x;
      if (a.dot == 3 && blockIdx.x == 0) st->iter_a += 1;
      if (a.dot_region == PART_PQ && blockIdx.x == 0) st->nparts_pq = (int)gridDim.x;
    }
  }
}

// ---------------------------------------------------------------------------
// Row pass (modes of RowMode): rows 2 p, 2 p + 1 of one component in one
// complex sequence
// ---------------------------------------------------------------------------
template <typename T, int N, int MODE>
__global__ __launch_bounds__(W2<N>::NT) void w2_row_kernel(RowArgs<T> a) {
  using G = W2<N>;
  constexpr int NT = G::NT, LPS = G::LPS, H = (N + 1) / 2;
  constexpr int RB = 2 * G::SPB;                        // rows per block
  constexpr int TOT = G::SPG * H;                       // half-spectrum entries of a group, pair fastest
  constexpr int IT = (TOT + G::GT - 1) / G::GT;
  unsigned bx, by;
  w2_xcd_order(bx, by);
  const int pb = a.bt.live ? a.bt.live[by] : (int)by;
  DevState* st = a.st + pb;
  const ProbEntry* pe = a.bt.tab ? a.bt.tab + pb : nullptr;
  Partials parts = a.parts;
  parts.base += (long long)pb * a.bt.pstride;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* tw = reinterpret_cast<cx<T>*>(smem_raw);
  T* cond = reinterpret_cast<T*>(tw + N + G::SPB * N);
  uint8_t* phs = reinterpret_cast<uint8_t*>(cond) + ((size_t)a.n_phases * sizeof(T) + 15) / 16 * 16;
  // block = (row block, component), the component fastest
  const int al = (int)(bx & 1u);
  const int rb = (int)(bx >> 1);
  const int nrows = (int)a.nrows;
  const long long nvox = (long long)nrows * N;
  const int row0 = rb * RB;
  const W2Lane<N> ln;
  const int rowA = row0 + 2 * ln.seq;
  const bool hasA = ln.act && rowA < nrows, hasB = ln.act && rowA + 1 < nrows;
  cx<T>* buf = tw + N + ln.seq * N;
  cx<T>* gbuf = tw + N + ln.group * G::SPG * N;         // the group's sequences
  const int grow0 = row0 + 2 * ln.group * G::SPG;
  const long long vo = (long long)pb * a.bt.vstride;
  cx<T>* spec = (al == 0 ? a.spec[0] : a.spec[1]) + vo;

  cx<T> A[IT], B[IT];
  if constexpr (MODE != ROW_FWD) {
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int e = ln.in_group + G::GT * it;
      const int k = e / G::SPG, ra = grow0 + 2 * (e - k * G::SPG);
      const cx<T>* sp = spec + (long long)k * nrows + ra;
      A[it] = (e < TOT && ra < nrows) ? sp[0] : cx<T>{T(0), T(0)};
      B[it] = (e < TOT && ra + 1 < nrows) ? sp[1] : cx<T>{T(0), T(0)};
    }
  }
  W2Twiddles<T, N, NT> twv;
  twv.fetch(a.tw);
  if (gated_out_stable(st, a.gate)) return;
  // the tables of the block: every load is issued before the LDS stores
  {
    const uint8_t* phase = pe ? pe->phase : a.phase;
    const int rows_here = nrows - row0 < RB ? nrows - row0 : RB;
    const int nb = rows_here * N;
    const uint8_t* src = phase + (long long)row0 * N;
    if ((reinterpret_cast<uintptr_t>(src) & 3u) == 0) {
      constexpr int PW = (RB * N / 4 + NT - 1) / NT;  // phase words per thread
      const uint32_t* s4 = reinterpret_cast<const uint32_t*>(src);
      uint32_t* d4 = reinterpret_cast<uint32_t*>(phs);
      uint32_t pw[PW];
#pragma unroll
      for (int u = 0; u < PW; ++u) {
        const int i = (int)threadIdx.x + NT * u;
        pw[u] = i < nb / 4 ? s4[i] : 0u;
      }
#pragma unroll
      for (int u = 0; u < PW; ++u) {
        const int i = (int)threadIdx.x + NT * u;
        if (i < nb / 4) d4[i] = pw[u];
      }
      for (int i = (nb / 4) * 4 + threadIdx.x; i < nb; i += NT) phs[i] = src[i];
    } else {
      constexpr int PB = (RB * N + NT - 1) / NT < 16 ? (RB * N + NT - 1) / NT : 16;  // bytes in flight per thread
      for (int i0 = threadIdx.x; i0 < nb; i0 += NT * PB) {
        uint8_t v[PB];
#pragma unroll
        for (int u = 0; u < PB; ++u) v[u] = i0 + NT * u < nb ? src[i0 + NT * u] : (uint8_t)0;
#pragma unroll
        for (int u = 0; u < PB; ++u)
          if (i0 + NT * u < nb) phs[i0 + NT * u] = v[u];
      }
    }
  }
  const T* csrc = a.cond + (long long)pb * kCondStride;
  for (int i = threadIdx.x; i < a.n_phases; i += NT) cond[i] = csrc[i];
  twv.put(tw);
  __syncthreads();
  const T l0 = pe ? (T)pe->l0 : a.l0;
  const T Ea = (a.flags & ROWF_STATE_E) ? (T)st->E[al] : (al == 0 ? a.E[0] : a.E[1]);
  const uint8_t* pA = phs + 2 * ln.seq * N;             // phases of rowA, then rowA + 1
  cx<T> v[9];
  if constexpr (MODE == ROW_FWD) {
    // real rows in (or the constant E), times dL when asked; a batched
    // problem without a warm start projects the zero field
    const double* rin = pe ? (pe->x0 ? pe->x0 + al * nvox : nullptr) : (al == 0 ? a.real_in[0] : a.real_in[1]);
#pragma unroll
    for (int r = 0; r < 9; ++r) {
      const int x = ln.j + LPS * r;
      T t[2] = {T(0), T(0)};
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (!(u == 0 ? hasA : hasB)) continue;
        T val = (a.flags & ROWF_CONST_E) ? Ea : (rin ? (T)rin[(long long)(rowA + u) * N + x] : T(0));
        if (a.flags & ROWF_DL) val *= cond[pA[u * N + x]] - l0;
        t[u] = val;
      }
      v[r] = cx<T>{t[0], t[1]};
    }
  } else {
    // two Hermitian half rows -> one full complex row, inverse transform
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int e = ln.in_group + G::GT * it;
      if (e >= TOT) continue;
      const int k = e / G::SPG;
      cx<T>* sq = gbuf + (e - k * G::SPG) * N;
      sq[k] = cx<T>{A[it].re - B[it].im, A[it].im + B[it].re};
      if (k > 0) sq[N - k] = cx<T>{A[it].re + B[it].im, B[it].re - A[it].im};
    }
    fft_sync<N>();
    cx<T> z[9];
    wave_fft_lds_regs<T, N, +1>(buf, tw, ln.j, ln.act, z);
    if constexpr (MODE == ROW_INV || MODE == ROW_FUSED_OUT) {
      double* out = pe ? (pe->e_out ? pe->e_out + al * nvox : nullptr) : (al == 0 ? a.real_out[0] : a.real_out[1]);
      const double* add = al == 0 ? a.real_add[0] : a.real_add[1];
      double acc = 0.0;
#pragma unroll
      for (int r = 0; r < 9; ++r) {
        const int x = ln.j + LPS * r;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          if (!(u == 0 ? hasA : hasB)) continue;
          const long long g = (long long)(rowA + u) * N + x;
          const int q = pA[u * N + x];
          double val = (double)Ea + (double)((u == 0 ? z[r].re : z[r].im) * a.inv_n);
          if (a.flags & ROWF_DL_OUT) val *= (double)cond[q] - (double)l0;
          if (a.flags & ROWF_ADD) val += add[g];
          if (out) out[g] = val;
          if (a.flags & ROWF_LEFF) acc += (double)cond[q] * val;
        }
      }
      if (a.flags & ROWF_LEFF)
        store_partial<NT>(acc, parts.region(MODE == ROW_INV ? PART_AUX : PART_PQ) + (long long)rb * 3 + al);
    }
    if constexpr (MODE == ROW_INV) {
      return;
    } else {
      // polarisation dL (E + u) at the nodes (Sec. 2.2, Eq. (17))
#pragma unroll
      for (int r = 0; r < 9; ++r) {
        const int x = ln.j + LPS * r;
        T t0 = T(0), t1 = T(0);
        if (hasA) t0 = (cond[pA[x]] - l0) * (Ea + z[r].re * a.inv_n);
        if (hasB) t1 = (cond[pA[N + x]] - l0) * (Ea + z[r].im * a.inv_n);
        v[r] = cx<T>{t0, t1};
      }
    }
  }
  if constexpr (MODE != ROW_INV) {
    wave_fft<T, N, -1>(v, buf, tw, ln.j, ln.act);
    fft_sync<N>();
    // split the two rows' spectra
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int e = ln.in_group + G::GT * it;
      if (e >= TOT) continue;
      const int k = e / G::SPG, qq = e - k * G::SPG, ra = grow0 + 2 * qq;
      const cx<T> Y = gbuf[qq * N + k];
      const cx<T> Ym = gbuf[qq * N + (k == 0 ? 0 : N - k)];
      const T half = T(0.5);
      cx<T>* sp = spec + (long long)k * nrows + ra;
      if (ra < nrows) sp[0] = cx<T>{(Y.re + Ym.re) * half, (Y.im - Ym.im) * half};
      if (ra + 1 < nrows) sp[1] = cx<T>{(Y.im + Ym.im) * half, (Ym.re - Y.re) * half};
    }
  }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------

namespace {

template <typename T, int N>
hipError_t launch_w2_row_n(const RowArgs<T>& a, hipStream_t s) {
  using G = W2<N>;
  const size_t lds = (size_t)(N + G::SPB * N) * sizeof(cx<T>) + ((size_t)a.n_phases * sizeof(T) + 15) / 16 * 16 +
                     ((size_t)2 * G::SPB * N + 3) / 4 * 4;
  const dim3 grid(2u * (unsigned)row_blocks(a), (unsigned)(a.bt.nprob > 1 ? a.bt.nprob : 1));
  if (a.mode == ROW_FUSED) hipLaunchKernelGGL((w2_row_kernel<T, N, ROW_FUSED>), grid, dim3(G::NT), lds, s, a);
  else if (a.mode == ROW_INV) hipLaunchKernelGGL((w2_row_kernel<T, N, ROW_INV>), grid, dim3(G::NT), lds, s, a);
  else if (a.mode == ROW_FUSED_OUT) {
    if constexpr (sizeof(T) == 8) hipLaunchKernelGGL((w2_row_kernel<T, N, ROW_FUSED_OUT>), grid, dim3(G::NT), lds, s, a);
  }
  else hipLaunchKernelGGL((w2_row_kernel<T, N, ROW_FWD>), grid, dim3(G::NT), lds, s, a);
  return hipGetLastError();
}

template <typename T, int N>
hipError_t launch_w2_col_n(const ColArgs<T>& a, hipStream_t s) {
  using G = W2<N>;
  const size_t lds = (size_t)(N + G::SPB * N) * sizeof(cx<T>);
  const dim3 grid((unsigned)col_blocks(a), (unsigned)(a.bt.nprob > 1 ? a.bt.nprob : 1));
  if (a.mode == COL_INV_C) hipLaunchKernelGGL((w2_inv_kernel<T, N>), grid, dim3(G::NT), lds, s, a);
  else hipLaunchKernelGGL((w2_fwd_kernel<T, N>), grid, dim3(G::NT), lds, s, a);
  return hipGetLastError();
}

}  // namespace

template <typename T>
hipError_t launch_w2_row(const RowArgs<T>& a, hipStream_t s) {
  if (sizeof(T) == 4 && a.mode == ROW_FUSED_OUT) return hipErrorInvalidValue;  // FP64 only
  switch (a.n) {
    case 729: return launch_w2_row_n<T, 729>(a, s);
    case 243: return launch_w2_row_n<T, 243>(a, s);
    case 81: return launch_w2_row_n<T, 81>(a, s);
    default: return hipErrorInvalidValue;
  }
}

template <typename T>
hipError_t launch_w2_col(const ColArgs<T>& a, hipStream_t s) {
  switch (a.L) {
    case 729: return launch_w2_col_n<T, 729>(a, s);
    case 243: return launch_w2_col_n<T, 243>(a, s);
    case 81: return launch_w2_col_n<T, 81>(a, s);
    default: return hipErrorInvalidValue;
  }
}

template hipError_t launch_w2_row<double>(const RowArgs<double>&, hipStream_t);
template hipError_t launch_w2_row<float>(const RowArgs<float>&, hipStream_t);
template hipError_t launch_w2_col<double>(const ColArgs<double>&, hipStream_t);
template hipError_t launch_w2_col<float>(const ColArgs<float>&, hipStream_t);

}  // namespace lshom
