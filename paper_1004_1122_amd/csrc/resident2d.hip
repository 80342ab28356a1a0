// CG (and basic-scheme) iterations of a small 2-D image by one block: the two
// fields of the apply stay in LDS through both transforms, both ways, x, r, p
// and the Green factors in registers, and the scalars of the iteration never
// leave the block.  A batch runs one block per image.
//
// A small image is bound by latency: of the 28 us of a 63^2 FP64 iteration on
// four launches about half is launches, waits for the previous launch's sums
// and memory latency, on a chip that is otherwise empty.  Here an iteration
// has block barriers only: its two waves per SIMD issue an instruction in 27% of
// their cycles and wait, for LDS and at barriers, in 55% (counters of a 63^2
// solve; an FP32 build took the same time).  63^2: 27 -> 18 us per iteration (1024
// threads spilled 300 registers; x, r and p in global memory 23 us; one copy
// of the transform code in place of four, with the inverse ones as transforms
// of conjugates, 22 us).  Solves: 63^2, 21 iterations, 0.73 -> 0.55 ms; 64 of
// 63^2 2.2 -> 0.96 ms; 1000 of 64^2 16.9 -> 4.7 ms.
#include <hip/hip_runtime.h>

#include "kernels.hpp"
#include "reduce.hpp"

namespace lshom {

namespace {

constexpr int kNT = kResidentThreads;

__host__ __device__ inline size_t res_align(size_t v) { return (v + 15) & ~(size_t)15; }

// Byte offsets of the block's LDS arrays.
struct ResidentLds {
  size_t tw0, tw1, cond, phase, total;
  __host__ __device__ ResidentLds(int N0, int N1, int ss0, int ss1, int n_phases) {
    constexpr size_t elem = sizeof(cx<double>);
    const int h = N1 / 2 + 1, pairs = (N0 + 1) / 2;
    const size_t a = (size_t)2 * h * ss0, b = (size_t)2 * pairs * ss1;
    tw0 = res_align((a > b ? a : b) * elem);
    tw1 = res_align(tw0 + (size_t)N0 * elem);
    cond = res_align(tw1 + (size_t)N1 * elem);
    phase = res_align(cond + (size_t)n_phases * (elem / 2));
    total = phase + (size_t)N0 * N1;
  }
};

// 1 / |xi| of half-spectrum entry (k0, k1) and the components of xi; 0 where
// the Green operator vanishes (k = 0, Nyquist modes of even axes).
__device__ __forceinline__ double res_inv_norm(const ResidentArgs& a, int k0, int k1, double* x0, double* x1) {
  const int f0 = k0 <= a.N0 / 2 ? k0 : k0 - a.N0;
  *x0 = (double)f0 * a.cinv[0];
  *x1 = (double)k1 * a.cinv[1];
  const double k2 = *x0 * *x0 + *x1 * *x1;
  const bool nyquist = ((a.N0 & 1) == 0 && k0 == a.N0 / 2) || ((a.N1 & 1) == 0 && k1 == a.N1 / 2);
  return k2 > 0.0 && !nyquist ? 1.0 / sqrt(k2) : 0.0;
}

template <int RS, bool BASIC>
__global__ __launch_bounds__(kNT) void resident_kernel(ResidentArgs a) {
  constexpr int PE = kResidentPerThread / 2 + 1;  // spectral entries per thread, at most
  const int pb = a.bt.live ? a.bt.live[blockIdx.x] : (int)blockIdx.x;
  DevState* st = a.st + pb;
  // only this block writes the flags, after the barriers below
  if (gated_out_stable(st, a.gate)) return;
  const ProbEntry* pe = a.bt.tab ? a.bt.tab + pb : nullptr;
  Partials parts = a.parts;
  parts.base += (long long)pb * a.bt.pstride;
  const long long vo = (long long)pb * a.bt.vstride;
  const int tid = threadIdx.x;
  const int N0 = a.N0, N1 = a.N1, h = a.h, ss0 = a.ss0, ss1 = a.ss1;
  const int pairs = (N0 + 1) / 2;
  const int f1off = h * ss0;
  // entries before N0 and from w1 on have no mirror image in the half spectrum
  const int w1 = (N1 & 1) ? h * N0 : (h - 1) * N0;
  const int entries = h * N0, pair_entries = 2 * pairs * h, nodes = 2 * pairs * N1;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const ResidentLds lds(N0, N1, ss0, ss1, a.n_phases);
  cx<double>* F = reinterpret_cast<cx<double>*>(smem_raw);  // columns (al h + k1) ss0 + k0, or rows (al pairs + p) ss1 + x
  cx<double>* tw0 = reinterpret_cast<cx<double>*>(smem_raw + lds.tw0);
  cx<double>* tw1 = reinterpret_cast<cx<double>*>(smem_raw + lds.tw1);
  double* cond = reinterpret_cast<double*>(smem_raw + lds.cond);
  uint8_t* phs = smem_raw + lds.phase;
  const uint8_t* phase = pe ? pe->phase : a.phase;
  for (int i = tid; i < N0; i += kNT) tw0[i] = a.tw[0][i];
  for (int i = tid; i < N1; i += kNT) tw1[i] = a.tw[1][i];
  for (int i = tid; i < a.n_phases; i += kNT) cond[i] = a.cond[(long long)pb * kCondStride + i];
  for (int i = tid; i < N0 * N1; i += kNT) phs[i] = phase[i];
  cx<double>* __restrict__ X = a.x + vo;
  cx<double>* __restrict__ Rv = a.r + vo;
  cx<double>* __restrict__ P = a.p + vo;
  const double l0 = pe ? pe->l0 : a.l0;
  const double cs = (1.0 / l0) * (BASIC ? -1.0 : 1.0);
  const double E0 = BASIC ? st->E[0] : 0.0, E1 = BASIC ? st->E[1] : 0.0;
  const double tol2b2 = st->tol2b2;
  const int max_iter = st->max_iter;
  int k = st->iter_a, k_last = st->iter_u;
  // the sums the last launch left: (r, r) of this iterate and of the one before
  double cur = 0.0, prev = 0.0;
  if (!BASIC) {
    cur = sum_partials<kNT>(parts.region(k & 1), st->nparts[k & 1]);
    if (k > 0) prev = sum_partials<kNT>(parts.region((k + 1) & 1), st->nparts[(k + 1) & 1]);
  }
  __syncthreads();
  // the thread's entries of x, r, p and i khat stay in registers
  cx<double> xv[PE], rv[PE], pv[PE];
  double ka[PE], kb[PE];
  int at[PE];  // LDS place of the entry in field 0
#pragma unroll
  for (int u = 0; u < PE; ++u) {
    const int i = tid + u * kNT;
    ka[u] = kb[u] = 0.0;
    at[u] = 0;
    xv[u] = rv[u] = pv[u] = cx<double>{0.0, 0.0};
    if (i < entries) {
      const int k1 = (int)fdiv((uint32_t)i, a.fd_n0), k0 = i - k1 * N0;
      double x0, x1;
      const double inv = res_inv_norm(a, k0, k1, &x0, &x1);
      at[u] = k1 * ss0 + k0;
      ka[u] = x0 * inv;
      kb[u] = x1 * inv;
      xv[u] = X[i];
      if constexpr (!BASIC) {
        rv[u] = Rv[i];
        pv[u] = P[i];
      }
    }
  }
  double alpha = st->alpha_log, pq = st->pq_log, rr_log = st->rr_log;
  int status = 0, done = 0;
  for (int it = 0; it < a.iters; ++it) {
    double beta = 0.0;
    const double rr = cur * a.inv_n;
    if constexpr (!BASIC) {
      // the direction step's tests (cg_direction), the same in every thread
      bool stop = false;
      if (!isfinite(rr)) {
        status = -6;
        done = 1;
        stop = true;
      } else if (rr <= tol2b2) {
        done = 1;
        stop = true;
      } else if (k >= max_iter) {
        status = -5;
        done = 1;
        stop = true;
      }
      k_last = k;
      rr_log = rr;
      if (stop) break;
      const double rr_prev = prev * a.inv_n;
      beta = (k == 0 || rr_prev == 0.0) ? 0.0 : rr / rr_prev;
    }
    // p = r + beta p; fields i khat_a p
#pragma unroll
    for (int u = 0; u < PE; ++u) {
      const int i = tid + u * kNT;
      if (i < entries) {
        cx<double> c = xv[u];
        if constexpr (!BASIC) c = pv[u] = cx<double>{rv[u].re + beta * pv[u].re, rv[u].im + beta * pv[u].im};
        F[at[u]] = cx<double>{-ka[u] * c.im, ka[u] * c.re};
        F[at[u] + f1off] = cx<double>{-kb[u] * c.im, kb[u] * c.re};
      }
    }
    __syncthreads();
    fft_lds<double, +1, kNT, RS, true>(F, 2 * h, ss0, a.plan[0], tw0, tid);
    // columns -> packed row pairs (two Hermitian half rows in one sequence)
    cx<double> va[PE], vb[PE];
#pragma unroll
    for (int u = 0; u < PE; ++u) {
      const int e = tid + u * kNT;
      if (e < pair_entries) {
        const int q = (int)fdiv((uint32_t)e, a.fd_h), k1 = e - q * h;
        const int al = q >= pairs ? 1 : 0, p = q - al * pairs;
        const cx<double>* col = F + (al * h + k1) * ss0 + 2 * p;
        va[u] = col[0];
        vb[u] = 2 * p + 1 < N0 ? col[1] : cx<double>{0.0, 0.0};
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PE; ++u) {
      const int e = tid + u * kNT;
      if (e < pair_entries) {
        const int q = (int)fdiv((uint32_t)e, a.fd_h), k1 = e - q * h;
        cx<double>* row = F + q * ss1;
        row[k1] = cx<double>{va[u].re - vb[u].im, va[u].im + vb[u].re};
        if (k1 >= 1 && N1 - k1 >= h) row[N1 - k1] = cx<double>{va[u].re + vb[u].im, vb[u].re - va[u].im};
      }
    }
    __syncthreads();
    fft_lds<double, +1, kNT, RS, true>(F, 2 * pairs, ss1, a.plan[1], tw1, tid);
    // polarisation dL (E + u) at the nodes (Sec. 2.2, Eq. (17))
#pragma unroll 4
    for (int i = tid; i < nodes; i += kNT) {
      const int q = (int)fdiv((uint32_t)i, a.fd_n1), x = i - q * N1;
      const int al = q >= pairs ? 1 : 0, ra = 2 * (q - al * pairs);
      const double E = al ? E1 : E0;
      const cx<double> z = F[q * ss1 + x];
      const double t0 = (cond[phs[ra * N1 + x]] - l0) * (E + z.re * a.inv_n);
      const double t1 = ra + 1 < N0 ? (cond[phs[(ra + 1) * N1 + x]] - l0) * (E + z.im * a.inv_n) : 0.0;
      F[q * ss1 + x] = cx<double>{t0, t1};
    }
    __syncthreads();
    fft_lds<double, -1, kNT, RS, true>(F, 2 * pairs, ss1, a.plan[1], tw1, tid);
    // packed row pairs -> columns
#pragma unroll
    for (int u = 0; u < PE; ++u) {
      const int e = tid + u * kNT;
      if (e < pair_entries) {
        const int q = (int)fdiv((uint32_t)e, a.fd_h), k1 = e - q * h;
        const cx<double> Y = F[q * ss1 + k1], Ym = F[q * ss1 + (k1 == 0 ? 0 : N1 - k1)];
        const double half = 0.5;
        va[u] = cx<double>{(Y.re + Ym.re) * half, (Y.im - Ym.im) * half};
        vb[u] = cx<double>{(Y.im + Ym.im) * half, (Ym.re - Y.re) * half};
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PE; ++u) {
      const int e = tid + u * kNT;
      if (e < pair_entries) {
        const int q = (int)fdiv((uint32_t)e, a.fd_h), k1 = e - q * h;
        const int al = q >= pairs ? 1 : 0, p = q - al * pairs;
        cx<double>* col = F + (al * h + k1) * ss0 + 2 * p;
        col[0] = va[u];
        if (2 * p + 1 < N0) col[1] = vb[u];
      }
    }
    __syncthreads();
    fft_lds<double, -1, kNT, RS, true>(F, 2 * h, ss0, a.plan[0], tw0, tid);
    // q = p + (1 / l0) (-i khat) . tau_hat and (p, q)
    cx<double> qv[PE];
    double acc = 0.0;
#pragma unroll
    for (int u = 0; u < PE; ++u) {
      const int i = tid + u * kNT;
      if (i < entries) {
        const cx<double> f0 = F[at[u]], f1 = F[at[u] + f1off];
        const cx<double> t = {ka[u] * f0.re + kb[u] * f1.re, ka[u] * f0.im + kb[u] * f1.im};
        const double w = i < N0 || i >= w1 ? 1.0 : 2.0;
        cx<double> val = {cs * t.im, -cs * t.re};
        if constexpr (BASIC) {
          const cx<double> old = xv[u];
          xv[u] = val;
          const double dr = val.re - old.re, di = val.im - old.im;
          acc += w * (dr * dr + di * di);
        } else {
          val.re += pv[u].re;
          val.im += pv[u].im;
          qv[u] = val;
          acc += w * (pv[u].re * val.re + pv[u].im * val.im);
        }
      }
    }
    acc = block_sum_all<kNT>(acc);
    if constexpr (BASIC) {
      // the step is the residual of iterate k, which became k + 1
      const double step = acc * a.inv_n;
      rr_log = step;
      k_last = k;
      k += 1;
      if (!isfinite(step)) {
        status = -6;
        done = 1;
      } else if (step <= tol2b2) {
        done = 1;
      } else if (k >= max_iter) {
        status = -5;
        done = 1;
      }
      if (done) break;
      continue;
    }
    pq = acc * a.inv_n;
    if (!(pq > 0.0) || !isfinite(pq)) {
      status = -6;
      done = 1;
      break;
    }
    alpha = rr / pq;
    const double ta = alpha;
    acc = 0.0;
#pragma unroll
    for (int u = 0; u < PE; ++u) {
      const int i = tid + u * kNT;
      if (i < entries) {
        xv[u].re += ta * pv[u].re;
        xv[u].im += ta * pv[u].im;
        rv[u].re -= ta * qv[u].re;
        rv[u].im -= ta * qv[u].im;
        const double w = i < N0 || i >= w1 ? 1.0 : 2.0;
        acc += w * (rv[u].re * rv[u].re + rv[u].im * rv[u].im);
      }
    }
    prev = cur;
    cur = block_sum_all<kNT>(acc);
    k += 1;
  }
#pragma unroll
  for (int u = 0; u < PE; ++u) {
    const int i = tid + u * kNT;
    if (i < entries) {
      X[i] = xv[u];
      if constexpr (!BASIC) {
        Rv[i] = rv[u];
        P[i] = pv[u];
      }
    }
  }
  if (tid == 0) {
    st->iter_a = k;
    st->iter_u = k_last;
    st->rr_log = rr_log;
    if (status) st->status = status;
    if (done) st->done = 1;
    if constexpr (!BASIC) {
      st->alpha_log = alpha;
      st->pq_log = pq;
      // the sums for the next launch
      parts.region(k & 1)[0] = cur;
      parts.region((k + 1) & 1)[0] = prev;
      st->nparts[0] = 1;
      st->nparts[1] = 1;
    }
  }
}

template <int RS>
hipError_t launch_resident_rs(const ResidentArgs& a, bool basic, hipStream_t s) {
  const ResidentLds lds(a.N0, a.N1, a.ss0, a.ss1, a.n_phases);
  const dim3 grid((unsigned)(a.bt.nprob > 1 ? a.bt.nprob : 1));
  if (basic) hipLaunchKernelGGL((resident_kernel<RS, true>), grid, dim3(kNT), lds.total, s, a);
  else hipLaunchKernelGGL((resident_kernel<RS, false>), grid, dim3(kNT), lds.total, s, a);
  return hipGetLastError();
}

}  // namespace

bool resident_fits(const int64_t* N, size_t lds_limit) {
  const int n0 = (int)N[0], n1 = (int)N[1];
  // butterflies of 11, 13 and 17 overflow the registers at this block size
  for (int p : {11, 13, 17})
    if (N[0] % p == 0 || N[1] % p == 0) return false;
  // kResidentPoints: the largest image is about 67 x 67.  With twice as many per
  // thread 75^2 took 41 us per iteration, against 33 us on the block passes
  const long long cols = 2ll * (n1 / 2 + 1) * n0, rows = 2ll * ((n0 + 1) / 2) * n1;
  if (cols > kResidentPoints || rows > kResidentPoints) return false;
  // entries a thread carries, and between the two layouts
  if (cols / 2 > (long long)kNT * (kResidentPerThread / 2 + 1)) return false;
  const long long pair_entries = 2ll * ((n0 + 1) / 2) * (n1 / 2 + 1);
  if (pair_entries > (long long)kNT * (kResidentPerThread / 2 + 1)) return false;
  return ResidentLds(n0, n1, lds_odd_stride(n0), lds_odd_stride(n1), kCondStride).total <= lds_limit;
}

hipError_t launch_resident(const ResidentArgs& a, bool basic, hipStream_t s) {
  const int r0 = plan_radix_set(a.plan[0]), r1 = plan_radix_set(a.plan[1]);
  if (r0 == RADIX_POW3 && r1 == RADIX_POW3) return launch_resident_rs<RADIX_POW3>(a, basic, s);
  if (r0 == RADIX_POW2 && r1 == RADIX_POW2) return launch_resident_rs<RADIX_POW2>(a, basic, s);
  if (r0 == RADIX_WIDE || r1 == RADIX_WIDE) return hipErrorInvalidValue;
  return launch_resident_rs<RADIX_ALL>(a, basic, s);
}

}  // namespace lshom
