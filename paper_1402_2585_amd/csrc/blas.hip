// BLAS-1 kernels with device-resident coefficients and FP64 reductions.
#include "blas.h"

#include <algorithm>

namespace hdk {

namespace {

constexpr int kT = 256;
constexpr int kMaxGrid = 1024;  // workgroups of a launch over all right-hand sides

// Workgroups per right-hand side: at least eight elements a thread, and at
// most four workgroups per CU over all right-hand sides.  These kernels are
// bound by HBM (or the Infinity Cache), which 1024 workgroups with several
// loads in flight a thread saturate; with 1024 per right-hand side (up to
// 16384) the tickets of the reductions cost more than the data: on 4 x
// 12^3 x 24 x 8 16-bit fields, 3888 tickets of about 10 ns each kept k_xpay
// at 54.6 us for 96 MB.
inline int nblocks(size_t n, int nrhs = 1) {
  size_t b = (n + kT * 8 - 1) / (kT * 8);
  const size_t most = std::max(16, kMaxGrid / std::max(1, nrhs));
  if (b < 1) b = 1;
  if (b > most) b = most;
  return (int)b;
}

template <typename R>
__device__ __forceinline__ double nrm(cplx<R> a) {
  return (double)a.re * a.re + (double)a.im * a.im;
}

__device__ __forceinline__ void coef(const double* num, bool cnum, const double* den,
                                     const double* den2, double lam, int rhs, double& re,
                                     double& im, int dstr) {
  double d = den[rhs * dstr];
  if (den2) d += lam * den2[rhs];
  if (d == 0.0) {
    re = im = 0.0;
    return;
  }
  if (cnum) {
    re = num[2 * rhs] / d;
    im = num[2 * rhs + 1] / d;
  } else {
    re = num[rhs] / d;
    im = 0.0;
  }
}

// Workgroup sums of one right-hand side's NQ quantities, reduced over the
// grid inside the producing kernel: each workgroup stores its partials with
// coherent device-scope stores, waits for them to complete and takes a
// ticket; the workgroup that takes the last ticket sums every partial in a
// fixed order (the result does not depend on which one it is), writes
// res[NQ * rhs + q] and resets the ticket counters.  Tickets come in two
// levels, kTicketSubs counters of a right-hand side and one for the last of
// each, every counter on a cache line of its own: atomics on one address run
// one after another (about 10 ns each), so a single counter would hold 1024
// workgroups up for 10 us.  No workgroup waits for another, and no cache
// maintenance is needed.
template <int NQ>
__device__ __forceinline__ void reduce_out(double (&v)[NQ], Red red, int rhs, double* res, double* host = nullptr) {
  __shared__ double lds[NQ * 16];
  __shared__ int last;
  constexpr int nslots = kMaxPartials / NQ;
  double* part = red.partials + (size_t)rhs * kMaxPartials;
  block_sum<NQ>(v, lds);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int q = 0; q < NQ; ++q)
      __hip_atomic_store(part + q * nslots + blockIdx.x, v[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_s_waitcnt(0);
    last = last_ticket(red.counters, rhs, gridDim.x, blockIdx.x);
  }
  __syncthreads();
  if (!last) return;
  double s[NQ];
  const int G = (int)gridDim.x, B = (int)blockDim.x;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    s[q] = 0.0;
    // four partials per trip, loads first (the last workgroup's sum is on
    // the kernel's critical path)
    for (int i0 = threadIdx.x; i0 < G; i0 += 4 * B) {
      double a[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        a[u] = i0 + u * B < G ? __hip_atomic_load(part + q * nslots + i0 + u * B, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT)
                              : 0.0;
#pragma unroll
      for (int u = 0; u < 4; ++u) s[q] += a[u];
    }
  }
  block_sum<NQ>(s, lds);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) res[NQ * rhs + q] = s[q];
    if (host) __hip_atomic_store(host + rhs, s[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// Sum of the per-workgroup partials of a kernel that does not finish its own
// reduction (the hop kernel's fused norm: one partial per workgroup, up to
// ~10^5).  One 1024-thread workgroup per right-hand side; each lane keeps
// eight independent accumulators so eight loads are in flight per trip
// (fixed order: deterministic).
constexpr int kFinT = 1024;
template <int NQ>
__global__ void __launch_bounds__(kFinT) k_finalize(const double* __restrict__ partials, int nslots,
                                                    int nblocks, size_t rstride, double* __restrict__ res,
                                                    FinCg cg) {
  const int rhs = blockIdx.x;
  const double* p = partials + (size_t)rhs * rstride;
  __shared__ double lds[kFinT / 64];
  for (int q = 0; q < NQ; ++q) {
    const double* pq = p + (size_t)q * nslots;
    double s[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    int i = threadIdx.x;
    for (; i + 7 * kFinT < nblocks; i += 8 * kFinT) {
#pragma unroll
      for (int u = 0; u < 8; ++u) s[u] += pq[i + u * kFinT];
    }
    for (; i < nblocks; i += kFinT) s[0] += pq[i];
    double t = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
    t = wave_sum(t);
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0) {
      double r = 0.0;
      for (int w = 0; w < kFinT / 64; ++w) r += lds[w];
      if (NQ == 1) fin_store(r, rhs, res, cg);
      else res[NQ * rhs + q] = r;
    }
    __syncthreads();
  }
}

// Fields are stored as T (cplx<R>, or bf16c with FP32 arithmetic).  The
// streaming kernels move Vec<T>::V consecutive values per lane and operand
// with one load or store: one complex for cplx<R>, four bf16c (16 bytes) for
// the 16-bit storage, so a lane keeps as many bytes in flight as in complex64
// or wider.  n must be a multiple of V (the launchers check).
template <typename T>
struct Vec {
  static constexpr int V = 1;
  using R = typename St<T>::R;
  __device__ __forceinline__ static void ld(const T* p, size_t g, cplx<R> (&o)[1]) { o[0] = St<T>::ld(p + g); }
  __device__ __forceinline__ static void st(T* p, size_t g, const cplx<R> (&v)[1]) { St<T>::st(p + g, v[0]); }
};
struct alignas(16) bf16c4 {
  bf16c v[4];
};
template <>
struct Vec<bf16c> {
  static constexpr int V = 4;
  __device__ __forceinline__ static void ld(const bf16c* p, size_t g, cplx<float> (&o)[4]) {
    const bf16c4 q = reinterpret_cast<const bf16c4*>(p)[g];
#pragma unroll
    for (int k = 0; k < 4; ++k) o[k] = St<bf16c>::ld(&q.v[k]);
  }
  __device__ __forceinline__ static void st(bf16c* p, size_t g, const cplx<float> (&v)[4]) {
    bf16c4 q;
#pragma unroll
    for (int k = 0; k < 4; ++k) St<bf16c>::st(&q.v[k], v[k]);
    reinterpret_cast<bf16c4*>(p)[g] = q;
  }
};
// f(g) for this thread's groups g = tid, tid + S, ... < m (S threads in the
// grid), two at a time while both exist: f issues the loads of both before
// its arithmetic.
template <typename F>
__device__ __forceinline__ void stream2(size_t m, F f) {
  const size_t S = (size_t)gridDim.x * kT;
  size_t g = (size_t)blockIdx.x * kT + threadIdx.x;
  for (; g + S < m; g += 2 * S) {
    const size_t at[2] = {g, g + S};
    f(at);
  }
  if (g < m) {
    const size_t at[1] = {g};
    f(at);
  }
}

template <typename T>
__global__ void __launch_bounds__(kT) k_norm2(const T* __restrict__ x, size_t n, Red red,
                                              double* res) {
  using R = typename St<T>::R;
  const int rhs = blockIdx.y;
  x += rhs * n;
  constexpr int V = Vec<T>::V;
  double acc = 0.0;
  stream2(n / V, [&](const auto& at) {
    constexpr int U = sizeof(at) / sizeof(at[0]);
    cplx<R> v[U][V];
#pragma unroll
    for (int u = 0; u < U; ++u) Vec<T>::ld(x, at[u], v[u]);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 0; k < V; ++k) acc += nrm(v[u][k]);
  });
  double v[1] = {acc};
  reduce_out<1>(v, red, rhs, res);
}

template <typename T>
__global__ void __launch_bounds__(kT) k_dot(const T* __restrict__ a, const T* __restrict__ b,
                                            size_t n, Red red, double* res) {
  const int rhs = blockIdx.y;
  a += rhs * n;
  b += rhs * n;
  double re = 0.0, im = 0.0;
  stream2(n, [&](const auto& at) {
    constexpr int U = sizeof(at) / sizeof(at[0]);
    cplx<typename St<T>::R> x[U], y[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = St<T>::ld(a + at[u]), y[u] = St<T>::ld(b + at[u]);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      re += (double)x[u].re * y[u].re + (double)x[u].im * y[u].im;
      im += (double)x[u].re * y[u].im - (double)x[u].im * y[u].re;
    }
  });
  double v[2] = {re, im};
  reduce_out<2>(v, red, rhs, res);
}

template <typename T, int MODE>
__global__ void __launch_bounds__(kT)
k_update(T* __restrict__ x, T* __restrict__ r, const T* __restrict__ p, const T* __restrict__ w,
         size_t n, const double* num, bool cnum, const double* den, const double* den2, double lam,
         Red red, double* rr, int dstr) {
  constexpr bool X0 = MODE & kUpdX0, XONLY = MODE & kUpdXOnly;
  using R = typename St<T>::R;
  const int rhs = blockIdx.y;
  const size_t off = rhs * n;
  double are, aim;
  coef(num, cnum, den, den2, lam, rhs, are, aim, dstr);
  const cplx<R> a = cmk((R)are, (R)aim);
  const R l = (R)lam;
  constexpr int V = Vec<T>::V;
  x += off;
  r += off;
  p += off;
  w += off;
  double acc = 0.0;
  stream2(n / V, [&](const auto& at) {
    constexpr int U = sizeof(at) / sizeof(at[0]);
    cplx<R> pv[U][V], wv[U][V], xv[U][V], rv[U][V];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      Vec<T>::ld(p, at[u], pv[u]);
      if constexpr (!XONLY) {
        Vec<T>::ld(w, at[u], wv[u]);
        Vec<T>::ld(r, at[u], rv[u]);
      }
      if constexpr (!X0) Vec<T>::ld(x, at[u], xv[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int k = 0; k < V; ++k) {
        if constexpr (X0) xv[u][k] = cmk((R)0, (R)0);
        xv[u][k] = xv[u][k] + a * pv[u][k];
        if constexpr (!XONLY) {
          if (den2) wv[u][k] = wv[u][k] + l * pv[u][k];
          rv[u][k] = rv[u][k] - a * wv[u][k];
          acc += nrm(rv[u][k]);
        }
      }
      Vec<T>::st(x, at[u], xv[u]);
      if constexpr (!XONLY) Vec<T>::st(r, at[u], rv[u]);
    }
  });
  if (!XONLY && rr) {
    double v[1] = {acc};
    reduce_out<1>(v, red, rhs, rr);
  }
}

template <typename T>
__global__ void __launch_bounds__(kT)
k_xpay(T* __restrict__ p, const T* __restrict__ y, size_t n, const double* num, bool cnum,
       const double* den, double sign, Red red, double* pp, int dstr) {
  using R = typename St<T>::R;
  const int rhs = blockIdx.y;
  const size_t off = rhs * n;
  double bre, bim;
  coef(num, cnum, den, nullptr, 0.0, rhs, bre, bim, dstr);
  const cplx<R> b = cmk((R)(sign * bre), (R)(sign * bim));
  constexpr int V = Vec<T>::V;
  p += off;
  y += off;
  double acc = 0.0;
  stream2(n / V, [&](const auto& at) {
    constexpr int U = sizeof(at) / sizeof(at[0]);
    cplx<R> yv[U][V], pv[U][V];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      Vec<T>::ld(y, at[u], yv[u]);
      Vec<T>::ld(p, at[u], pv[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int k = 0; k < V; ++k) {
        pv[u][k] = yv[u][k] + b * pv[u][k];
        acc += nrm(pv[u][k]);
      }
      Vec<T>::st(p, at[u], pv[u]);
    }
  });
  if (pp) {
    double v[1] = {acc};
    reduce_out<1>(v, red, rhs, pp);
  }
}

// The rest of a CG step whose residual the hop has updated: x += alpha p and
// p = r + beta p in one pass (five fields instead of the six that an update
// of x and one of p would move), alpha as formed with <p, H p>, beta = num / den.
template <typename T, bool X0>
__global__ void __launch_bounds__(kT)
k_cg_xp(T* __restrict__ x, T* __restrict__ p, const T* __restrict__ r, size_t n, const double* alpha,
        const double* num, const double* den, Red red, double* pp) {
  using R = typename St<T>::R;
  const int rhs = blockIdx.y;
  const size_t off = rhs * n;
  double bre, bim;
  coef(num, false, den, nullptr, 0.0, rhs, bre, bim, 1);
  const R a = (R)alpha[rhs], b = (R)bre;
  constexpr int V = Vec<T>::V;
  x += off;
  p += off;
  r += off;
  double acc = 0.0;
  stream2(n / V, [&](const auto& at) {
    constexpr int U = sizeof(at) / sizeof(at[0]);
    cplx<R> xv[U][V], pv[U][V], rv[U][V];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      Vec<T>::ld(p, at[u], pv[u]);
      Vec<T>::ld(r, at[u], rv[u]);
      if constexpr (!X0) Vec<T>::ld(x, at[u], xv[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int k = 0; k < V; ++k) {
        xv[u][k] = X0 ? a * pv[u][k] : xv[u][k] + a * pv[u][k];
        pv[u][k] = rv[u][k] + b * pv[u][k];
        acc += nrm(pv[u][k]);
      }
      Vec<T>::st(x, at[u], xv[u]);
      Vec<T>::st(p, at[u], pv[u]);
    }
  });
  if (pp) {
    double v[1] = {acc};
    reduce_out<1>(v, red, rhs, pp);
  }
}

// r -= alpha (w + lam p), rr = |r|^2 (rr_host, nullable: pinned memory that
// takes it too)
template <typename T>
__global__ void __launch_bounds__(kT)
k_cg_r(T* __restrict__ r, const T* __restrict__ p, const T* __restrict__ w, size_t n, const double* alpha, double lam,
       Red red, double* rr, double* rr_host) {
  using R = typename St<T>::R;
  const int rhs = blockIdx.y;
  const size_t off = rhs * n;
  const R a = (R)alpha[rhs], l = (R)lam;
  constexpr int V = Vec<T>::V;
  r += off;
  p += off;
  w += off;
  double acc = 0.0;
  stream2(n / V, [&](const auto& at) {
    constexpr int U = sizeof(at) / sizeof(at[0]);
    cplx<R> rv[U][V], pv[U][V], wv[U][V];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      Vec<T>::ld(r, at[u], rv[u]);
      Vec<T>::ld(w, at[u], wv[u]);
      if (lam != 0.0) Vec<T>::ld(p, at[u], pv[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int k = 0; k < V; ++k) {
        if (lam != 0.0) wv[u][k] = wv[u][k] + l * pv[u][k];
        rv[u][k] = rv[u][k] - a * wv[u][k];
        acc += nrm(rv[u][k]);
      }
      Vec<T>::st(r, at[u], rv[u]);
    }
  });
  double v[1] = {acc};
  reduce_out<1>(v, red, rhs, rr, rr_host);
}

// Fixed-count CG on 16-bit fields (M_IRS), first step: r = p = bf16(b) for
// b complex64 [site][12][Ls] and r, p 16-bit [site][Ls][12] (rounded to
// nearest even as every 16-bit store), and rr[rhs] = |r|^2 of the rounded
// values.  One (site, s) row of 12 values per thread; rows per RHS.
__global__ void __launch_bounds__(kT)
k_mirs16_init(bf16c* __restrict__ r, bf16c* __restrict__ p, const c64* __restrict__ b, size_t rows, int Ls,
              Red red, double* rr) {
  const int rhs = blockIdx.y;
  const size_t off = (size_t)rhs * rows * 12;
  double acc = 0.0;
  for (size_t row = (size_t)blockIdx.x * kT + threadIdx.x; row < rows; row += (size_t)gridDim.x * kT) {
    const size_t site = row / Ls;
    const int s = (int)(row - site * Ls);
    const c64* f = b + off + site * 12 * Ls + s;
    bf16c4 q[3];
#pragma unroll
    for (int c = 0; c < 12; ++c) {
      St<bf16c>::st(&q[c >> 2].v[c & 3], f[c * Ls]);
      acc += nrm(St<bf16c>::ld(&q[c >> 2].v[c & 3]));
    }
    const size_t o = (off + site * 12 * Ls + (size_t)s * 12) / 4;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      reinterpret_cast<bf16c4*>(r)[o + k] = q[k];
      reinterpret_cast<bf16c4*>(p)[o + k] = q[k];
    }
  }
  double v[1] = {acc};
  reduce_out<1>(v, red, rhs, rr);
}

// Its last step: only x is still needed, x_out = x + alpha p rounded to 16
// bits as the stored x would be, written in complex64 [site][12][Ls]
// (x == nullptr: x = 0); alpha as in k_update.
__global__ void __launch_bounds__(kT)
k_mirs16_last(c64* __restrict__ xo, const bf16c* __restrict__ x, const bf16c* __restrict__ p, size_t rows,
              int Ls, const double* num, const double* den, const double* den2, double lam) {
  const int rhs = blockIdx.y;
  const size_t off = (size_t)rhs * rows * 12;
  double are, aim;
  coef(num, false, den, den2, lam, rhs, are, aim, 1);
  const cplx<float> a = cmk((float)are, (float)aim);
  for (size_t row = (size_t)blockIdx.x * kT + threadIdx.x; row < rows; row += (size_t)gridDim.x * kT) {
    const size_t site = row / Ls;
    const int s = (int)(row - site * Ls);
    const size_t o = (off + site * 12 * Ls + (size_t)s * 12) / 4;
    c64* f = xo + off + site * 12 * Ls + s;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const bf16c4 pq = reinterpret_cast<const bf16c4*>(p)[o + k];
      bf16c4 xq;
      if (x) xq = reinterpret_cast<const bf16c4*>(x)[o + k];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const cplx<float> xv = x ? St<bf16c>::ld(&xq.v[e]) : cmk(0.f, 0.f);
        bf16c t;
        St<bf16c>::st(&t, xv + a * St<bf16c>::ld(&pq.v[e]));
        f[(4 * k + e) * Ls] = St<bf16c>::ld(&t);
      }
    }
  }
}

template <typename R>
__global__ void k_axpby(cplx<R>* __restrict__ y, const cplx<R>* __restrict__ x, R a, R b,
                        size_t total) {
  for (size_t i = (size_t)blockIdx.x * kT + threadIdx.x; i < total; i += (size_t)gridDim.x * kT)
    y[i] = a * x[i] + b * y[i];
}

template <typename Ry, typename Rx>
__global__ void k_axpy_mixed(cplx<Ry>* __restrict__ y, const cplx<Rx>* __restrict__ x,
                             const double* s, size_t n, bool sqrt_s) {
  const int rhs = blockIdx.y;
  const size_t off = rhs * n;
  const Ry f = s ? (Ry)(sqrt_s ? sqrt(s[rhs]) : s[rhs]) : (Ry)1;
  for (size_t i = (size_t)blockIdx.x * kT + threadIdx.x; i < n; i += (size_t)gridDim.x * kT) {
    const cplx<Rx> v = x[off + i];
    y[off + i] = y[off + i] + f * cmk((Ry)v.re, (Ry)v.im);
  }
}

template <typename Ry, typename Rx>
__global__ void k_scale_copy(cplx<Ry>* __restrict__ y, const cplx<Rx>* __restrict__ x,
                             const double* v, bool invsqrt, size_t n) {
  const int rhs = blockIdx.y;
  const size_t off = rhs * n;
  double s = v ? v[rhs] : 1.0;
  if (invsqrt) s = s > 0.0 ? 1.0 / sqrt(s) : 0.0;
  for (size_t i = (size_t)blockIdx.x * kT + threadIdx.x; i < n; i += (size_t)gridDim.x * kT) {
    const cplx<Rx> a = x[off + i];
    y[off + i] = cmk((Ry)(s * a.re), (Ry)(s * a.im));
  }
}

template <typename T>
__global__ void k_zero(T* __restrict__ y, size_t total) {
  using R = typename St<T>::R;
  constexpr int V = Vec<T>::V;
  cplx<R> z[V];
#pragma unroll
  for (int k = 0; k < V; ++k) z[k] = cmk((R)0, (R)0);
  for (size_t g = (size_t)blockIdx.x * kT + threadIdx.x; g < total / V; g += (size_t)gridDim.x * kT)
    Vec<T>::st(y, g, z);
}

}  // namespace

#define LAUNCH_CHECK() HDCG_HIP(hipGetLastError())

int launch_finalize(int nq, const double* partials, int nslots, int nblocks, int nrhs, double* res,
                    hipStream_t st, size_t rstride, const FinCg& cg) {
  if (nblocks > nslots || (size_t)nq * nslots > rstride) return fail(DWF_ERR_ARG, "too many partial sums");
  if (nq == 1)
    hipLaunchKernelGGL((k_finalize<1>), dim3(nrhs), dim3(kFinT), 0, st, partials, nslots, nblocks, rstride, res, cg);
  else
    hipLaunchKernelGGL((k_finalize<2>), dim3(nrhs), dim3(kFinT), 0, st, partials, nslots, nblocks, rstride, res, cg);
  LAUNCH_CHECK();
  return DWF_OK;
}

template <typename T>
int norm2_t(Red red, const T* x, size_t n, int nrhs, double* res, hipStream_t st) {
  if (n % Vec<T>::V) return fail(DWF_ERR_ARG, "16-bit fields need a multiple of 4 complex values");
  if (nrhs > 64) return fail(DWF_ERR_ARG, "nrhs > 64");
  hipLaunchKernelGGL((k_norm2<T>), dim3(nblocks(n, nrhs), nrhs), dim3(kT), 0, st, x, n, red, res);
  LAUNCH_CHECK();
  return DWF_OK;
}
template <typename T>
int dot_t(Red red, const T* a, const T* b, size_t n, int nrhs, double* res, hipStream_t st) {
  if (nrhs > 64) return fail(DWF_ERR_ARG, "nrhs > 64");
  hipLaunchKernelGGL((k_dot<T>), dim3(nblocks(n, nrhs), nrhs), dim3(kT), 0, st, a, b, n, red, res);
  LAUNCH_CHECK();
  return DWF_OK;
}
template <typename T>
int update_t(Red red, T* x, T* r, const T* p, const T* w, size_t n, int nrhs, const double* num,
             bool cnum, const double* den, const double* den2, double lam, double* rr,
             hipStream_t st, int dstr, int mode) {
  if (n % Vec<T>::V) return fail(DWF_ERR_ARG, "16-bit fields need a multiple of 4 complex values");
  if (nrhs > 64) return fail(DWF_ERR_ARG, "nrhs > 64");
  if (mode < 0 || mode > (kUpdX0 | kUpdXOnly)) return fail(DWF_ERR_ARG, "update: bad mode");
  const dim3 grid(nblocks(n, nrhs), nrhs);
#define HDCG_UPDATE(M)                                                                                      \
  hipLaunchKernelGGL((k_update<T, M>), grid, dim3(kT), 0, st, x, r, p, w, n, num, cnum, den, den2, lam, red, \
                     rr, dstr)
  switch (mode) {
    case 0: HDCG_UPDATE(0); break;
    case kUpdX0: HDCG_UPDATE(kUpdX0); break;
    case kUpdXOnly: HDCG_UPDATE(kUpdXOnly); break;
    default: HDCG_UPDATE(kUpdX0 | kUpdXOnly); break;
  }
#undef HDCG_UPDATE
  LAUNCH_CHECK();
  return DWF_OK;
}
template <typename T>
int xpay_t(Red red, T* p, const T* y, size_t n, int nrhs, const double* num, bool cnum,
           const double* den, double sign, double* pp, hipStream_t st, int dstr) {
  if (n % Vec<T>::V) return fail(DWF_ERR_ARG, "16-bit fields need a multiple of 4 complex values");
  if (nrhs > 64) return fail(DWF_ERR_ARG, "nrhs > 64");
  hipLaunchKernelGGL((k_xpay<T>), dim3(nblocks(n, nrhs), nrhs), dim3(kT), 0, st, p, y, n, num, cnum, den,
                     sign, red, pp, dstr);
  LAUNCH_CHECK();
  return DWF_OK;
}
template <typename T>
int b_cg_xp(Red red, T* x, T* p, const T* r, size_t n, int nrhs, const double* alpha, const double* num,
            const double* den, bool x0, double* pp, hipStream_t st) {
  if (n % Vec<T>::V) return fail(DWF_ERR_ARG, "16-bit fields need a multiple of 4 complex values");
  if (nrhs > 64) return fail(DWF_ERR_ARG, "nrhs > 64");
  const dim3 grid(nblocks(n, nrhs), nrhs);
  if (x0) hipLaunchKernelGGL((k_cg_xp<T, true>), grid, dim3(kT), 0, st, x, p, r, n, alpha, num, den, red, pp);
  else hipLaunchKernelGGL((k_cg_xp<T, false>), grid, dim3(kT), 0, st, x, p, r, n, alpha, num, den, red, pp);
  LAUNCH_CHECK();
  return DWF_OK;
}
template <typename T>
int b_cg_r(Red red, T* r, const T* p, const T* w, size_t n, int nrhs, const double* alpha, double lam, double* rr,
           double* rr_host, hipStream_t st) {
  if (n % Vec<T>::V) return fail(DWF_ERR_ARG, "16-bit fields need a multiple of 4 complex values");
  if (nrhs > 64) return fail(DWF_ERR_ARG, "nrhs > 64");
  hipLaunchKernelGGL((k_cg_r<T>), dim3(nblocks(n, nrhs), nrhs), dim3(kT), 0, st, r, p, w, n, alpha, lam, red, rr,
                     rr_host);
  LAUNCH_CHECK();
  return DWF_OK;
}
template <typename T>
int zero_t(T* y, size_t total, hipStream_t st) {
  if (total % Vec<T>::V) return fail(DWF_ERR_ARG, "16-bit fields need a multiple of 4 complex values");
  hipLaunchKernelGGL((k_zero<T>), dim3(nblocks(total)), dim3(kT), 0, st, y, total);
  LAUNCH_CHECK();
  return DWF_OK;
}

template <typename R>
int b_norm2(Red red, const cplx<R>* x, size_t n, int nrhs, double* res, hipStream_t st) {
  return norm2_t(red, x, n, nrhs, res, st);
}
template <typename R>
int b_dot(Red red, const cplx<R>* a, const cplx<R>* b, size_t n, int nrhs, double* res,
          hipStream_t st) {
  return dot_t(red, a, b, n, nrhs, res, st);
}
template <typename R>
int b_update(Red red, cplx<R>* x, cplx<R>* r, const cplx<R>* p, const cplx<R>* w, size_t n,
             int nrhs, const double* num, bool cnum, const double* den, const double* den2,
             double lam, double* rr, hipStream_t st, int dstr, int mode) {
  return update_t(red, x, r, p, w, n, nrhs, num, cnum, den, den2, lam, rr, st, dstr, mode);
}
template <typename R>
int b_xpay(Red red, cplx<R>* p, const cplx<R>* y, size_t n, int nrhs, const double* num, bool cnum,
           const double* den, double sign, double* pp, hipStream_t st, int dstr) {
  return xpay_t(red, p, y, n, nrhs, num, cnum, den, sign, pp, st, dstr);
}
int b_mirs16_init(Red red, bf16c* r, bf16c* p, const c64* b, size_t n, int nrhs, int Ls, double* rr,
                  hipStream_t st) {
  if (n % 12 || (n / 12) % Ls) return fail(DWF_ERR_ARG, "M_IRS: field size not a whole number of site rows");
  if (nrhs > 64) return fail(DWF_ERR_ARG, "nrhs > 64");
  hipLaunchKernelGGL(k_mirs16_init, dim3(nblocks(n, nrhs), nrhs), dim3(kT), 0, st, r, p, b, n / 12, Ls, red, rr);
  LAUNCH_CHECK();
  return DWF_OK;
}
int b_mirs16_last(c64* x_out, const bf16c* x, const bf16c* p, size_t n, int nrhs, int Ls, const double* num,
                  const double* den, const double* den2, double lam, hipStream_t st) {
  if (n % 12 || (n / 12) % Ls) return fail(DWF_ERR_ARG, "M_IRS: field size not a whole number of site rows");
  hipLaunchKernelGGL(k_mirs16_last, dim3(nblocks(n, nrhs), nrhs), dim3(kT), 0, st, x_out, x, p, n / 12, Ls, num, den,
                     den2, lam);
  LAUNCH_CHECK();
  return DWF_OK;
}
template <typename R>
int b_axpby(cplx<R>* y, const cplx<R>* x, double a, double b, size_t total, hipStream_t st) {
  hipLaunchKernelGGL((k_axpby<R>), dim3(nblocks(total)), dim3(kT), 0, st, y, x, (R)a, (R)b, total);
  LAUNCH_CHECK();
  return DWF_OK;
}
template <typename Ry, typename Rx>
int b_axpy_mixed(cplx<Ry>* y, const cplx<Rx>* x, const double* s, size_t n, int nrhs,
                 hipStream_t st, bool sqrt_s) {
  hipLaunchKernelGGL((k_axpy_mixed<Ry, Rx>), dim3(nblocks(n, nrhs), nrhs), dim3(kT), 0, st, y, x, s, n, sqrt_s);
  LAUNCH_CHECK();
  return DWF_OK;
}
template <typename Ry, typename Rx>
int b_scale_copy(cplx<Ry>* y, const cplx<Rx>* x, const double* v, bool invsqrt, size_t n, int nrhs,
                 hipStream_t st) {
  hipLaunchKernelGGL((k_scale_copy<Ry, Rx>), dim3(nblocks(n, nrhs), nrhs), dim3(kT), 0, st, y, x, v,
                     invsqrt, n);
  LAUNCH_CHECK();
  return DWF_OK;
}
template <typename R>
int b_zero(cplx<R>* y, size_t total, hipStream_t st) {
  return zero_t(y, total, st);
}

#define INST_CG(T)                                                                                                   \
  template int b_cg_xp<T>(Red, T*, T*, const T*, size_t, int, const double*, const double*, const double*, bool,      \
                          double*, hipStream_t);                                                                      \
  template int b_cg_r<T>(Red, T*, const T*, const T*, size_t, int, const double*, double, double*, double*,           \
                         hipStream_t);
INST_CG(c128)
INST_CG(c64)
INST_CG(bf16c)

#define INST(R)                                                                                   \
  template int b_norm2<R>(Red, const cplx<R>*, size_t, int, double*, hipStream_t);               \
  template int b_dot<R>(Red, const cplx<R>*, const cplx<R>*, size_t, int, double*, hipStream_t); \
  template int b_update<R>(Red, cplx<R>*, cplx<R>*, const cplx<R>*, const cplx<R>*, size_t, int, \
                           const double*, bool, const double*, const double*, double, double*,   \
                           hipStream_t, int, int);                                                \
  template int b_xpay<R>(Red, cplx<R>*, const cplx<R>*, size_t, int, const double*, bool,        \
                         const double*, double, double*, hipStream_t, int);                       \
  template int b_axpby<R>(cplx<R>*, const cplx<R>*, double, double, size_t, hipStream_t);        \
  template int b_zero<R>(cplx<R>*, size_t, hipStream_t);
INST(double)
INST(float)
template int b_axpy_mixed<double, float>(cplx<double>*, const cplx<float>*, const double*, size_t, int, hipStream_t, bool);
template int b_axpy_mixed<double, double>(cplx<double>*, const cplx<double>*, const double*, size_t, int, hipStream_t, bool);
template int b_axpy_mixed<float, float>(cplx<float>*, const cplx<float>*, const double*, size_t, int, hipStream_t, bool);
template int b_scale_copy<float, double>(cplx<float>*, const cplx<double>*, const double*, bool, size_t, int, hipStream_t);
template int b_scale_copy<double, float>(cplx<double>*, const cplx<float>*, const double*, bool, size_t, int, hipStream_t);
template int b_scale_copy<double, double>(cplx<double>*, const cplx<double>*, const double*, bool, size_t, int, hipStream_t);
template int b_scale_copy<float, float>(cplx<float>*, const cplx<float>*, const double*, bool, size_t, int, hipStream_t);

}  // namespace hdk
