// The hop stage for Ls <= 16, split over the four 16-lane rows of a wave.
//
// One wave owns the fifth-dimension column of one output site (Ls 9..16), or
// of floor(16 / Ls) sites: lane 16 row + j holds slice s = j mod Ls of the
// (j / Ls)-th of them, and the four rows share the work on it.  Row bit 0 is
// the upper spin component sp whose projection h_sp = u_sp + g A l a lane
// forms (the two components of a projected half-spinor go through the link
// independently), row bit 1 selects the directions x, y or z, t.  With
// A_x, A_z imaginary and A_y, A_t real, all rows run the same instructions;
// the rows differ only in the offset of the lower component they read
// (l_{1-sp} for x, y and l_sp for z, t), in the sign g, and in the links
// they read from LDS.  A lane loads six of a neighbour's twelve components
// for four of its eight directions: 24 loads, all issued before any
// arithmetic, as many bytes in flight as two whole spinors.
//
// The rows' sums U (upper sp) and L (lower l) are reduced and scattered with
// gfx950's row swaps, so that row 0 ends with spin 0, row 1 with spin 3, row
// 2 with spin 1 and row 3 with spin 2, three colours each: no LDS, no
// barrier.  The fifth-dimension factors are DPP shifts along j: the
// recurrence of M_5^-1 is a scan of log2(Ls) steps and one step more.
#pragma once

#include "hop_dev.h"

namespace hdk {

// The arithmetic of a stage is written with explicit fused multiply-adds, and
// the compiler forms no others in the functions that begin with this: every
// kernel they are part of (split or marched, one or several right-hand sides,
// any launch shape) gives the same bits.
#define HDCG_PINNED _Pragma("clang fp contract(off)")

constexpr int kDppShl = 0x100, kDppShr = 0x110, kDppRor = 0x120;
constexpr int kRowsUp = 0x5, kRowsDn = 0xa;  // rows that end with upper (P+) and lower (P-) spins

// lanes of the rows in MA take x shifted by DPP control CA, the other rows by
// CB; lanes shifted in from outside the row are 0 (the first shift writes all
// rows: no register to clear for the masked ones)
template <int CA, int CB, int MA>
__device__ __forceinline__ unsigned dpp_rows(unsigned x) {
  const int r = __builtin_amdgcn_mov_dpp((int)x, CA, 0xf, 0xf, true);
  return (unsigned)__builtin_amdgcn_update_dpp(r, (int)x, CB, 0xf ^ MA, 0xf, true);
}
template <int CA, int CB, int MA>
__device__ __forceinline__ float dpp_rows(float x) {
  return __uint_as_float(dpp_rows<CA, CB, MA>(__float_as_uint(x)));
}
template <int CA, int CB, int MA>
__device__ __forceinline__ double dpp_rows(double x) {
  const unsigned lo = dpp_rows<CA, CB, MA>((unsigned)__double2loint(x));
  const unsigned hi = dpp_rows<CA, CB, MA>((unsigned)__double2hiint(x));
  return __hiloint2double((int)hi, (int)lo);
}
__device__ __forceinline__ float lane_get(float x, int lane) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute(lane << 2, __float_as_int(x)));
}
__device__ __forceinline__ double lane_get(double x, int lane) {
  const int lo = __builtin_amdgcn_ds_bpermute(lane << 2, __double2loint(x));
  const int hi = __builtin_amdgcn_ds_bpermute(lane << 2, __double2hiint(x));
  return __hiloint2double(hi, lo);
}

// u: a row's part of its upper spin (rows 0..3: spins 0 1 0 1), l: of its
// lower one (3 2 2 3).  After the 16-lane swap u, l are (0 3 0 2), (1 2 1 3);
// with row 3's two exchanged, the 32-lane swap pairs equal spins, and the sum
// is spin 0, 3, 1, 2 in rows 0..3.
__device__ __forceinline__ void row_pair(unsigned& u, unsigned& l, bool row3) {
  const auto a = __builtin_amdgcn_permlane16_swap(u, l, false, false);
  const unsigned p = row3 ? a[1] : a[0], q = row3 ? a[0] : a[1];
  const auto b = __builtin_amdgcn_permlane32_swap(p, q, false, false);
  u = b[0];
  l = b[1];
}
__device__ __forceinline__ float row_reduce(float u, float l, bool row3) {
  unsigned a = __float_as_uint(u), b = __float_as_uint(l);
  row_pair(a, b, row3);
  return __uint_as_float(a) + __uint_as_float(b);
}
__device__ __forceinline__ double row_reduce(double u, double l, bool row3) {
  unsigned a0 = (unsigned)__double2loint(u), b0 = (unsigned)__double2loint(l);
  unsigned a1 = (unsigned)__double2hiint(u), b1 = (unsigned)__double2hiint(l);
  row_pair(a0, b0, row3);
  row_pair(a1, b1, row3);
  return __hiloint2double((int)a1, (int)a0) + __hiloint2double((int)b1, (int)b0);
}

// A load that is not expected to be used again (links, centre values).
template <typename T>
__device__ __forceinline__ T ld_once(const T* p) {
  typedef unsigned V __attribute__((ext_vector_type(sizeof(T) / 4)));
  const V w = __builtin_nontemporal_load(reinterpret_cast<const V*>(p));
  T t;
  __builtin_memcpy(&t, &w, sizeof(T));
  return t;
}

// Three consecutive components (one spin) of a column, as stored.
template <typename T>
struct Tri {
  T v[3];
  using R = typename St<T>::R;
  __device__ __forceinline__ void ld(const T* p, int stride) {
#pragma unroll
    for (int c = 0; c < 3; ++c) v[c] = p[c * stride];
  }
  __device__ __forceinline__ void ld1(const T* p, int stride) {
#pragma unroll
    for (int c = 0; c < 3; ++c) v[c] = ld_once(p + c * stride);
  }
  __device__ __forceinline__ cplx<R> get(int c) const { return v[c]; }
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int c = 0; c < 3; ++c) v[c] = cmk((R)0, (R)0);
  }
  __device__ __forceinline__ void take(bool other, const Tri& o) {
#pragma unroll
    for (int c = 0; c < 3; ++c) v[c] = cmk(other ? o.v[c].re : v[c].re, other ? o.v[c].im : v[c].im);
  }
};
template <>
struct Tri<bf16c> {
  unsigned v[3];
  __device__ __forceinline__ void ld(const bf16c* p, int) { __builtin_memcpy(v, p, 12); }
  __device__ __forceinline__ void ld1(const bf16c* p, int) { __builtin_memcpy(v, p, 12); }
  __device__ __forceinline__ cplx<float> get(int c) const { return bf16_word(v[c]); }
  __device__ __forceinline__ void zero() { v[0] = v[1] = v[2] = 0; }
  __device__ __forceinline__ void take(bool other, const Tri& o) {
#pragma unroll
    for (int c = 0; c < 3; ++c) v[c] = other ? o.v[c] : v[c];
  }
};
template <typename T>
__device__ __forceinline__ void tri_st(T* p, int stride, const cplx<typename St<T>::R> (&v)[3], bool nt) {
  if constexpr (kSMajor<T>) {
    unsigned w[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) w[c] = bf16_pack(v[c]);
    if (nt) {
#pragma unroll
      for (int c = 0; c < 3; ++c) __builtin_nontemporal_store(w[c], reinterpret_cast<unsigned*>(p) + c);
    } else {
      __builtin_memcpy(p, w, 12);
    }
  } else {
#pragma unroll
    for (int c = 0; c < 3; ++c) store_field(p + c * stride, v[c], nt);
  }
}

template <typename T>
__device__ __forceinline__ cplx<typename St<T>::R> tri_get(const Tri<T>& t, int c) {
  return t.get(c);
}
template <typename R>
__device__ __forceinline__ cplx<R> tri_get(const cplx<R> (&t)[3], int c) {
  return t[c];
}
// One direction of this row: KIND 0 imaginary A (x, z), 1 real (y, t); g the
// signed coefficient; h = u + g A l, U += W h, L += g A^+ W h (FIRST: U =, L =).
template <int KIND, bool FIRST = false, typename R, typename V>
__device__ __forceinline__ void split_dir(cplx<R> (&U)[3], cplx<R> (&L)[3], const V& u, const V& l,
                                          const cplx<R>* __restrict__ w, R g) {
  HDCG_PINNED
  cplx<R> h[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const cplx<R> a = tri_get(u, c), b = tri_get(l, c);
    h[c] = KIND == 0 ? cmk(fma(g, b.im, a.re), fma(-g, b.re, a.im)) : cmk(fma(g, b.re, a.re), fma(g, b.im, a.im));
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const cplx<R> w0 = w[a * 3 + 0], w1 = w[a * 3 + 1], w2 = w[a * 3 + 2];
    cplx<R> t = cmk(fma(-w0.im, h[0].im, w0.re * h[0].re), fma(w0.im, h[0].re, w0.re * h[0].im));
    cmac(t, w1, h[1]);
    cmac(t, w2, h[2]);
    if (FIRST) {
      U[a] = t;
      L[a] = KIND == 0 ? cmk(-g * t.im, g * t.re) : cmk(g * t.re, g * t.im);
      continue;
    }
    U[a].re += t.re;
    U[a].im += t.im;
    if (KIND == 0) {
      L[a].re = fma(-g, t.im, L[a].re);
      L[a].im = fma(g, t.re, L[a].im);
    } else {
      L[a].re = fma(g, t.re, L[a].re);
      L[a].im = fma(g, t.im, L[a].im);
    }
  }
}

// b x + c y
template <typename R>
__device__ __forceinline__ cplx<R> split_c5(R b, cplx<R> x, R c, cplx<R> y) {
  HDCG_PINNED
  return cmk(fma(b, x.re, c * y.re), fma(b, x.im, c * y.im));
}

// Where a lane stands in its wave.
struct SplitLane {
  int row, sub, s, spin;
  bool upper;  // ends with a P+ spin
};

// x[c] at slice s + 1 (rows MUP) or s - 1 (the other rows) of the same site,
// wrapping round the Ls slices
template <int LS, int MUP, typename R>
__device__ __forceinline__ R s_shift(R x, int src_lane) {
  if constexpr (LS == 16) return dpp_rows<kDppRor + 15, kDppRor + 1, MUP>(x);
  return lane_get(x, src_lane);
}

// v <- (b + c S) v, S taking s + 1 in the rows MUP and s - 1 in the others,
// -m times the wrapped entry at the wall
template <int LS, int MUP, typename R>
__device__ __forceinline__ void split_bcs(cplx<R> (&v)[3], const SplitLane& q, int Ls, R b, R c, R m) {
  HDCG_PINNED
  const bool up = (MUP >> q.row) & 1;
  const int sn = up ? (q.s + 1 < Ls ? q.s + 1 : 0) : (q.s > 0 ? q.s - 1 : Ls - 1);
  const R w = (up ? q.s + 1 < Ls : q.s > 0) ? c : -m * c;
  const int lane = q.row * 16 + q.sub * Ls + sn;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    v[k].re = fma(b, v[k].re, w * s_shift<LS, MUP>(v[k].re, lane));
    v[k].im = fma(b, v[k].im, w * s_shift<LS, MUP>(v[k].im, lane));
  }
}

// One step of the scan of M_5^-1: t += kap^K * (t K slices earlier in the
// row's chain), the chain ascending in s in the rows MLOW
template <int MLOW, int K, typename R>
__device__ __forceinline__ void split_scan(cplx<R> (&t)[3], R kapk, int pos) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const R re = dpp_rows<kDppShr + K, kDppShl + K, MLOW>(t[k].re);
    const R im = dpp_rows<kDppShr + K, kDppShl + K, MLOW>(t[k].im);
    // the chain starts inside the row
    t[k].re = fma(kapk, pos >= K ? re : (R)0, t[k].re);
    t[k].im = fma(kapk, pos >= K ? im : (R)0, t[k].im);
  }
}
// ... and with Ls = 16, round the row: o += kapk * (t K slices earlier)
template <int MLOW, int K, typename R>
__device__ __forceinline__ void split_turn(cplx<R> (&o)[3], const cplx<R> (&t)[3], R kapk) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    o[k].re = fma(kapk, dpp_rows<kDppRor + K, kDppRor + 16 - K, MLOW>(t[k].re), o[k].re);
    o[k].im = fma(kapk, dpp_rows<kDppRor + K, kDppRor + 16 - K, MLOW>(t[k].im), o[k].im);
  }
}

// The coefficients of split_m5inv for this lane.
template <typename R>
struct InvCoef {
  R k[4];  // of the scan's steps
  R last;  // of its last one
};
template <int LS, int MLOW, bool LAST, typename R>
__device__ __forceinline__ InvCoef<R> split_inv_coef(const SplitLane& q, int Ls, const HopArgs& A,
                                                     const R* __restrict__ pw) {
  const int pos = ((MLOW >> q.row) & 1) ? q.s : Ls - 1 - q.s;
  InvCoef<R> c;
  if constexpr (LS == 16) {
    const R m = (R)A.mass;
#pragma unroll
    for (int i = 0; i < 4; ++i) c.k[i] = pos < (1 << i) ? -m * (R)A.kp[i] : (R)A.kp[i];
    c.last = !LAST ? pw[0] : pos < 1 ? -m * (R)A.kc : (R)A.kc;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) c.k[i] = (R)A.kp[i];
    c.last = -(R)(A.mass * A.alpha * (LAST ? 1.0 : A.kap)) * pw[pos];
  }
  return c;
}

// split_m5inv's steps for six FP32 values at Ls = 16: two row-masked
// v_fmac_f32_dpp a value and step (the rows of each chain direction) instead
// of two moves and a multiply-add.  A value is read by DPP at least five
// instructions after it was written (two wait states are needed, which the
// compiler does not insert around inline assembly: hence the nops at both
// ends, the second for a reader of the results that is a DPP move).
#define HDCG_FMAC(D, S, COEF, CTRL, MASK) \
  "v_fmac_f32_dpp %" #D ", %" #S ", %" #COEF " " CTRL " row_mask:" MASK " bank_mask:0xf\n\t"
#define HDCG_STEP(COEF, CTRL, MASK)                                                                        \
  HDCG_FMAC(0, 0, COEF, CTRL, MASK) HDCG_FMAC(1, 1, COEF, CTRL, MASK) HDCG_FMAC(2, 2, COEF, CTRL, MASK)     \
      HDCG_FMAC(3, 3, COEF, CTRL, MASK) HDCG_FMAC(4, 4, COEF, CTRL, MASK) HDCG_FMAC(5, 5, COEF, CTRL, MASK)
#define HDCG_LAST(COEF, CTRL, MASK)                                                                        \
  HDCG_FMAC(6, 0, COEF, CTRL, MASK) HDCG_FMAC(7, 1, COEF, CTRL, MASK) HDCG_FMAC(8, 2, COEF, CTRL, MASK)     \
      HDCG_FMAC(9, 3, COEF, CTRL, MASK) HDCG_FMAC(10, 4, COEF, CTRL, MASK) HDCG_FMAC(11, 5, COEF, CTRL, MASK)
#define HDCG_SCAN16(A, B, C, D, LO, HI)                                                                    \
  "s_nop 1\n\t" HDCG_STEP(A, "row_ror:1", LO) HDCG_STEP(A, "row_ror:15", HI) HDCG_STEP(B, "row_ror:2", LO) \
      HDCG_STEP(B, "row_ror:14", HI) HDCG_STEP(C, "row_ror:4", LO) HDCG_STEP(C, "row_ror:12", HI)           \
          HDCG_STEP(D, "row_ror:8", LO) HDCG_STEP(D, "row_ror:8", HI)
#define HDCG_SIX(t) "+v"(t[0].re), "+v"(t[0].im), "+v"(t[1].re), "+v"(t[1].im), "+v"(t[2].re), "+v"(t[2].im)
template <int MLOW>
__device__ __forceinline__ void split_scan16(cplx<float> (&x)[3], const InvCoef<float>& k) {
#define HDCG_ASM(LO, HI)                               \
  asm(HDCG_SCAN16(6, 7, 8, 9, LO, HI) "s_nop 1"        \
      : HDCG_SIX(x)                                    \
      : "v"(k.k[0]), "v"(k.k[1]), "v"(k.k[2]), "v"(k.k[3]))
  if (MLOW == kRowsUp)
    HDCG_ASM("0x5", "0xa");
  else
    HDCG_ASM("0xa", "0x5");
#undef HDCG_ASM
}
template <int MLOW>
__device__ __forceinline__ void split_inv16(cplx<float> (&x)[3], const InvCoef<float>& k) {
  cplx<float> t[3] = {x[0], x[1], x[2]};
#define HDCG_ASM(LO, HI)                                                                                        \
  asm(HDCG_SCAN16(12, 13, 14, 15, LO, HI) HDCG_LAST(16, "row_ror:1", LO) HDCG_LAST(16, "row_ror:15", HI) "s_nop 1" \
      : HDCG_SIX(t), HDCG_SIX(x)                                                                                \
      : "v"(k.k[0]), "v"(k.k[1]), "v"(k.k[2]), "v"(k.k[3]), "v"(k.last))
  if (MLOW == kRowsUp)
    HDCG_ASM("0x5", "0xa");
  else
    HDCG_ASM("0xa", "0x5");
#undef HDCG_ASM
}
#undef HDCG_SIX
#undef HDCG_SCAN16
#undef HDCG_LAST
#undef HDCG_STEP
#undef HDCG_FMAC

// x <- alpha M_5^-1 x (rows MLOW: ascending in s): y = x + kap S y, S the
// shift along the row's chain with -mass at the wall.  The factor 1 / alpha is
// left to the stage that reads the result (HopArgs::qia).
//
// A scan gives y up to its own roundings, log2(Ls) of the size of y; one more
// step of the equation, from x itself, leaves one rounding of that size and
// damps the others by kap.  Without it M_5^-1 had 1.5 times the rounding error
// of the O(Ls) recurrence (FP32, Ls 16: 5.6e-8 against 3.7e-8 or 2.9e-8 with
// either choice of fused multiply-adds; with it 2.9e-8).  H against 64 bits,
// recurrence, scan alone, with the step: complex64 on 8^3 x 16 x 16 8.00e-8,
// 8.08e-8, 7.69e-8; complex128 on 16^4 x 16 1.910e-16, 1.952e-16, 1.902e-16.
//   Ls = 16: shifts round the whole row, t = (1 + k S)(1 + k^2 S^2) ... x
//     = (1 + mass kap^16) y, and y = x + kap / (1 + mass kap^16) S t;
//   else: z from z_{-1} = 0, and with c_s = mass kap^s / (1 + mass kap^Ls)
//     y_s = x_s + kap (z_{s-1} - c_s z_{Ls-1}).
// LAST = false: x <- M_5^-1 x without that step, for fields that are rounded
// to 16 bits next (2^-8 against a few 2^-24).
template <int LS, int MLOW, bool LAST, typename R>
__device__ __forceinline__ void split_m5inv(cplx<R> (&x)[3], const SplitLane& q, int Ls, const InvCoef<R>& k, R ia) {
  HDCG_PINNED
  if constexpr (!LAST) {
    const R f = LS == 16 ? k.last : ia;
#pragma unroll
    for (int c = 0; c < 3; ++c) x[c] = cmk(f * x[c].re, f * x[c].im);
  }
  if constexpr (LS == 16 && sizeof(R) == 4) {
    if constexpr (LAST) split_inv16<MLOW>(x, k);
    else split_scan16<MLOW>(x, k);
  } else if constexpr (LS == 16) {
    static_assert(LAST, "16-bit fields compute in FP32");
    cplx<R> t[3] = {x[0], x[1], x[2]};
    split_turn<MLOW, 1>(t, t, k.k[0]);
    split_turn<MLOW, 2>(t, t, k.k[1]);
    split_turn<MLOW, 4>(t, t, k.k[2]);
    split_turn<MLOW, 8>(t, t, k.k[3]);
    split_turn<MLOW, 1>(x, t, k.last);
  } else {
    const bool low = (MLOW >> q.row) & 1;
    const int pos = low ? q.s : Ls - 1 - q.s;
    cplx<R> t[3] = {x[0], x[1], x[2]};
    if (Ls > 1) split_scan<MLOW, 1>(t, k.k[0], pos);
    if (Ls > 2) split_scan<MLOW, 2>(t, k.k[1], pos);
    if (Ls > 4) split_scan<MLOW, 4>(t, k.k[2], pos);
    if (Ls > 8) split_scan<MLOW, 8>(t, k.k[3], pos);
    const int last = q.row * 16 + q.sub * Ls + (low ? Ls - 1 : 0);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const R re = lane_get(t[c].re, last), im = lane_get(t[c].im, last);
      if constexpr (LAST) {
        const R pre = dpp_rows<kDppShr + 1, kDppShl + 1, MLOW>(t[c].re);
        const R pim = dpp_rows<kDppShr + 1, kDppShl + 1, MLOW>(t[c].im);
        x[c].re = fma(k.k[0], fma(k.last, re, pos >= 1 ? pre : (R)0), x[c].re);
        x[c].im = fma(k.k[0], fma(k.last, im, pos >= 1 ? pim : (R)0), x[c].im);
      } else {
        x[c] = cmk(fma(k.last, re, t[c].re), fma(k.last, im, t[c].im));
      }
    }
  }
}

// The row's spin of the stage's output from the rows' parts U, L of the hop:
// reduction over the rows, then the fifth-dimension factors (inv: M_5^-1's
// coefficients, EPI_INV; cx, cy: the centre field at s and at the slice M_5
// couples it to, the other stages, whose input is alpha times M_5^-1's result
// but for 16-bit fields).
template <typename R, bool DAG, int EPI, int LS, bool MOB, typename T>
__device__ __forceinline__ void split_finish(cplx<R> (&acc)[3], const cplx<R> (&U)[3], const cplx<R> (&L)[3],
                                             const Tri<T>& cx, const Tri<T>& cy, const SplitLane& q, int Ls,
                                             const HopArgs& A, const InvCoef<R>& inv) {
  HDCG_PINNED
  const bool row3 = q.row == 3;
#pragma unroll
  for (int k = 0; k < 3; ++k)
    acc[k] = cmk(row_reduce(U[k].re, L[k].re, row3), row_reduce(U[k].im, L[k].im, row3));
  // Mobius, adjoint chain: C_5^+ = b5 + c5 K^+ on the hop result first
  // (P+ from s+1, P- from s-1)
  if (MOB && DAG) split_bcs<LS, kRowsUp>(acc, q, Ls, (R)A.b5, (R)A.c5, (R)A.mass);
  if (EPI == EPI_INV) {
    split_m5inv<LS, DAG ? kRowsDn : kRowsUp, !kSMajor<T>>(acc, q, Ls, inv, (R)A.ia);
    // Mobius: C_5 after M_5^-1, for the second hop (P+ from s-1, P- from s+1)
    if (MOB && !DAG) split_bcs<LS, kRowsDn>(acc, q, Ls, (R)A.b5, (R)A.c5, (R)A.mass);
  } else {
    // M_5 couples P+ to s-1 and P- to s+1; the adjoint swaps the two
    const R al = (R)A.alpha, be = (R)A.beta, m = (R)A.mass, qu = kSMajor<T> ? (R)0.25 : (R)A.qia;
    const bool wall = (q.upper != DAG) ? q.s == 0 : q.s == Ls - 1;
    const R f = wall ? -m * be : be;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      // FP32: the largest term last, the product that is exact in Shamir's M_5
      // (beta = -1) as the plain one: two roundings, one of them small (H
      // against 64 bits 7.74e-8 -> 7.29e-8).  FP64 keeps the order of the
      // definition, M_5 c first: a 64-bit reference has the same roundings there.
      const cplx<R> x = cx.get(k), y = cy.get(k);
      if constexpr (sizeof(R) == 4)
        acc[k] = cmk(fma(al, x.re, fma(-qu, acc[k].re, f * y.re)), fma(al, x.im, fma(-qu, acc[k].im, f * y.im)));
      else
        acc[k] = cmk(fma(-qu, acc[k].re, fma(al, x.re, f * y.re)), fma(-qu, acc[k].im, fma(al, x.im, f * y.im)));
    }
  }
}

// acc <- r - a (acc + lam p): the residual of a CG step from w = acc
template <typename R, typename T>
__device__ __forceinline__ void split_residual(cplx<R> (&acc)[3], const Tri<T>& r, const Tri<T>& p, const HopArgs& A,
                                               int rhs) {
  HDCG_PINNED
  const R a = (R)A.cg_alpha[rhs], l = (R)A.cg_lam;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    if (A.cg_p) {
      const cplx<R> v = p.get(k);
      acc[k] = cmk(fma(l, v.re, acc[k].re), fma(l, v.im, acc[k].im));
    }
    const cplx<R> v = r.get(k);
    acc[k] = cmk(fma(-a, acc[k].re, v.re), fma(-a, acc[k].im, v.im));
  }
}

// The norm of one right-hand side, finished by the grid's last workgroup in a
// fixed order (sum: the workgroup's, in thread 0)
__device__ __forceinline__ void split_norm(double sum, const HopArgs& A, int rhs, int wg) {
  __shared__ int last;
  __shared__ double lds[16];
  double* part = A.partials + (size_t)rhs * A.pstride;
  if (threadIdx.x == 0) {
    __hip_atomic_store(part + wg, sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_s_waitcnt(0);
    last = last_ticket(A.counters, rhs, gridDim.x, blockIdx.x);
  }
  __syncthreads();
  if (!last) return;
  double s[1] = {0.0};
  const int G = (int)gridDim.x, B = (int)blockDim.x;
  for (int i0 = threadIdx.x; i0 < G; i0 += 4 * B) {
    double a[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      a[u] = i0 + u * B < G ? __hip_atomic_load(part + i0 + u * B, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.0;
#pragma unroll
    for (int u = 0; u < 4; ++u) s[0] += a[u];
  }
  block_sum<1>(s, lds);
  if (threadIdx.x == 0) fin_store(s[0], rhs, A.result, A.fin);
}

// LS > 0 fixes Ls at compile time.  LOOP: a wave takes several sites of the
// workgroup's block and several right-hand sides one after another (else
// exactly one of each).  Dynamic LDS: spw * kLinkLd complex.
template <typename R, bool DAG, int EPI, int LS, bool MOB, typename T, bool LOOP>
__global__ void __launch_bounds__(sizeof(R) == 8 ? 256 : 1024)
hop_split_kernel(T* __restrict__ out, const T* __restrict__ in, const T* __restrict__ center,
                 const cplx<R>* __restrict__ gauge, const R* __restrict__ pw, HopArgs A) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const Geom& g = A.g;
  const int Ls = LS > 0 ? LS : g.Ls;
  const int NS = 16 / Ls;  // sites per wave
  const int wg = (A.remap && !A.order) ? xcd_remap(blockIdx.x, gridDim.x) : (int)blockIdx.x;
  const int rhs0 = blockIdx.y * A.rg;
  const int nr = LOOP ? min(A.rg, A.nrhs - rhs0) : 1;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  SplitLane q;
  q.row = lane >> 4;
  const int j = lane & 15;
  q.sub = LS == 16 ? 0 : j / Ls;
  q.s = j - q.sub * Ls;
  q.spin = q.row == 0 ? 0 : q.row == 1 ? 3 : q.row == 2 ? 1 : 2;
  q.upper = !(q.row & 1);
  const int sp = q.row & 1, zt = q.row >> 1;
  const int lsp = zt ? sp : 1 - sp;
  constexpr bool NT = sizeof(R) == 8;  // non-temporal loads are chosen in complex128 only
  constexpr R SF = DAG ? (R)1 : (R)-1;
  // signs of A on this row: x +, z (+, -); y (-, +), t +
  const R g0 = (zt && sp) ? -SF : SF, g1 = (!zt && !sp) ? -SF : SF;
  const size_t col = (size_t)12 * Ls;
  // Mobius: the first stage of M_pc hops C_5 in
  constexpr bool C5IN = MOB && !DAG && EPI == EPI_INV;
  const bool lane_in = LS == 16 || q.sub < NS;

  // this wave's links in LDS: wave-private rows, written and read by the
  // same wave (LDS operations of one wave complete in order)
  cplx<R>* links = reinterpret_cast<cplx<R>*>(smem_raw);  // [spw][kLinkLd]
  const int per = NS * nw;                                // sites of one pass of the workgroup
  const int passes = LOOP ? (A.spw + per - 1) / per : 1;
  constexpr int NL = LS > 0 ? (72 + 4 * LS - 1) / (4 * LS) : 1;
  const int e0 = q.row * Ls + q.s;

  InvCoef<R> inv;
  if (EPI == EPI_INV) inv = split_inv_coef<LS, DAG ? kRowsDn : kRowsUp, !kSMajor<T>>(q, Ls, A, pw);
  for (int rr = 0; rr < nr; ++rr) {
    const int rhs = rhs0 + rr;
    const T* __restrict__ inr = in + rhs * A.field;
    double nrm = 0.0;
    for (int pass = 0; pass < passes; ++pass) {
      const int first = (pass * nw + wave) * NS;
      const int want = LS > 8 ? first : first + q.sub;
      const bool valid = want < A.spw && (A.bx > 0 || wg * A.spw + want < g.Vh);
      if (LS > 8 && !valid) continue;  // the same for the whole wave
      // lanes without a site or slice of their own repeat the work of
      // another (all loads in range) and store nothing
      const bool active = valid && lane_in;
      const int vloc = LS > 8 || active ? want : 0;
      Site c;
      const int v = hop_site(A, wg, vloc, c);
      Tri<T> u[4], l[4], cx, cy, rv, pv;
      Tri<T> us[C5IN ? 4 : 1], ls[C5IN ? 4 : 1];
      const int s_dn = q.s > 0 ? q.s - 1 : Ls - 1, s_up = q.s + 1 < Ls ? q.s + 1 : 0;
      cplx<R> lk[NL];
      cplx<R>* myl = links + (size_t)vloc * kLinkLd;
      {
        const cplx<R>* G = gauge + (size_t)v * 72;
        if constexpr (LS > 0) {
          if (!LOOP || rr == 0) {
#pragma unroll
            for (int k = 0; k < NL; ++k) lk[k] = NT && A.nt & 2 ? ld_once(G + min(e0 + k * 4 * LS, 71)) : G[min(e0 + k * 4 * LS, 71)];
          }
        } else {
          if (!LOOP || rr == 0)
            for (int e = e0; e < 72; e += 4 * Ls) myl[e] = G[e];
        }
        int nb[8];
        hop_neighbours(g, c, nb);
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          const T* p = inr + (size_t)(zt ? nb[4 + d] : nb[d]) * col;
          if constexpr (kSMajor<T>) {
            u[d].ld(p + q.s * 12 + sp * 3, 1);
            l[d].ld(p + q.s * 12 + 6 + lsp * 3, 1);
            if constexpr (C5IN) {
              us[d].ld(p + s_dn * 12 + sp * 3, 1);
              ls[d].ld(p + s_up * 12 + 6 + lsp * 3, 1);
            }
          } else {
            u[d].ld(p + sp * 3 * Ls + q.s, Ls);
            l[d].ld(p + (6 + lsp * 3) * Ls + q.s, Ls);
            if constexpr (C5IN) {
              us[d].ld(p + sp * 3 * Ls + s_dn, Ls);
              ls[d].ld(p + (6 + lsp * 3) * Ls + s_up, Ls);
            }
          }
        }
        if (EPI != EPI_INV) {
          const T* cen = center + rhs * A.field + (size_t)v * col;
          const int sn = (q.upper != DAG) ? s_dn : s_up;
          if constexpr (kSMajor<T>) {
            cx.ld(cen + q.s * 12 + q.spin * 3, 1);
            cy.ld(cen + sn * 12 + q.spin * 3, 1);
          } else {
            if (NT && A.nt & 4) cx.ld1(cen + q.spin * 3 * Ls + q.s, Ls); else cx.ld(cen + q.spin * 3 * Ls + q.s, Ls);
            if (NT && A.nt & 4) cy.ld1(cen + q.spin * 3 * Ls + sn, Ls); else cy.ld(cen + q.spin * 3 * Ls + sn, Ls);
          }
        }
        if (EPI == EPI_RES) {
          const size_t at = rhs * A.field + (size_t)v * col + (kSMajor<T> ? q.s * 12 + q.spin * 3 : q.spin * 3 * Ls + q.s);
          rv.ld(out + at, Ls);
          if (A.cg_p) pv.ld(static_cast<const T*>(A.cg_p) + at, Ls);
        }
        if constexpr (LS > 0) {
          if (!LOOP || rr == 0) {
#pragma unroll
            for (int k = 0; k < NL; ++k)
              if (e0 + k * 4 * LS < 72) myl[e0 + k * 4 * LS] = lk[k];
          }
        }
      }
      __builtin_amdgcn_wave_barrier();
      cplx<R> U[3], L[3];
      {
        const cplx<R>* W = myl + (zt ? 18 : 0);
        if constexpr (C5IN) {
          // C_5 = b5 + c5 K on the neighbours: P+ (u) from s-1, P- (l) from
          // s+1, -mass at the wrap
          const R b5 = (R)A.b5, c5 = (R)A.c5, m = (R)A.mass;
          const R wu = q.s > 0 ? c5 : -m * c5, wl = q.s + 1 < Ls ? c5 : -m * c5;
          cplx<R> a[4][3], b[4][3];
#pragma unroll
          for (int d = 0; d < 4; ++d)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
              a[d][k] = split_c5(b5, u[d].get(k), wu, us[d].get(k));
              b[d][k] = split_c5(b5, l[d].get(k), wl, ls[d].get(k));
            }
          split_dir<0, true>(U, L, a[0], b[0], W, g0);
          split_dir<0>(U, L, a[1], b[1], W + 36, -g0);
          split_dir<1>(U, L, a[2], b[2], W + 9, g1);
          split_dir<1>(U, L, a[3], b[3], W + 45, -g1);
        } else {
          split_dir<0, true>(U, L, u[0], l[0], W, g0);
          split_dir<0>(U, L, u[1], l[1], W + 36, -g0);
          split_dir<1>(U, L, u[2], l[2], W + 9, g1);
          split_dir<1>(U, L, u[3], l[3], W + 45, -g1);
        }
      }
      cplx<R> acc[3];
      split_finish<R, DAG, EPI, LS, MOB>(acc, U, L, cx, cy, q, Ls, A, inv);
      if (EPI == EPI_RES) split_residual<R, T>(acc, rv, pv, A, rhs);
      if (EPI != EPI_INV && A.partials && active) {
#pragma unroll
        for (int k = 0; k < 3; ++k)
          nrm = fma((double)acc[k].im, (double)acc[k].im, fma((double)acc[k].re, (double)acc[k].re, nrm));
      }
      if (active) {
        T* o = out + rhs * A.field + (size_t)v * col;
        if constexpr (kSMajor<T>)
          tri_st<T>(o + q.s * 12 + q.spin * 3, 1, acc, A.nt & 1);
        else
          tri_st<T>(o + q.spin * 3 * Ls + q.s, Ls, acc, A.nt & 1);
      }
    }
    if (EPI != EPI_INV && A.partials) {
      double vv[1] = {nrm};
      __shared__ double red[2][16];  // two: a wave may be one right-hand side ahead of thread 0
      block_sum<1>(vv, red[rr & 1]);
      if (A.counters)
        split_norm(vv[0], A, rhs, wg);
      else
        store_partial<1>(vv, A.partials + (size_t)rhs * A.pstride, 0, wg);
    }
  }
}

}  // namespace hdk
