// The hop stage marched along t with the input columns in LDS (Shamir,
// Ls = 8, 12 or 16, complex64 and complex128).
//
// hop_split_kernel reads each input column from the caches by up to eight
// waves: on 24^3 x 48 x 16 in complex64 H takes 1.87 ms with the real
// neighbours, 1.59 ms when every neighbour column is in L2 and 1.12 ms when
// it is in L1, so a quarter of the time is the traffic between L2 and L1.
// Here a workgroup owns a tile of bx x by x bz pairs of real sites (2 xh, 2 xh
// + 1) and marches over bt planes of t.  On every plane one site of a pair is
// an output site and the other an input site, with the same checkerboard
// index, so each wave (pair) loads one input column per plane, and three
// planes of the tile's columns sit in LDS: of an output's eight neighbours
// the pair's own column serves x, t - 1 and t + 1, the tile's other columns
// serve those inside it, and only the neighbours across the tile's faces are
// loaded from memory (for 2 x 4 x 2 pairs three columns per output instead of
// eight).  The next plane's column, links, face neighbours and centre values
// are loaded while this plane is computed; one barrier per plane.
//
// Lanes and arithmetic are hop_split_kernel's: the results are the same, bit
// for bit.
//
// What bounds it now: in complex64 the vector units (600 instructions a site
// and plane, 4 waves a SIMD) as much as HBM; a workgroup's 16 waves fill a
// CU, so a short march pays its three-plane start-up (16^4: slower than the
// split form).  H, split against marching: complex64 24^3 x 48 x 16 1.87 and
// 1.66 ms, 32^3 x 64 x 16 5.95 and 4.65 ms (5.0 TB/s of algorithmic bytes);
// complex128 24^3 x 48 x 16 3.26 and 3.02 ms, 16^4 x 16 282 and 270 us.
// 16-bit fields, half the bytes for the same instructions, have no marched
// form: 1.02 and 1.01 ms on 24^3 x 48, 8 right-hand sides on 16^3 x 32 1.53
// and 1.55 ms.
#pragma once

#include "hop_split.h"

namespace hdk {

// barrier that orders LDS only: the loads in flight for the next plane stay
// in flight across it
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Keeps a direction's arithmetic in place: otherwise it is moved behind the
// next plane's loads, with all its operands in registers.
template <typename R>
__device__ __forceinline__ void march_pin(cplx<R> (&U)[3], cplx<R> (&L)[3]) {
#pragma unroll
  for (int c = 0; c < 3; ++c) asm volatile("" : "+v"(U[c].re), "+v"(U[c].im), "+v"(L[c].re), "+v"(L[c].im));
  __builtin_amdgcn_sched_barrier(0);
}
// A lane's share of a column: elements e0, e0 + 4 Ls, e0 + 8 Ls.
template <typename T>
struct Share {
  T a, b, c;
};
template <typename T, int LS>
__device__ __forceinline__ Share<T> march_col(const T* __restrict__ in, int v, int e0) {
  const T* c = in + (size_t)v * (12 * LS) + e0;
  return {c[0], c[4 * LS], c[8 * LS]};
}
template <typename T, int LS>
__device__ __forceinline__ void march_put(T* col, int e0, const Share<T>& o) {
  col[e0] = o.a;
  col[e0 + 4 * LS] = o.b;
  col[e0 + 8 * LS] = o.c;
}
// ... and of the links: e0, e0 + 4 Ls (, e0 + 8 Ls), the last lanes entry 71
// (several lanes then store the same value; no branch)
template <typename R, int LS>
__device__ __forceinline__ Share<cplx<R>> march_links(const cplx<R>* __restrict__ gauge, int v, int e0) {
  const cplx<R>* G = gauge + (size_t)v * 72;
  return {G[e0], G[min(e0 + 4 * LS, 71)], G[min(e0 + 8 * LS, 71)]};
}
template <typename R, int LS>
__device__ __forceinline__ void march_put_links(cplx<R>* links, int e0, const Share<cplx<R>>& o) {
  links[e0] = o.a;
  links[min(e0 + 4 * LS, 71)] = o.b;
  if constexpr (8 * LS < 72) links[min(e0 + 8 * LS, 71)] = o.c;
}
// two spins of column v of a field, where wanted
template <typename T, int COL>
__device__ __forceinline__ void march_halo(Tri<T>& a, Tri<T>& b, const T* __restrict__ f, int v, int offa, int offb,
                                           int cs, bool want) {
  Tri<T> x, y;  // unread where not wanted
  if (want) {
    const T* c = f + (size_t)v * COL;
    x.ld(c + offa, cs);
    y.ld(c + offb, cs);
  }
  a = x;
  b = y;
}

// EPI_RES: this lane's values of r and p (if wanted)
template <typename T, int COL>
__device__ __forceinline__ void march_step(Tri<T>& r, Tri<T>& p, const T* rf, const T* pf, int v, int off, int cs) {
  r.ld(rf + (size_t)v * COL + off, cs);
  if (pf) p.ld(pf + (size_t)v * COL + off, cs);
}

// Grid: tiles x right-hand sides, a right-hand side after the other: tiles that
// share faces are in flight together and meet in L2.  That is worth more than
// the links of a tile's several right-hand sides in one pass over them (H in
// complex64 on 24^3 x 48 x 16, 16 right-hand sides: 25.0 against 29.6 ms, with
// 2, 4 and 8 at a time 25.7, 26.8 and 28.4).  by, bz >= 2.
template <typename R, bool DAG, int EPI, int LS, typename T>
__global__ void __launch_bounds__(sizeof(R) == 8 ? 512 : 1024)
hop_march_kernel(T* __restrict__ out, const T* __restrict__ in, const T* __restrict__ center,
                 const cplx<R>* __restrict__ gauge, const R* __restrict__ pw, HopArgs A) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const Geom& g = A.g;
  constexpr int Ls = LS, NS = 16 / LS;
  const int wg = blockIdx.x, rhs = blockIdx.y;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  SplitLane q;
  q.row = lane >> 4;
  const int j = lane & 15;
  q.sub = LS == 16 ? 0 : j / Ls;
  q.s = j - q.sub * Ls;
  q.spin = q.row == 0 ? 0 : q.row == 1 ? 3 : q.row == 2 ? 1 : 2;
  q.upper = !(q.row & 1);
  const int sp = q.row & 1, zt = q.row >> 1;
  const int lsp = zt ? sp : 1 - sp;
  constexpr R SF = DAG ? (R)1 : (R)-1;
  const R g0 = (zt && sp) ? -SF : SF, g1 = (!zt && !sp) ? -SF : SF;
  const bool active = LS == 16 || q.sub < NS;
  constexpr int col = 12 * LS;
  // component offsets of this lane within a column: its upper and lower spin,
  // and the spin it ends with
  constexpr int cs = LS;
  const int offu = q.s + sp * 3 * cs, offl = q.s + (6 + lsp * 3) * cs, offo = q.s + q.spin * 3 * cs;
  const int sn = (q.upper != DAG) ? (q.s > 0 ? q.s - 1 : Ls - 1) : (q.s + 1 < Ls ? q.s + 1 : 0);
  const int offn = sn + q.spin * 3 * cs;

  // tile, pair and its neighbours
  int gx, gy, gz, gt;
  hop_block(A, wg, gx, gy, gz, gt);
  const int npair = A.bx * A.by * A.bz;
  const int p = LS > 8 ? wave : wave * NS + q.sub;  // (LS 12: the idle lanes repeat slices of the same pair)
  const int xl = p & (A.bx - 1), yl = (p >> A.lbx) & (A.by - 1), zl = p >> (A.lbx + A.lby);
  const int xh = gx * A.bx + xl, y = gy * A.by + yl, z = gz * A.bz + zl;
  const int xp = xh + 1 == g.Xh ? 0 : xh + 1, xm = xh == 0 ? g.Xh - 1 : xh - 1;
  const int yn = yl == 0 ? (y == 0 ? g.Y - 1 : y - 1) : (y + 1 == g.Y ? 0 : y + 1);  // across the tile's face
  const int zn = zl == 0 ? (z == 0 ? g.Z - 1 : z - 1) : (z + 1 == g.Z ? 0 : z + 1);
  const int plane = g.Xh * g.Y * g.Z;
  const int own = xh + g.Xh * (y + g.Y * z);
  const bool edge_y = yl == 0 || yl == A.by - 1, edge_z = zl == 0 || zl == A.bz - 1;
  const bool halo_b = !zt && edge_y;  // in slot 2 (y+) or 3 (y-)
  const bool b_plus = yl != 0;
  const int at_b = xh + g.Xh * (yn + g.Y * z);
  const int t0 = gt * A.bt, n = A.bt;

  // LDS: [3][npair][col] columns, then [npair][kLinkLd] links
  const int slot_sz = npair * col;
  const int links_at = (int)(((size_t)3 * slot_sz * sizeof(T) + 15) / 16 * 16);
  T* const ring = reinterpret_cast<T*>(smem_raw);
  cplx<R>* const links = reinterpret_cast<cplx<R>*>(smem_raw + links_at) + p * kLinkLd;
  const T* inr = in + rhs * A.field;
  const T* cen = EPI != EPI_INV ? center + rhs * A.field : nullptr;
  const int e0 = q.row * LS + q.s;  // this lane's first element of the column and of the links
  const int at_z = xh + g.Xh * (y + g.Y * zn), at_row = g.Xh * (y + g.Y * z);

  // b: the output site of the pair is the odd-x one; the pair's own column is
  // then its x- neighbour and x+ is the next pair's
  const int par = y + z + A.out_parity;
  Tri<T> hau, hal, hbu, hbl, cx, cy, rv, pv;
  hau.zero(), hal.zero(), hbu.zero(), hbl.zero(), cx.zero(), cy.zero(), rv.zero(), pv.zero();
  const T* pstep = EPI == EPI_RES && A.cg_p ? static_cast<const T*>(A.cg_p) + rhs * A.field : nullptr;
  {
    const Share<T> oa = march_col<T, LS>(inr, own + plane * (t0 == 0 ? g.T - 1 : t0 - 1), e0);
    const Share<T> ob = march_col<T, LS>(inr, own + plane * t0, e0);
    const Share<T> oc = march_col<T, LS>(inr, own + plane * (t0 + 1 == g.T ? 0 : t0 + 1), e0);
    const Share<cplx<R>> lk = march_links<R, LS>(gauge, own + plane * t0, e0);
    const int b = (par + t0) & 1;
    const bool ha = zt ? edge_z : (b ? xl == A.bx - 1 : xl == 0);
    march_halo<T, col>(hau, hal, inr, (zt ? at_z : at_row + (b ? xp : xm)) + plane * t0, offu, offl, cs, ha);
    march_halo<T, col>(hbu, hbl, inr, at_b + plane * t0, offu, offl, cs, halo_b);
    if (EPI != EPI_INV) march_halo<T, col>(cx, cy, cen, own + plane * t0, offo, offn, cs, true);
    if (EPI == EPI_RES) march_step<T, col>(rv, pv, out + rhs * A.field, pstep, own + plane * t0, offo, cs);
    march_put<T, LS>(ring + p * col, e0, oa);
    march_put<T, LS>(ring + slot_sz + p * col, e0, ob);
    march_put<T, LS>(ring + 2 * slot_sz + p * col, e0, oc);
    march_put_links<R, LS>(links, e0, lk);
  }
  InvCoef<R> inv;
  if (EPI == EPI_INV) inv = split_inv_coef<LS, DAG ? kRowsDn : kRowsUp, !kSMajor<T>>(q, Ls, A, pw);
  lds_barrier();

  double nrm = 0.0;
  int s_prev = 0, s_cur = 1, s_next = 2;
  for (int k = 0; k < n; ++k) {
    const int t = t0 + k;
    const bool more = k + 1 < n;
    // (the last plane loads its own successors' again: no branch around the
    // registers of the next plane)
    const int t1 = more ? t + 1 : t, t2 = more ? (t + 2 >= g.T ? t + 2 - g.T : t + 2) : t;
    const Share<T> oc = march_col<T, LS>(inr, own + plane * t2, e0);
    const Share<cplx<R>> lk = march_links<R, LS>(gauge, own + plane * t1, e0);
    __builtin_amdgcn_sched_barrier(0);
    const int b = (par + t) & 1;
    cplx<R> U[3], L[3];
    {
      const cplx<R>* W = links + (zt ? 18 : 0);
      const bool ha = zt ? edge_z : (b ? xl == A.bx - 1 : xl == 0);
      const bool a_plus = zt ? zl != 0 : b;
      const int dz = A.bx * A.by;
      // the four slots' columns in LDS (a face neighbour's is replaced by the
      // own pair's, whose value is not taken)
      const bool h0 = ha && a_plus, h1 = ha && !a_plus, h2 = halo_b && b_plus, h3 = halo_b && !b_plus;
      const int at0 = s_cur * slot_sz + (h0 ? p : zt ? p + dz : b ? p + 1 : p) * col;
      const int at1 = s_cur * slot_sz + (h1 ? p : zt ? p - dz : b ? p : p - 1) * col;
      const int at2 = zt ? s_next * slot_sz + p * col : s_cur * slot_sz + (h2 ? p : p + A.bx) * col;
      const int at3 = zt ? s_prev * slot_sz + p * col : s_cur * slot_sz + (h3 ? p : p - A.bx) * col;
      // each slot's values are read from LDS while the one before is computed
      Tri<T> u, l, u1, l1;
      u.ld(ring + at0 + offu, cs), l.ld(ring + at0 + offl, cs);
      u1.ld(ring + at1 + offu, cs), l1.ld(ring + at1 + offl, cs);
      u.take(h0, hau), l.take(h0, hal);
      split_dir<0, true>(U, L, u, l, W, g0);
      march_pin(U, L);
      u.ld(ring + at2 + offu, cs), l.ld(ring + at2 + offl, cs);
      u1.take(h1, hau), l1.take(h1, hal);
      split_dir<0>(U, L, u1, l1, W + 36, -g0);
      march_pin(U, L);
      u1.ld(ring + at3 + offu, cs), l1.ld(ring + at3 + offl, cs);
      u.take(h2, hbu), l.take(h2, hbl);
      split_dir<1>(U, L, u, l, W + 9, g1);
      march_pin(U, L);
      u1.take(h3, hbu), l1.take(h3, hbl);
      split_dir<1>(U, L, u1, l1, W + 45, -g1);
      march_pin(U, L);
      {
        const int b1 = more ? 1 - b : b;
        const bool ha1 = zt ? edge_z : (b1 ? xl == A.bx - 1 : xl == 0);
        march_halo<T, col>(hau, hal, inr, (zt ? at_z : at_row + (b1 ? xp : xm)) + plane * t1, offu, offl, cs, ha1);
        march_halo<T, col>(hbu, hbl, inr, at_b + plane * t1, offu, offl, cs, halo_b);
      }
    }
    cplx<R> acc[3];
    split_finish<R, DAG, EPI, LS, false>(acc, U, L, cx, cy, q, Ls, A, inv);
    {
      if (EPI == EPI_RES) split_residual<R, T>(acc, rv, pv, A, rhs);
      if (EPI != EPI_INV && A.partials && active) {
#pragma unroll
        for (int c = 0; c < 3; ++c)
          nrm = fma((double)acc[c].im, (double)acc[c].im, fma((double)acc[c].re, (double)acc[c].re, nrm));
      }
      if (active) tri_st<T>(out + rhs * A.field + (size_t)(own + plane * t) * col + offo, cs, acc, A.nt & 1);
      {
        // the plane behind is read by its own wave alone, and that is done
        march_put<T, LS>(ring + s_prev * slot_sz + p * col, e0, oc);
        march_put_links<R, LS>(links, e0, lk);
        if (EPI != EPI_INV) march_halo<T, col>(cx, cy, cen, own + plane * t1, offo, offn, cs, true);
        if (EPI == EPI_RES) march_step<T, col>(rv, pv, out + rhs * A.field, pstep, own + plane * t1, offo, cs);
      }
    }
    lds_barrier();
    const int s_free = s_prev;
    s_prev = s_cur;
    s_cur = s_next;
    s_next = s_free;
  }
  if (EPI != EPI_INV && A.partials) {
    double vv[1] = {nrm};
    __shared__ double red[16];
    block_sum<1>(vv, red);
    store_partial<1>(vv, A.partials + (size_t)rhs * A.pstride, 0, wg);
  }
}

}  // namespace hdk
