// What the kernels of the hop stages share: site coordinates and orders,
// arguments, the 16-bit layout.
#pragma once

#include <type_traits>

#include "fine_op.h"

namespace hdk {

enum { EPI_INV = 0, EPI_SUB = 1, EPI_RES = 2 };

// ------------------------------------------------------------ coordinates --
struct Site {
  int x, y, z, t, xh;
  int rest;  // y + Y (z + Z t)
  int zt;    // z + Z t
};

__device__ __forceinline__ Site site_coords(int v, int parity, const Geom& g) {
  Site c;
  c.xh = v % g.Xh;
  c.rest = v / g.Xh;
  c.y = c.rest % g.Y;
  c.zt = c.rest / g.Y;
  c.z = c.zt % g.Z;
  c.t = c.zt / g.Z;
  c.x = 2 * c.xh + ((c.y + c.z + c.t + parity) & 1);
  return c;
}

template <typename R>
__device__ __forceinline__ void store_field(cplx<R>* p, cplx<R> v, bool nt) {
  if (nt) {
    __builtin_nontemporal_store(v.re, &p->re);
    __builtin_nontemporal_store(v.im, &p->im);
  } else {
    *p = v;
  }
}
// 16-bit fields keep each site s-major, [s][spin*colour] (48 bytes per
// (site, s)), where the wider types keep [spin*colour][s]: a lane, which owns
// one s of one site, then moves its twelve values with three 16-byte
// accesses instead of twelve 4-byte ones.
template <typename T>
constexpr bool kSMajor = std::is_same<T, bf16c>::value;
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ cplx<float> bf16_word(unsigned w) {
  return cmk(__uint_as_float(w << 16), __uint_as_float(w & 0xffff0000u));
}
__device__ __forceinline__ unsigned bf16_pack(cplx<float> v) {
  return f32x2_to_bf16x2(v.re, v.im);
}

struct HopArgs {
  Geom g;
  int out_parity;
  int spw;            // sites per workgroup
  int bx, by, bz, bt; // 4D site block per workgroup in (x/2, y, z, t), powers of two; bx = 0: linear cb order
  int lbx, lby, lbz;  // log2 of bx, by, bz
  int nbx, nby, nbz;  // block-grid extents
  int remap;          // XCD-contiguous workgroup order
  int nt;             // non-temporal: 1 output stores, 2 links, 4 centre values
  int morton;         // Morton (bit-interleaved) order of the block grid (power-of-two grids)
  int nbt;            // block-grid extent in t
  const int* order;   // nullable: block of workgroup blockIdx.x, packed gx | gy << 8 | gz << 16 | gt << 24
  int rg;             // right-hand sides per workgroup (blockIdx.y takes rg of the nrhs)
  int nrhs;
  size_t field;       // complex elements per rhs
  // fifth dimension: M_5 = alpha + beta K, recurrence of M_5^-1 y_s = ia x_s + kap y_{s-1},
  // Mobius C_5 = b5 + c5 K (K: P+ from s-1, P- from s+1, -mass at the wrap)
  double alpha, beta, ia, kap, b5, c5, mass;
  double kp[4];       // kap^1, kap^2, kap^4, kap^8
  double qia;         // ia / 4: the factor of a hop whose input is alpha M_5^-1 Dh in (Ls <= 16, not 16 bits)
  double kc;          // kap / (1 + mass kap^16)
  // EPI_RES: a per right-hand side (device), lam and p (nullable: no shift)
  const double* cg_alpha;
  const void* cg_p;
  double cg_lam;
  double* partials;   // norm of the output (not EPI_INV): [rhs][pstride] per-workgroup partials (nullable)
  size_t pstride;     // = number of workgroups
  unsigned* counters; // nullable: the grid finishes the norm itself, into
  double* result;     // [rhs]
  FinCg fin;
};

// Block coordinates of workgroup wg in the block grid (lexicographic or
// Morton order); uniform across the workgroup.
__device__ __forceinline__ void hop_block(const HopArgs& A, int wg, int& gx, int& gy, int& gz, int& gt) {
  if (A.order) {
    const int q = A.order[wg];
    gx = q & 255;
    gy = (q >> 8) & 255;
    gz = (q >> 16) & 255;
    gt = (q >> 24) & 255;
  } else if (A.morton) {
    // de-interleave the bits of wg over the four block-grid dimensions
    gx = gy = gz = gt = 0;
    int bit = 0, px = 0, py = 0, pz = 0, pt = 0;
    while ((1 << px) < A.nbx || (1 << py) < A.nby || (1 << pz) < A.nbz || (1 << pt) < A.nbt) {
      if ((1 << px) < A.nbx) gx |= ((wg >> bit++) & 1) << px++;
      if ((1 << py) < A.nby) gy |= ((wg >> bit++) & 1) << py++;
      if ((1 << pz) < A.nbz) gz |= ((wg >> bit++) & 1) << pz++;
      if ((1 << pt) < A.nbt) gt |= ((wg >> bit++) & 1) << pt++;
    }
  } else {
    int q = wg;
    gx = q % A.nbx; q /= A.nbx;
    gy = q % A.nby; q /= A.nby;
    gz = q % A.nbz;
    gt = q / A.nbz;
  }
}

// Coordinates and checkerboard index of the vloc-th output site of
// workgroup wg: either `spw` consecutive sites, or one bx*by*bz*bt block of
// the (x/2, y, z, t) grid, the blocks taken in lexicographic or Morton
// (bit-interleaved) order.  The index may exceed Vh - 1 only in the linear
// order's last workgroup (then the coordinates are not meaningful).
__device__ __forceinline__ int hop_site(const HopArgs& A, int wg, int vloc, Site& c) {
  const Geom& g = A.g;
  if (A.bx <= 0) {
    const int v = wg * A.spw + vloc;
    c = site_coords(v, A.out_parity, g);
    return v;
  }
  int gx, gy, gz, gt;
  hop_block(A, wg, gx, gy, gz, gt);
  c.xh = gx * A.bx + (vloc & (A.bx - 1));
  c.y = gy * A.by + ((vloc >> A.lbx) & (A.by - 1));
  c.z = gz * A.bz + ((vloc >> (A.lbx + A.lby)) & (A.bz - 1));
  c.t = gt * A.bt + (vloc >> (A.lbx + A.lby + A.lbz));
  c.zt = c.z + g.Z * c.t;
  c.rest = c.y + g.Y * c.zt;
  c.x = 2 * c.xh + ((c.y + c.z + c.t + A.out_parity) & 1);
  return c.xh + g.Xh * c.rest;
}

constexpr int kLinkLd = 73;  // LDS row of one site's 72 link entries (odd: no bank aliasing)

// Checkerboard indices of the eight neighbours of site c, in the order
// x+, x-, y+, y-, z+, z-, t+, t-.
__device__ __forceinline__ void hop_neighbours(const Geom& g, const Site& c, int (&nb)[8]) {
  const int rowyzt = c.rest * g.Xh;
  const int xp = (c.x + 1 == g.X) ? 0 : c.x + 1;
  const int xm = (c.x == 0) ? g.X - 1 : c.x - 1;
  nb[0] = (xp >> 1) + rowyzt;
  nb[1] = (xm >> 1) + rowyzt;
  const int yp = (c.y + 1 == g.Y) ? 0 : c.y + 1;
  const int ym = (c.y == 0) ? g.Y - 1 : c.y - 1;
  nb[2] = c.xh + g.Xh * (yp + g.Y * c.zt);
  nb[3] = c.xh + g.Xh * (ym + g.Y * c.zt);
  const int zp = (c.z + 1 == g.Z) ? 0 : c.z + 1;
  const int zm = (c.z == 0) ? g.Z - 1 : c.z - 1;
  const int bz = c.xh + g.Xh * c.y, sy = g.Xh * g.Y;
  nb[4] = bz + sy * (zp + g.Z * c.t);
  nb[5] = bz + sy * (zm + g.Z * c.t);
  const int tp = (c.t + 1 == g.T) ? 0 : c.t + 1;
  const int tm = (c.t == 0) ? g.T - 1 : c.t - 1;
  const int bt = c.xh + g.Xh * (c.y + g.Y * c.z), sz = g.Xh * g.Y * g.Z;
  nb[6] = bt + sz * tp;
  nb[7] = bt + sz * tm;
}

// bytes of LDS of a tile of npair pairs (tb, rb: bytes of a stored and of a
// link entry)
inline size_t march_lds(int npair, int Ls, size_t tb, size_t rb) {
  return ((size_t)3 * npair * 12 * Ls * tb + 15) / 16 * 16 + (size_t)npair * kLinkLd * rb;
}

// hop_ls.h: the stage on fields stored as T for one Ls (0: any up to 16)
template <typename R, typename T, int LS>
void launch_split_mob(bool dagger, int epi, bool mob, bool loop, dim3 grid, dim3 block, size_t lds, hipStream_t stream,
                      T* out, const T* in, const T* center, const cplx<R>* G, const R* pw, const HopArgs& A);
template <typename R, typename T, int LS>
void launch_march_ls(bool dagger, int epi, dim3 grid, dim3 block, size_t lds, hipStream_t stream, T* out, const T* in,
                     const T* center, const cplx<R>* G, const R* pw, const HopArgs& A);

}  // namespace hdk
