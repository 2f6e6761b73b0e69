// Launches of the split and the marched hop stage for one Ls, instantiated by
// hop_ls*.hip (one file for each group of Ls, so that they compile in
// parallel).
#pragma once

#include "hop_march.h"

namespace hdk {

template <typename R, int LS, bool MOB, typename T, bool LOOP>
static void launch_split_ls(bool dagger, int epi, dim3 grid, dim3 block, size_t lds, hipStream_t stream, T* out,
                            const T* in, const T* center, const cplx<R>* G, const R* pw, const HopArgs& A) {
#define HDCG_SPLIT(D, E) \
  hipLaunchKernelGGL((hop_split_kernel<R, D, E, LS, MOB, T, LOOP>), grid, block, lds, stream, out, in, center, G, pw, A)
  if (epi == EPI_RES) {
    HDCG_SPLIT(true, EPI_RES);  // the last stage of H
  } else if (epi == EPI_INV) {
    if (dagger) HDCG_SPLIT(true, EPI_INV);
    else HDCG_SPLIT(false, EPI_INV);
  } else {
    if (dagger) HDCG_SPLIT(true, EPI_SUB);
    else HDCG_SPLIT(false, EPI_SUB);
  }
#undef HDCG_SPLIT
}
template <typename R, typename T, int LS>
void launch_split_mob(bool dagger, int epi, bool mob, bool loop, dim3 grid, dim3 block, size_t lds,
                             hipStream_t stream, T* out, const T* in, const T* center, const cplx<R>* G, const R* pw,
                             const HopArgs& A) {
  if constexpr (LS > 0) {
    if (!loop) {
      if (mob) launch_split_ls<R, LS, true, T, false>(dagger, epi, grid, block, lds, stream, out, in, center, G, pw, A);
      else launch_split_ls<R, LS, false, T, false>(dagger, epi, grid, block, lds, stream, out, in, center, G, pw, A);
      return;
    }
  }
  if (mob) launch_split_ls<R, LS, true, T, true>(dagger, epi, grid, block, lds, stream, out, in, center, G, pw, A);
  else launch_split_ls<R, LS, false, T, true>(dagger, epi, grid, block, lds, stream, out, in, center, G, pw, A);
}
template <typename R, typename T, int LS>
void launch_march_ls(bool dagger, int epi, dim3 grid, dim3 block, size_t lds, hipStream_t stream, T* out,
                            const T* in, const T* center, const cplx<R>* G, const R* pw, const HopArgs& A) {
#define HDCG_MARCH(D, E) \
  hipLaunchKernelGGL((hop_march_kernel<R, D, E, LS, T>), grid, block, lds, stream, out, in, center, G, pw, A)
  if (epi == EPI_RES) {
    HDCG_MARCH(true, EPI_RES);
  } else if (epi == EPI_INV) {
    if (dagger) HDCG_MARCH(true, EPI_INV);
    else HDCG_MARCH(false, EPI_INV);
  } else {
    if (dagger) HDCG_MARCH(true, EPI_SUB);
    else HDCG_MARCH(false, EPI_SUB);
  }
#undef HDCG_MARCH
}

#define HDCG_HOP_ARGS(R, T) \
  dim3, dim3, size_t, hipStream_t, T*, const T*, const T*, const cplx<R>*, const R*, const HopArgs&
#define HDCG_HOP_SPLIT(LS)                                                                       \
  template void launch_split_mob<double, c128, LS>(bool, int, bool, bool, HDCG_HOP_ARGS(double, c128)); \
  template void launch_split_mob<float, c64, LS>(bool, int, bool, bool, HDCG_HOP_ARGS(float, c64));     \
  template void launch_split_mob<float, bf16c, LS>(bool, int, bool, bool, HDCG_HOP_ARGS(float, bf16c));
#define HDCG_HOP_MARCH(LS)                                                          \
  template void launch_march_ls<double, c128, LS>(bool, int, HDCG_HOP_ARGS(double, c128)); \
  template void launch_march_ls<float, c64, LS>(bool, int, HDCG_HOP_ARGS(float, c64));

}  // namespace hdk
