// Pivot searches across the lanes of a wave and the composition of
// interchanges, shared by the LU and the pivoted QR.  Internal, not part of
// the ABI.
#pragma once

#include <climits>

#include "common.h"
#include "wave.h"

namespace hif {

template <int CTRL>
__device__ __forceinline__ double dpp_max(double x) {
  const unsigned long long u = __double_as_longlong(x);
  const int lo = dpp<CTRL>(int(unsigned(u))), hi = dpp<CTRL>(int(unsigned(u >> 32)));
  return fmax(x, __longlong_as_double((static_cast<long long>(hi) << 32) | unsigned(lo)));
}
// Largest value of each aligned group of G = 4, 8 or 16 lanes, on all of them (no NaN).
template <int G>
__device__ __forceinline__ double group_max(double x) {
  x = dpp_max<kXor2>(dpp_max<kXor1>(x));
  if constexpr (G >= 8) x = dpp_max<kHalfMirror>(x);
  if constexpr (G >= 16) x = dpp_max<kMirror>(x);
  return x;
}
template <int G>
__device__ __forceinline__ int group_min(int x) {
  x = min(x, dpp<kXor1>(x));
  x = min(x, dpp<kXor2>(x));
  if constexpr (G >= 8) x = min(x, dpp<kHalfMirror>(x));
  if constexpr (G >= 16) x = min(x, dpp<kMirror>(x));
  return x;
}
// Largest value of the wave, on every lane (no NaN).
__device__ __forceinline__ double wave_max(double x) {
  x = group_max<16>(x);
  auto half = [&](auto sw) {
    const unsigned long long u = __double_as_longlong(x);
    const auto rl = sw(unsigned(u)), rh = sw(unsigned(u >> 32));
    const double a = __longlong_as_double((static_cast<long long>(rh[0]) << 32) | rl[0]);
    const double b = __longlong_as_double((static_cast<long long>(rh[1]) << 32) | rl[1]);
    x = fmax(a, b);
  };
  half([](unsigned v) { return __builtin_amdgcn_permlane16_swap(v, v, false, false); });
  half([](unsigned v) { return __builtin_amdgcn_permlane32_swap(v, v, false, false); });
  return x;
}

// Smallest value of the wave, on every lane.
__device__ __forceinline__ int wave_min(int x) {
  x = group_min<16>(x);
  auto r = __builtin_amdgcn_permlane16_swap(unsigned(x), unsigned(x), false, false);
  x = min(int(r[0]), int(r[1]));
  r = __builtin_amdgcn_permlane32_swap(unsigned(x), unsigned(x), false, false);
  return min(int(r[0]), int(r[1]));
}

// The interchanges rows J + jj <-> piv[jj] (jj < nj <= NE), in order, as one
// permutation: position dst[e] receives the present row src[e]; the first nj
// entries are the positions J + jj.  One wave; lane e holds entry e of the nj
// and entry e of the up to nj others.  Interchanges out of range (a singular
// block leaves none, or those of an earlier panel) are passed over.
__device__ __forceinline__ void compose_swaps(const int32_t* piv, int J, int nj, int n, int* s_dst, int* s_src,
                                              int* s_na) {
  const int lane = threadIdx.x & 63;
  const int my = lane < nj ? piv[lane] : -1;
  int src0 = J + lane, dst1 = -1, src1 = -1, nx = 0;
  for (int jj = 0; jj < nj; ++jj) {
    const int p = __builtin_amdgcn_readlane(my, jj);
    if (p <= J + jj || p >= n) continue;
    const int sj = __builtin_amdgcn_readlane(src0, jj);
    if (p < J + nj) {
      const int sp = __builtin_amdgcn_readlane(src0, p - J);
      if (lane == jj) src0 = sp;
      if (lane == p - J) src0 = sj;
    } else {
      const unsigned long long hit = __ballot(dst1 == p);
      int e;
      if (hit) {
        e = __ffsll(hit) - 1;
      } else {
        e = nx++;
        if (lane == e) dst1 = src1 = p;
      }
      const int sp = __builtin_amdgcn_readlane(src1, e);
      if (lane == jj) src0 = sp;
      if (lane == e) src1 = sj;
    }
  }
  if (lane < nj) {
    s_dst[lane] = J + lane;
    s_src[lane] = src0;
  }
  if (lane < nx) {
    s_dst[nj + lane] = dst1;
    s_src[nj + lane] = src1;
  }
  if (lane == 0) *s_na = nj + nx;
}

}  // namespace hif
