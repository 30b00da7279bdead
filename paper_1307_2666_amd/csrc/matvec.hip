// Exact on-the-fly y = A x for A = diag(a) + diag(b) K diag(c) (eqn 1.1 under
// the collocation of Section 3.1): K_ij = G(|x_i - x_j|) w_j off the
// diagonal, K_ii the cell integral.  O(N^2) pair evaluations; the waves of a
// workgroup share its targets and divide the sources, which they stream
// through LDS in tiles of their own; all right-hand sides (up to 8 per pass)
// share one kernel evaluation per pair.
#include <type_traits>

#include "common.h"

namespace hif {

namespace {

// Natural logarithm of a positive normal x, within about 2 ulp (the library's
// double-precision log carries extra-precise steps that cost several times as
// much, and the pair loop below is bound by it).  x = 2^e m with m in
// [sqrt(1/2), sqrt(2)); with s = (m - 1) / (m + 1), |s| <= 3 - 2 sqrt(2) <
// 0.1716, log m = 2 atanh(s) = 2 s + 2 s z P(z), z = s^2, P(z) = sum z^k /
// (2k + 3); the coefficients are those of P's Chebyshev expansion of degree 6
// on [0, (3 - 2 sqrt 2)^2], off by less than 2^-57 of the logarithm (the power
// series takes two more).  log x = e ln2_hi + (e ln2_lo + log m), ln2_hi
// holding 29 significant bits so that e ln2_hi is exact.
// The constants of the pair loop in registers: as literals each would be moved
// into place ahead of its fused multiply-add.
struct LogCoef {
  double c[7], lo, hi;
  __device__ LogCoef()
      : c{0.3333333333333333, 0.19999999999965573, 0.1428571430871919, 0.111111060617156, 0.09091416704888747,
          0.07666614987761301, 0.07300366937947979},
        lo(-4.2009150726810846e-11),
        hi(0.6931471806019545) {
#pragma unroll
    for (int k = 0; k < 7; ++k) asm volatile("" : "+v"(c[k]));
    asm volatile("" : "+v"(lo), "+v"(hi));
  }
};
__device__ __forceinline__ double log_pos(double x, const LogCoef& L) {
  double m = __builtin_amdgcn_frexp_mant(x);  // [0.5, 1)
  int e = __builtin_amdgcn_frexp_exp(x);
  const bool lo = m < 0.70710678118654752440;
  m = __builtin_amdgcn_ldexp(m, lo ? 1 : 0);
  e -= lo ? 1 : 0;
  const double f = m - 1.0;  // exact
  const double d = m + 1.0;
  double t = __builtin_amdgcn_rcp(d);
  t = fma(fma(-d, t, 1.0), t, t);  // one Newton step on 1 / d
  double q = f * t;
  q = fma(fma(-q, d, f), t, q);  // s = f / d, corrected once
  const double z = q * q;
  double p = L.c[6];
#pragma unroll
  for (int k = 5; k >= 0; --k) p = fma(p, z, L.c[k]);
  const double s2 = 2.0 * q;
  const double ed = double(e);
  const double r = fma(s2 * z, p, ed * L.lo);  // + e ln2_lo
  return fma(ed, L.hi, s2 + r);
}

// G(r) without its constant factor from the squared distance: log r^2 (2D) or
// 1 / r (3D).  1 / r: the hardware's estimate (2^-24 or better) and one
// third-order step; where r^2 is zero or overflows (their product is 0 times
// infinity) the estimate stands.
template <int D>
struct Green;
template <>
struct Green<2> {
  static constexpr double factor = -0.5 * kInv2Pi;
  LogCoef L;
  __device__ __forceinline__ double operator()(double r2) const { return log_pos(r2, L); }
};
template <>
struct Green<3> {
  static constexpr double factor = kInv4Pi;
  __device__ __forceinline__ double operator()(double r2) const {
    const double y = __builtin_amdgcn_rsq(r2), r = r2 * y;
    const double e = fma(-r, y, 1.0);
    const double v = fma(y * e, fma(e, 0.375, 0.5), y);
    return r == r ? v : y;
  }
};

// Workgroup of NW waves: L = 64 / SPL lanes hold TPT targets each (the same
// L TPT targets in every wave), lane group s = lane / L of wave w takes the
// sources s, s + SPL, ... of the tiles of 64 it streams, w, w + NW, ...  The
// partial sums are added over the groups and then the waves, in order.
// Bound by the vector ALU: per pair the distance, G (about 25 instructions in
// 2D, 7 in 3D) and one multiply-add per right-hand side (39 and 20 in all with
// 8 and 5 of them; 80% of the issue rate at 262144 points in 2D), against the
// LDS reads of a source's D + NR values, which TPT targets share.  Before, a
// workgroup's 256 lanes held a target each and passed over all sources, one
// wave a SIMD at 50000 points: 49999 points in 3D with 5 right-hand sides 7.5
// -> 2.1 ms, 65536 in 2D with 4 11.7 -> 4.9 ms, 262144 with 8 126 -> 87 ms,
// 5000 with one 0.85 -> 0.06 ms.
template <int D, int NR, int TPT, int SPL, int NW>
__global__ __launch_bounds__(64 * NW) void k_matvec(const double* __restrict__ pts, int64_t n,
                                                    const double* __restrict__ a, const double* __restrict__ b,
                                                    const double* __restrict__ c, const double* __restrict__ w,
                                                    double w_const, const double* __restrict__ selfk,
                                                    double self_const, const double* __restrict__ x,
                                                    double* __restrict__ y, int64_t ldx) {
  constexpr int L = 64 / SPL, WS = (D + NR + 1) & ~1;
  static_assert(L * TPT <= 64 * WS, "the partial sums reuse the tiles");
  alignas(16) __shared__ double st[NW][64][WS];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tl = lane % L, sl = lane / L;
  const int64_t i0 = blockIdx.x * int64_t(L * TPT);
  const Green<D> green;
  double xi[TPT][D], acc[TPT][NR];
#pragma unroll
  for (int u = 0; u < TPT; ++u) {
    const int64_t i = i0 + u * L + tl;
#pragma unroll
    for (int k = 0; k < D; ++k) xi[u][k] = i < n ? pts[i * D + k] : 4.0 + k;
#pragma unroll
    for (int v = 0; v < NR; ++v) acc[u][v] = 0.0;
  }
  double src[D + NR];  // this lane's source of the next tile
  auto fetch = [&](int64_t j0) {
    const int64_t j = j0 + lane;
    if (j < n) {
#pragma unroll
      for (int k = 0; k < D; ++k) src[k] = pts[j * D + k];
      const double wc = (w ? w[j] : w_const) * (c ? c[j] : 1.0);
#pragma unroll
      for (int v = 0; v < NR; ++v) src[D + v] = wc * x[v * ldx + j];
    } else {
      // Weight 0, anywhere: in 2D G is finite also at a target; in 3D the pair
      // is dropped below.
#pragma unroll
      for (int k = 0; k < D; ++k) src[k] = 2.0 + k;
#pragma unroll
      for (int v = 0; v < NR; ++v) src[D + v] = 0.0;
    }
  };
  fetch(int64_t(wv) * 64);
  for (int64_t j0 = int64_t(wv) * 64; j0 < n; j0 += 64 * NW) {
    __builtin_amdgcn_wave_barrier();  // the wave's own tile: its LDS accesses are in order
#pragma unroll
    for (int k = 0; k < D + NR; ++k) st[wv][lane][k] = src[k];
    if (j0 + 64 * NW < n) fetch(j0 + 64 * NW);
    __builtin_amdgcn_wave_barrier();
    const int cnt = int(n - j0 < 64 ? n - j0 : 64);  // sources of the tile
    const int self0 = int(i0 - j0 > -4096 ? i0 - j0 : -4096);  // of the tile's first source; any far off will do
    auto pass = [&](auto some_dropped) {
#pragma unroll 2
      for (int t = 0; t < 64; t += SPL) {
        double s[WS];
        const double* row = st[wv][t + sl];
#pragma unroll
        for (int k = 0; k < WS; k += 2) {
          const double2 v = *reinterpret_cast<const double2*>(row + k);
          s[k] = v.x;
          s[k + 1] = v.y;
        }
#pragma unroll
        for (int u = 0; u < TPT; ++u) {
          double r2 = 0.0;
#pragma unroll
          for (int k = 0; k < D; ++k) {
            const double dd = xi[u][k] - s[k];
            r2 = k == 0 ? dd * dd : fma(dd, dd, r2);
          }
          double g;
          if constexpr (decltype(some_dropped)::value) {  // by a select: the self pair, in 3D also what is past n
            bool drop = j0 + t + sl == i0 + u * L + tl;
            if constexpr (D == 3) drop = t + sl == self0 + u * L + tl || t + sl >= cnt;
            g = green(drop ? 1.0 : r2);
            g = drop ? 0.0 : g;
          } else {
            g = green(r2);
          }
#pragma unroll
          for (int v = 0; v < NR; ++v) acc[u][v] = fma(g, s[D + v], acc[u][v]);
        }
      }
    };
    if ((j0 < i0 + L * TPT && j0 + 64 > i0) || (D == 3 && cnt < 64))
      pass(std::true_type{});
    else
      pass(std::false_type{});
  }
  // partial sums: over the lane groups, then the waves
#pragma unroll
  for (int u = 0; u < TPT; ++u)
#pragma unroll
    for (int v = 0; v < NR; ++v)
#pragma unroll
      for (int o = L; o < 64; o *= 2) acc[u][v] += __shfl_xor(acc[u][v], o, 64);
  double* part = &st[0][0][0];
#pragma unroll
  for (int v = 0; v < NR; ++v) {
    __syncthreads();  // the tiles, or the sums of the last vector, have been read
    if (sl == 0) {
#pragma unroll
      for (int u = 0; u < TPT; ++u) part[wv * 64 * WS + u * L + tl] = acc[u][v];
    }
    __syncthreads();
    for (int e = tid; e < L * TPT; e += 64 * NW) {
      const int64_t i = i0 + e;
      if (i >= n) continue;
      double s = 0.0;
#pragma unroll
      for (int k = 0; k < NW; ++k) s += part[k * 64 * WS + e];
      const double ai = a ? a[i] : 0.0, bi = b ? b[i] : 1.0, ci = c ? c[i] : 1.0;
      const double si = selfk ? selfk[i] : self_const;
      const double xv = x[v * ldx + i];
      y[v * ldx + i] = ai * xv + bi * (Green<D>::factor * s + si * ci * xv);
    }
  }
}

template <int D, int NR>
void launch_nr(const double* pts, int64_t n, const double* a, const double* b, const double* c, const double* w,
               double w_const, const double* selfk, double self_const, const double* x, double* y, hipStream_t s) {
  // Targets per workgroup: 64 TPT / SPL.
  auto run = [&](auto tpt, auto spl, auto nw) {
    constexpr int TPT = decltype(tpt)::value, SPL = decltype(spl)::value, NW = decltype(nw)::value;
    const int64_t tw = 64 / SPL * TPT;
    hipLaunchKernelGGL((k_matvec<D, NR, TPT, SPL, NW>), dim3(unsigned((n + tw - 1) / tw)), dim3(64 * NW), 0, s, pts, n,
                       a, b, c, w, w_const, selfk, self_const, x, y, n);
  };
  using std::integral_constant;
  constexpr integral_constant<int, (NR <= 4 ? 4 : 2)> many;  // targets a lane: as many as leave 3 waves a SIMD
  if (n >= (int64_t(1) << 18))
    run(many, integral_constant<int, 1>{}, integral_constant<int, 4>{});
  else if (n >= (int64_t(1) << 15))  // four lanes a target: workgroups for every CU
    run(many, integral_constant<int, 4>{}, integral_constant<int, 4>{});
  else  // fewer targets and more waves a workgroup
    run(integral_constant<int, 1>{}, integral_constant<int, 4>{}, integral_constant<int, 8>{});
  HIF_HIP(hipGetLastError());
}

template <int D>
void launch(const double* pts, int64_t n, const double* a, const double* b, const double* c, const double* w,
            double w_const, const double* selfk, double self_const, const double* x, double* y, int64_t nrhs,
            hipStream_t s) {
  const int64_t passes = (nrhs + 7) / 8;
  for (int64_t p = 0; p < passes; ++p) {  // right-hand sides divided evenly
    const int64_t v0 = nrhs * p / passes, nr = nrhs * (p + 1) / passes - v0;
    const double* xv = x + v0 * n;
    double* yv = y + v0 * n;
#define HIF_CASE(NR) \
  case NR: launch_nr<D, NR>(pts, n, a, b, c, w, w_const, selfk, self_const, xv, yv, s); break;
    switch (nr) {
      HIF_CASE(1) HIF_CASE(2) HIF_CASE(3) HIF_CASE(4) HIF_CASE(5) HIF_CASE(6) HIF_CASE(7) HIF_CASE(8)
    }
#undef HIF_CASE
  }
}

}  // namespace

void matvec_impl(const double* pts, int64_t n, int dim, const double* a, const double* b, const double* c,
                 const double* w, double w_const, const double* selfk, double self_const, const double* x,
                 double* y, int64_t nrhs, hipStream_t s) {
  if (dim == 2)
    launch<2>(pts, n, a, b, c, w, w_const, selfk, self_const, x, y, nrhs, s);
  else
    launch<3>(pts, n, a, b, c, w, w_const, selfk, self_const, x, y, nrhs, s);
}

}  // namespace hif
