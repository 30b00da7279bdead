// Factored apply / solve sweeps: F = U_0^{-T} ... D ... V_0^{-1} and
// F^{-1} = V_0 ... D^{-1} ... U_0^T (eqns rskelf, hifie2, hifie3) and their
// transposes.  A group record holds T, the row-pivoted LU of B_rr
// (P B_rr = L U), L_sr = B_sr U^{-1} and U_rs = L^{-1} P B_rs (the operators
// R_p, S_p of Lemma 2.1 with Q = [I 0; -T I] of Lemma 2.4, (redundant,
// skeleton) order).  Per group:
//   solve   up:   u_r -= T^T u_s;  u_r = L^{-1} P u_r;     u_s -= L_sr u_r
//           down: u_r -= U_rs u_s; u_r = U^{-1} u_r;       u_s -= T u_r
//   solve_T up:   u_r -= T^T u_s;  u_r = U^{-T} u_r;       u_s -= U_rs^T u_r
//           down: u_r -= L_sr^T u_s; u_r = P^T L^{-T} u_r; u_s -= T u_r
//   apply   up:   x_s += T x_r;    x_r = U x_r + U_rs x_s
//           down: y_s += L_sr y_r; y_r = P^T L y_r;        y_r += T^T y_s
//   apply_T up:   x_s += T x_r;    x_r = L^T P x_r + L_sr^T x_s
//           down: y_s += U_rs^T y_r; y_r = U^T y_r;        y_r += T^T y_s
// with the top block A_L (LU with pivoting) solved or applied in between.
// "up" visits sub-levels finest first, "down" in reverse; the groups of one
// sub-level touch disjoint DOFs and run as one launch, one workgroup each.
// Vectors are [nrhs][N] in the caller's order; every product works in place
// through the records' global DOF indices.
#include <mutex>
#include <string>
#include <type_traits>

#include "common.h"
#include "wave.h"

namespace hif {

namespace {

constexpr int kBlock = 256;

struct SwArgs {
  const GroupRec* recs;
  const int32_t* iarena;
  const double* darena;
  double* u;
  double* work;
  int64_t N;
  int nrhs;
  int op;
};

// u[yi[i]] += sgn * sum_j M[i*ld + j] u[xi[j]]   (one wave per row)
__device__ void gemv_rows(const double* M, int nrow, int ncol, int ld, const int32_t* yi, const int32_t* xi,
                          double* u, int64_t N, int nrhs, double sgn) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
  for (int i = wv; i < nrow; i += nw) {
    const double* mr = M + int64_t(i) * ld;
    for (int v = 0; v < nrhs; ++v) {
      const double* uv = u + v * N;
      double s = 0.0;
      for (int j = lane; j < ncol; j += 64) s += mr[j] * uv[xi[j]];
      s = wave_sum(s);
      if (lane == 0) u[v * N + yi[i]] += sgn * s;
    }
  }
}

// u[yi[j]] += sgn * sum_i M[i*ld + j] u[xi[i]]   (one thread per column and RHS)
__device__ void gemv_cols(const double* M, int nrow, int ncol, int ld, const int32_t* yi, const int32_t* xi,
                          double* u, int64_t N, int nrhs, double sgn) {
  for (int e = threadIdx.x; e < ncol * nrhs; e += blockDim.x) {
    const int j = e % ncol, v = e / ncol;
    const double* uv = u + v * N;
    double s = 0.0;
    for (int i = 0; i < nrow; ++i) s += M[int64_t(i) * ld + j] * uv[xi[i]];
    u[v * N + yi[j]] += sgn * s;
  }
}

// Triangular pieces on u_r = u[v*N + idx[i]], i < n, all RHS; LU is n x n
// row-major holding unit-lower L and upper U; piv the row interchanges.
__device__ void swaps_fwd(const int32_t* piv, int n, const int32_t* idx, double* u, int64_t N, int nrhs) {
  for (int v = threadIdx.x; v < nrhs; v += blockDim.x)
    for (int j = 0; j < n; ++j)
      if (piv[j] != j) {
        double* a = u + v * N + idx[j];
        double* b = u + v * N + idx[piv[j]];
        const double t = *a; *a = *b; *b = t;
      }
  __syncthreads();
}
__device__ void swaps_rev(const int32_t* piv, int n, const int32_t* idx, double* u, int64_t N, int nrhs) {
  for (int v = threadIdx.x; v < nrhs; v += blockDim.x)
    for (int j = n - 1; j >= 0; --j)
      if (piv[j] != j) {
        double* a = u + v * N + idx[j];
        double* b = u + v * N + idx[piv[j]];
        const double t = *a; *a = *b; *b = t;
      }
  __syncthreads();
}
// x = L^{-1} x (unit lower), column oriented
__device__ void solve_L(const double* LU, int n, const int32_t* idx, double* u, int64_t N, int nrhs) {
  for (int j = 0; j < n - 1; ++j) {
    const int w = n - 1 - j;
    for (int e = threadIdx.x; e < w * nrhs; e += blockDim.x) {
      const int i = j + 1 + e % w, v = e / w;
      u[v * N + idx[i]] -= LU[int64_t(i) * n + j] * u[v * N + idx[j]];
    }
    __syncthreads();
  }
  __syncthreads();
}
// x = U^{-1} x
__device__ void solve_U(const double* LU, int n, const int32_t* idx, double* u, int64_t N, int nrhs) {
  for (int j = n - 1; j >= 0; --j) {
    const double inv = 1.0 / LU[int64_t(j) * n + j];
    for (int e = threadIdx.x; e < j * nrhs; e += blockDim.x) {
      const int i = e % j, v = e / j;
      u[v * N + idx[i]] -= LU[int64_t(i) * n + j] * (u[v * N + idx[j]] * inv);
    }
    __syncthreads();
  }
  for (int e = threadIdx.x; e < n * nrhs; e += blockDim.x) {
    const int i = e % n, v = e / n;
    u[v * N + idx[i]] /= LU[int64_t(i) * n + i];
  }
  __syncthreads();
}
// x = U^{-T} x (U^T lower)
__device__ void solve_UT(const double* LU, int n, const int32_t* idx, double* u, int64_t N, int nrhs) {
  for (int j = 0; j < n; ++j) {
    const double inv = 1.0 / LU[int64_t(j) * n + j];
    const int w = n - 1 - j;
    for (int e = threadIdx.x; e < w * nrhs; e += blockDim.x) {
      const int i = j + 1 + e % w, v = e / w;
      u[v * N + idx[i]] -= LU[int64_t(j) * n + i] * (u[v * N + idx[j]] * inv);
    }
    __syncthreads();
  }
  for (int e = threadIdx.x; e < n * nrhs; e += blockDim.x) {
    const int i = e % n, v = e / n;
    u[v * N + idx[i]] /= LU[int64_t(i) * n + i];
  }
  __syncthreads();
}
// x = L^{-T} x (L^T unit upper)
__device__ void solve_LT(const double* LU, int n, const int32_t* idx, double* u, int64_t N, int nrhs) {
  for (int j = n - 1; j > 0; --j) {
    for (int e = threadIdx.x; e < j * nrhs; e += blockDim.x) {
      const int i = e % j, v = e / j;
      u[v * N + idx[i]] -= LU[int64_t(j) * n + i] * u[v * N + idx[j]];
    }
    __syncthreads();
  }
  __syncthreads();
}
// x = op(x) through the work buffer: mode 0: U x, 1: L x, 2: L^T x, 3: U^T x
__device__ void tri_mul(const double* LU, int n, const int32_t* idx, double* u, double* work, int64_t N, int nrhs,
                        int mode) {
  for (int e = threadIdx.x; e < n * nrhs; e += blockDim.x) {
    const int i = e % n, v = e / n;
    const double* uv = u + v * N;
    double s = 0.0;
    if (mode == 0) {
      for (int j = i; j < n; ++j) s += LU[int64_t(i) * n + j] * uv[idx[j]];
    } else if (mode == 1) {
      s = uv[idx[i]];
      for (int j = 0; j < i; ++j) s += LU[int64_t(i) * n + j] * uv[idx[j]];
    } else if (mode == 2) {
      s = uv[idx[i]];
      for (int j = i + 1; j < n; ++j) s += LU[int64_t(j) * n + i] * uv[idx[j]];
    } else {
      for (int j = 0; j <= i; ++j) s += LU[int64_t(j) * n + i] * uv[idx[j]];
    }
    work[v * N + idx[i]] = s;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < n * nrhs; e += blockDim.x) {
    const int i = e % n, v = e / n;
    u[v * N + idx[i]] = work[v * N + idx[i]];
  }
  __syncthreads();
}

__global__ void k_up(SwArgs A) {
  const GroupRec R = A.recs[blockIdx.x];
  const int r = R.r, k = R.k;
  const int32_t* rd = A.iarena + R.idx;
  const int32_t* sk = rd + r;
  const int32_t* piv = sk + k;
  const double* T = A.darena + R.off;
  const double* Lsr = T + int64_t(k) * r;
  const double* Urs = Lsr + int64_t(k) * r;
  const double* LU = Urs + int64_t(r) * k;
  double* u = A.u;
  const int64_t N = A.N;
  const int nr = A.nrhs;
  if (A.op <= 1) {
    if (k > 0) gemv_cols(T, k, r, r, rd, sk, u, N, nr, -1.0);  // u_r -= T^T u_s
    __syncthreads();
    if (A.op == 0) {
      swaps_fwd(piv, r, rd, u, N, nr);
      solve_L(LU, r, rd, u, N, nr);
      if (k > 0) gemv_rows(Lsr, k, r, r, sk, rd, u, N, nr, -1.0);  // u_s -= L_sr u_r
    } else {
      solve_UT(LU, r, rd, u, N, nr);
      if (k > 0) gemv_cols(Urs, r, k, k, sk, rd, u, N, nr, -1.0);  // u_s -= U_rs^T u_r
    }
  } else {
    if (k > 0) gemv_rows(T, k, r, r, sk, rd, u, N, nr, 1.0);  // x_s += T x_r
    __syncthreads();
    if (A.op == 2) {
      tri_mul(LU, r, rd, u, A.work, N, nr, 0);                     // x_r = U x_r
      if (k > 0) gemv_rows(Urs, r, k, k, rd, sk, u, N, nr, 1.0);   //      + U_rs x_s
    } else {
      swaps_fwd(piv, r, rd, u, N, nr);
      tri_mul(LU, r, rd, u, A.work, N, nr, 2);                     // x_r = L^T P x_r
      if (k > 0) gemv_cols(Lsr, k, r, r, rd, sk, u, N, nr, 1.0);   //      + L_sr^T x_s
    }
  }
}

__global__ void k_down(SwArgs A) {
  const GroupRec R = A.recs[blockIdx.x];
  const int r = R.r, k = R.k;
  const int32_t* rd = A.iarena + R.idx;
  const int32_t* sk = rd + r;
  const int32_t* piv = sk + k;
  const double* T = A.darena + R.off;
  const double* Lsr = T + int64_t(k) * r;
  const double* Urs = Lsr + int64_t(k) * r;
  const double* LU = Urs + int64_t(r) * k;
  double* u = A.u;
  const int64_t N = A.N;
  const int nr = A.nrhs;
  if (A.op <= 1) {
    if (A.op == 0) {
      if (k > 0) gemv_rows(Urs, r, k, k, rd, sk, u, N, nr, -1.0);  // u_r -= U_rs u_s
      __syncthreads();
      solve_U(LU, r, rd, u, N, nr);
    } else {
      if (k > 0) gemv_cols(Lsr, k, r, r, rd, sk, u, N, nr, -1.0);  // u_r -= L_sr^T u_s
      __syncthreads();
      solve_LT(LU, r, rd, u, N, nr);
      swaps_rev(piv, r, rd, u, N, nr);
    }
    if (k > 0) gemv_rows(T, k, r, r, sk, rd, u, N, nr, -1.0);  // u_s -= T u_r
  } else {
    if (A.op == 2) {
      if (k > 0) gemv_rows(Lsr, k, r, r, sk, rd, u, N, nr, 1.0);  // y_s += L_sr y_r
      __syncthreads();
      tri_mul(LU, r, rd, u, A.work, N, nr, 1);                    // y_r = P^T L y_r
      swaps_rev(piv, r, rd, u, N, nr);
    } else {
      if (k > 0) gemv_cols(Urs, r, k, k, sk, rd, u, N, nr, 1.0);  // y_s += U_rs^T y_r
      __syncthreads();
      tri_mul(LU, r, rd, u, A.work, N, nr, 3);                    // y_r = U^T y_r
    }
    if (k > 0) gemv_cols(T, k, r, r, rd, sk, u, N, nr, 1.0);  // y_r += T^T y_s
  }
}

// ---------------------------------------------------------------------------
// LDS-staged solve / solve_T.  The entries u_r, u_s of a group (or the top
// block's entries) are gathered into LDS once; the products and the blocked
// triangular solves (64-column diagonal blocks solved by one wave with
// shuffles, then one update of the remaining rows) run there, and the results
// are scattered back.  The row interchanges use the gather index perm,
// (P x)[i] = x[perm[i]].
// ---------------------------------------------------------------------------
constexpr int kNbT = 64;
constexpr int kMaxV = 8;       // right-hand sides per pass
static_assert(kMaxV == 8, "the row products reduce their kMaxV sums with wave_rs8, 4 rows with wave_rs32");
constexpr int kCapL = 16384;   // LDS doubles, largest records and the top block
// Sub-levels with at least this many records run 64, 128 or 256 threads per
// record (launch-shape table), fewer records 1024 threads each.
constexpr int kManyRecords = 1024;
// Top blocks of at least this many unknowns are solved by the many-workgroup
// blocked triangular solves: one workgroup walks the block's rows with the
// loads of one workgroup in flight (a solve with a top of 152: 93 us against
// 61, of 474: 527 against 286, of 2872: 5360 against 161; applies of 152: 72
// against 51).  Below two 64-row blocks there is nothing to hand over.
constexpr int64_t kTopSplitMin = 128;

// Loads in flight per lane in the products below.  A workgroup waits for
// memory at most a few times in a product then: a wait (with the address
// translation of a record's pages, each touched once) costs 1 - 2 us here.
constexpr int kU = 16;

// y[v*ys + i] += sgn * sum_j M[i*ld + j] x[v*xs + j]   (one wave per row).  A
// wave takes R rows and 64 C columns of each at a time, R C loads before any is
// used (16 rows of up to 64 columns at a time were slower than 4: the code is
// run a few times per workgroup, and four times as much of it has to be
// fetched); TRI >= 0 keeps one triangle: 0 the columns j >= i, 1 the columns
// j < i, and reads no column that its rows do not reach (the applies of 64
// records of about 480 redundant unknowns: 177 us a sweep when all were read and
// a select chose between entry and zero, 104 so).
template <int R, int C, int TRI>
__device__ __forceinline__ void l_gemv_n_rc(const double* __restrict__ M, int nrow, int ncol, int ld, const double* x,
                                            int xs, double* y, int ys, int nv, double sgn) {
  constexpr bool kOnce = R > 2;  // the columns fit: a row is finished before the next
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  for (int i0 = wv; i0 < nrow; i0 += R * nw) {
    double acc[kOnce ? 1 : R][kMaxV];
    if constexpr (!kOnce)
#pragma unroll
      for (int q = 0; q < R; ++q)
#pragma unroll
        for (int v = 0; v < kMaxV; ++v) acc[q][v] = 0.0;
    auto put = [&](double (&a)[kMaxV], int i) {
      const double t = wave_rs8(a);
      const int v = lane >> 3;
      if ((lane & 7) == 0 && v < nv && i < nrow) y[v * ys + i] += sgn * t;
    };
    // the columns that the triangle has in these rows
    const int jb = TRI == 0 ? i0 & ~63 : 0, je = TRI == 1 ? min(ncol, i0 + (R - 1) * nw) : ncol;
    for (int j0 = jb; j0 < je; j0 += 64 * C) {
      double m[R][C];
#pragma unroll
      for (int q = 0; q < R; ++q)
#pragma unroll
        for (int h = 0; h < C; ++h) {
          const int i = min(i0 + q * nw, nrow - 1), j = j0 + 64 * h + lane;
          m[q][h] = M[int64_t(i) * ld + min(j, je - 1)];
        }
#pragma unroll
      for (int q = 0; q < R; ++q) {
        if (i0 + q * nw >= nrow) break;
        double(&a)[kMaxV] = acc[kOnce ? 0 : q];
        if constexpr (kOnce)
#pragma unroll
          for (int v = 0; v < kMaxV; ++v) a[v] = 0.0;
#pragma unroll
        for (int h = 0; h < C; ++h) {
          // (a select on the entry would put its load behind a branch of its own)
          const int i = i0 + q * nw, j = j0 + 64 * h + lane;
          if (j < je && (TRI != 0 || j >= i) && (TRI != 1 || j < i))
#pragma unroll
            for (int v = 0; v < kMaxV; ++v)
              if (v < nv) a[v] += m[q][h] * x[v * xs + j];
        }
        if constexpr (kOnce) put(a, i0 + q * nw);
      }
    }
    if constexpr (!kOnce)
#pragma unroll
      for (int q = 0; q < R; ++q) put(acc[q], i0 + q * nw);
  }
}

template <int TRI = -1>
__device__ __forceinline__ void l_gemv_n(const double* __restrict__ M, int nrow, int ncol, int ld, const double* x, int xs, double* y,
                         int ys, int nv, double sgn) {
  if (ncol <= 0) return;
  if (ncol <= 64)
    l_gemv_n_rc<4, 1, TRI>(M, nrow, ncol, ld, x, xs, y, ys, nv, sgn);
  else if (ncol <= 128)
    l_gemv_n_rc<4, 2, TRI>(M, nrow, ncol, ld, x, xs, y, ys, nv, sgn);
  else if (ncol <= 256)
    l_gemv_n_rc<4, 4, TRI>(M, nrow, ncol, ld, x, xs, y, ys, nv, sgn);
  else
    l_gemv_n_rc<2, 8, TRI>(M, nrow, ncol, ld, x, xs, y, ys, nv, sgn);
}

// y[v*ys + j] += sgn * sum_i M[i*ld + j] x[v*xs + i]   (one thread per column).
// With few columns the waves split the rows: wave w takes column group
// w % ncg (64 columns) and row slice w / ncg (at least 8 rows each), and the
// slices add their partial sums in slice order (deterministic).  TRI >= 0 keeps
// one triangle: 2 the rows i > j, 3 the rows i <= j.  Every thread of the
// workgroup calls it; it ends synchronized.
template <int TRI = -1>
__device__ __forceinline__ void l_gemv_t(const double* __restrict__ M, int nrow, int ncol, int ld, const double* x, int xs, double* y,
                         int ys, int nv, double sgn) {
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  if (ncol <= 0 || nrow <= 0) {
    __syncthreads();
    return;
  }
  const int ncg = (ncol + 63) / 64;
  const bool split = ncg <= nw;
  const int nrs = split ? min((nrow + 7) / 8, nw / ncg) : 1;
  const int cg = split ? wv % ncg : 0, rs = split ? wv / ncg : 0;
  const bool active = !split || wv < ncg * nrs;
  const int ib = split ? (nrow * rs) / nrs : 0, ie = split ? (nrow * (rs + 1)) / nrs : nrow;
  double acc[kMaxV];
  for (int j = split ? cg * 64 + lane : threadIdx.x; active && j < ncol; j += split ? ncol : blockDim.x) {
#pragma unroll
    for (int v = 0; v < kMaxV; ++v) acc[v] = 0.0;
    for (int i0 = ib; i0 < ie; i0 += kU) {
      double mv[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) mv[u] = M[int64_t(min(i0 + u, ie - 1)) * ld + j];
#pragma unroll
      for (int u = 0; u < kU; ++u)
        if (i0 + u < ie) {
          if ((TRI != 2 || i0 + u > j) && (TRI != 3 || i0 + u <= j))
#pragma unroll
            for (int v = 0; v < kMaxV; ++v)
              if (v < nv) acc[v] += mv[u] * x[v * xs + i0 + u];
        }
    }
    if (!split)
#pragma unroll
      for (int v = 0; v < kMaxV; ++v)
        if (v < nv) y[v * ys + j] += sgn * acc[v];
  }
  if (split) {
    const int j = cg * 64 + lane;
    for (int p = 0; p < nrs; ++p) {
      __syncthreads();
      if (active && rs == p && j < ncol)
#pragma unroll
        for (int v = 0; v < kMaxV; ++v)
          if (v < nv) y[v * ys + j] += sgn * acc[v];
    }
  }
  __syncthreads();
}

// The value of lane l, a scalar.
__device__ __forceinline__ double lane_value(double x, int l) {
  const uint64_t b = uint64_t(__double_as_longlong(x));
  const uint32_t lo = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(b)), l));
  const uint32_t hi = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(b >> 32)), l));
  return __longlong_as_double((long long)((uint64_t(hi) << 32) | lo));
}

// One triangle of a diagonal block of at most kNbT rows, packed in LDS: entry
// (a, c) of a lower triangle at a (a + 1) / 2 + c, of an upper one the same
// with rows and columns reversed.  Triangular numbers are a permutation modulo
// a power of two, so a column is read without bank conflicts.
__host__ __device__ constexpr int tri_len(int nb) { return nb * (nb + 1) / 2; }

constexpr int kSu = 8;  // columns of the triangle read together

template <bool UPPER>
__device__ __forceinline__ int tri_at(int nb, int a, int c) {
  return UPPER ? tri_len(nb - 1 - a) + nb - 1 - c : tri_len(a) + c;
}

template <bool UPPER>
__device__ __forceinline__ void tri_stage(const double* __restrict__ LU, int n, int j0, double* tri) {
  const int nb = min(kNbT, n - j0);
  const double* M = LU + int64_t(j0) * n + j0;
  const int c = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  for (int a0 = w; a0 < nb; a0 += kU * nw) {
    double m[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) m[u] = M[int64_t(min(a0 + u * nw, nb - 1)) * n + min(c, nb - 1)];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int a = a0 + u * nw;
      if (a < nb && c < nb && (UPPER ? c >= a : c <= a)) tri[tri_at<UPPER>(nb, a, c)] = m[u];
    }
  }
}

// x = M^{-1} x, M a triangle of the row-major n x n LU: MODE 0 its unit lower
// L, 1 its upper U, 2 U^T, 3 L^T.  By blocks of 64 rows: a wave per right-hand
// side (or two) substitutes within the block, lane = row, each solved entry
// broadcast through a scalar register; then the rows not yet solved take the
// block's product.  The substitution is a chain of dependent steps, so its
// triangle is read from LDS (read from memory by rows, eight entries per lane
// at a time, and broadcast through LDS, a 64-row block took about 12 us).  The
// first triangle is in tri when this is called (tri_first, ordered by a
// barrier); the next is staged while the rows are updated.
template <int MODE>
__device__ __forceinline__ void tri_first(const double* __restrict__ LU, int n, double* tri) {
  if (n > 0) tri_stage<MODE == 1 || MODE == 2>(LU, n, MODE == 0 || MODE == 2 ? 0 : ((n - 1) / kNbT) * kNbT, tri);
}

template <int MODE>
__device__ __forceinline__ void l_solve(const double* __restrict__ LU, int n, double* x, int xs, int nv, double* tri) {
  constexpr bool kFwd = MODE == 0 || MODE == 2, kUp = MODE == 1 || MODE == 2;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  const int nblk = (n + kNbT - 1) / kNbT;
  for (int jb = 0; jb < nblk; ++jb) {
    const int j0 = (kFwd ? jb : nblk - 1 - jb) * kNbT, nb = min(kNbT, n - j0), row = min(lane, nb - 1);
    // a wave takes right-hand sides v and v + nw together: one read of each
    // entry of the triangle for both
    for (int v = wv; v < nv; v += 2 * nw) {
      auto pass = [&](auto two_c) {
        constexpr bool TWO = decltype(two_c)::value;
        double xi = x[v * xs + j0 + row], xj = TWO ? x[(v + nw) * xs + j0 + row] : 0.0;
        // a quotient is a product with the reciprocal and one correction
        double d = 1.0, di = 1.0;
        if constexpr (kUp) {
          d = tri[tri_at<true>(nb, row, row)];
          di = 1.0 / d;
        }
        auto quot = [&](double b) {
          const double q = b * di;
          return __builtin_fma(__builtin_fma(-q, d, b), di, q);
        };
        for (int c0 = 0; c0 < nb; c0 += kSu) {
          double m[kSu];
#pragma unroll
          for (int u = 0; u < kSu; ++u) {
            const int c = kFwd ? min(c0 + u, nb - 1) : max(nb - 1 - c0 - u, 0);
            // the entry of column c (of row c of U or L in the transposed
            // solves) that lane's row takes; any entry where it takes none
            if constexpr (MODE == 0) m[u] = tri[tri_at<false>(nb, max(row, c), c)];
            if constexpr (MODE == 1) m[u] = tri[tri_at<true>(nb, min(row, c), c)];
            if constexpr (MODE == 2) m[u] = tri[tri_at<true>(nb, c, max(row, c))];
            if constexpr (MODE == 3) m[u] = tri[tri_at<false>(nb, c, min(row, c))];
          }
#pragma unroll
          for (int u = 0; u < kSu; ++u)
            if (c0 + u < nb) {
              const int c = kFwd ? c0 + u : nb - 1 - c0 - u;
              if constexpr (kUp) {
                const double qi = quot(xi);
                xi = lane == c ? qi : xi;
                if constexpr (TWO) {
                  const double qj = quot(xj);
                  xj = lane == c ? qj : xj;
                }
              }
              const bool take = kFwd ? lane > c : lane < c;
              const double ti = xi - m[u] * lane_value(xi, c);
              xi = take ? ti : xi;
              if constexpr (TWO) {
                const double tj = xj - m[u] * lane_value(xj, c);
                xj = take ? tj : xj;
              }
            }
        }
        if constexpr (kUp) {
          // Not so where the reciprocal is no normal number or its product with
          // an entry is infinite (the correction then makes NaN): those blocks
          // are done again.
          const bool fine = __builtin_amdgcn_class(di, 0x108) && __builtin_fabs(xi) < __builtin_inf() &&
                            (!TWO || __builtin_fabs(xj) < __builtin_inf());
          if (!__all(fine)) return false;
        }
        if (lane < nb) {
          x[v * xs + j0 + lane] = xi;
          if constexpr (TWO) x[(v + nw) * xs + j0 + lane] = xj;
        }
        return true;
      };
      if (v + nw < nv ? pass(std::true_type{}) : pass(std::false_type{})) [[likely]]
        continue;
      if constexpr (kUp)
        for (int w = v; w < min(nv, v + 2 * nw); w += nw) {  // by divisions
          const double d = tri[tri_at<true>(nb, row, row)];
          double xi = x[w * xs + j0 + row];
#pragma clang loop unroll(disable)
          for (int u = 0; u < nb; ++u) {
            const int c = kFwd ? u : nb - 1 - u;
            const double m = tri[kFwd ? tri_at<true>(nb, c, max(row, c)) : tri_at<true>(nb, min(row, c), c)];
            if (lane == c) xi = xi / d;
            const double xc = lane_value(xi, c);
            if (kFwd ? lane > c : lane < c) xi -= m * xc;
          }
          if (lane < nb) x[w * xs + j0 + lane] = xi;
        }
    }
    __syncthreads();
    if (jb + 1 < nblk) {
      tri_stage<kUp>(LU, n, kFwd ? j0 + kNbT : j0 - kNbT, tri);
      const int rest = n - j0 - nb;
      if constexpr (MODE == 0)  // the rows below: x_i -= L(i, block) x_block
        l_gemv_n(LU + int64_t(j0 + nb) * n + j0, rest, nb, n, x + j0, xs, x + j0 + nb, xs, nv, -1.0);
      if constexpr (MODE == 1)  // the rows above: x_i -= U(i, block) x_block
        l_gemv_n(LU + j0, j0, nb, n, x + j0, xs, x, xs, nv, -1.0);
      if constexpr (MODE == 2)  // the entries below: x_i -= sum_c U(j0 + c, i) x_{j0 + c}
        l_gemv_t(LU + int64_t(j0) * n + j0 + nb, nb, rest, n, x + j0, xs, x + j0 + nb, xs, nv, -1.0);
      if constexpr (MODE == 3)  // the entries above: x_i -= sum_c L(j0 + c, i) x_{j0 + c}
        l_gemv_t(LU + int64_t(j0) * n, nb, j0, n, x + j0, xs, x, xs, nv, -1.0);
      __syncthreads();
    }
  }
}

// x = M x through the scratch tp (both [nv][n] in LDS), M a triangle of the
// row-major n x n LU: mode 0 U (columns j >= i), 1 the unit lower L (x_i plus
// columns j < i), both one wave per row; mode 2 the unit upper L^T (x_i plus
// rows j > i of L), 3 U^T (rows j <= i of U), both one thread per column.
__device__ __forceinline__ void l_trmv(const double* __restrict__ LU, int n, double* x, double* tp, int nv, int mode) {
  for (int e = threadIdx.x; e < nv * n; e += blockDim.x) tp[e] = mode == 1 || mode == 2 ? x[e] : 0.0;
  __syncthreads();
  if (mode == 0)
    l_gemv_n<0>(LU, n, n, n, x, n, tp, n, nv, 1.0);
  else if (mode == 1)
    l_gemv_n<1>(LU, n, n, n, x, n, tp, n, nv, 1.0);
  else if (mode == 2)
    l_gemv_t<2>(LU, n, n, n, x, n, tp, n, nv, 1.0);
  else
    l_gemv_t<3>(LU, n, n, n, x, n, tp, n, nv, 1.0);
  __syncthreads();
  for (int e = threadIdx.x; e < nv * n; e += blockDim.x) x[e] = tp[e];
  __syncthreads();
}

// x = P x (fwd) or P^T x through the scratch tp, both [nv][n] in LDS.
__device__ __forceinline__ void l_permute(const int32_t* perm, int n, double* x, double* tp, int nv, bool fwd) {
  for (int e = threadIdx.x; e < nv * n; e += blockDim.x) {
    const int v = e / n, i = e % n;
    if (fwd)
      tp[e] = x[v * n + perm[i]];
    else
      tp[v * n + perm[i]] = x[e];
  }
  __syncthreads();
  for (int e = threadIdx.x; e < nv * n; e += blockDim.x) x[e] = tp[e];
  __syncthreads();
}

// One group per workgroup of 64 .. 1024 threads; OP 0 solve, 1 solve_T, 2 apply,
// 3 apply_T (the per-group steps in the header of this file); DOWN: the
// downward sweep, else the upward one (finest sub-level first).  The LDS
// holds cap doubles (sized by the launch to the sub-level's largest record)
// and, in the solves, a diagonal block; the caller guarantees 2r + k <= cap.
// Registers are capped for 4 waves per SIMD: 1024 records of 256 threads
// then all run at once, 4 per CU.  Bound by the chain of a record's steps,
// each a wait for memory.  A kernel per sweep, triangles through LDS, sums
// across lanes in the vector ALU and column products split over all waves:
// the sub-levels of a 512^2 solve 885 -> 844 us, of the four 24^3 sweeps 588
// -> 505 us.
template <int OP, bool DOWN>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4))) void k_sweep_lds(SwArgs A, int cap) {
  extern __shared__ double sm[];
  double* tri = sm + cap;  // the solves' diagonal block
  const GroupRec R = A.recs[blockIdx.x];
  const int r = R.r, k = R.k;
  const int32_t* rd = A.iarena + R.idx;
  const int32_t* sk = rd + r;
  const int32_t* perm = sk + k + r;
  const double* T = A.darena + R.off;
  const double* Lsr = T + int64_t(k) * r;
  const double* Urs = Lsr + int64_t(k) * r;
  const double* LU = Urs + int64_t(r) * k;
  const int64_t N = A.N;
  const int tid = threadIdx.x, bs = blockDim.x;
  const int nvb = max(1, min(A.nrhs, cap / (2 * r + k)));
  for (int v0 = 0; v0 < A.nrhs; v0 += nvb) {
    const int nv = min(nvb, A.nrhs - v0);
    double* xr = sm;           // [nv][r]
    double* xs = sm + nv * r;  // [nv][k]
    double* tp = xs + nv * k;  // [nv][r]
    // the first diagonal block of the solves, on its way with the vectors
    if constexpr (OP < 2) tri_first<2 * OP + int(DOWN)>(LU, r, tri);
    double* u = A.u + v0 * N;
    for (int e = tid; e < nv * r; e += bs) xr[e] = u[(e / r) * N + rd[e % r]];
    for (int e = tid; e < nv * k; e += bs) xs[e] = u[(e / k) * N + sk[e % k]];
    __syncthreads();
    if constexpr (OP == 0 && !DOWN) {
      if (k > 0) l_gemv_t(T, k, r, r, xs, k, xr, r, nv, -1.0);  // u_r -= T^T u_s
      __syncthreads();
      l_permute(perm, r, xr, tp, nv, true);                     // u_r = P u_r
      l_solve<0>(LU, r, xr, r, nv, tri);                        // u_r = L^{-1} u_r
      if (k > 0) l_gemv_n(Lsr, k, r, r, xr, r, xs, k, nv, -1.0);  // u_s -= L_sr u_r
    } else if constexpr (OP == 0) {
      if (k > 0) l_gemv_n(Urs, r, k, k, xs, k, xr, r, nv, -1.0);  // u_r -= U_rs u_s
      __syncthreads();
      l_solve<1>(LU, r, xr, r, nv, tri);                           // u_r = U^{-1} u_r
      if (k > 0) l_gemv_n(T, k, r, r, xr, r, xs, k, nv, -1.0);    // u_s -= T u_r
    } else if constexpr (OP == 1 && !DOWN) {
      if (k > 0) l_gemv_t(T, k, r, r, xs, k, xr, r, nv, -1.0);    // u_r -= T^T u_s
      __syncthreads();
      l_solve<2>(LU, r, xr, r, nv, tri);                           // u_r = U^{-T} u_r
      if (k > 0) l_gemv_t(Urs, r, k, k, xr, r, xs, k, nv, -1.0);  // u_s -= U_rs^T u_r
    } else if constexpr (OP == 1) {
      if (k > 0) l_gemv_t(Lsr, k, r, r, xs, k, xr, r, nv, -1.0);  // u_r -= L_sr^T u_s
      __syncthreads();
      l_solve<3>(LU, r, xr, r, nv, tri);                           // u_r = L^{-T} u_r
      l_permute(perm, r, xr, tp, nv, false);                       // u_r = P^T u_r
      if (k > 0) l_gemv_n(T, k, r, r, xr, r, xs, k, nv, -1.0);    // u_s -= T u_r
    } else if constexpr (OP == 2 && !DOWN) {
      if (k > 0) l_gemv_n(T, k, r, r, xr, r, xs, k, nv, 1.0);     // x_s += T x_r
      __syncthreads();
      l_trmv(LU, r, xr, tp, nv, 0);                                // x_r = U x_r
      if (k > 0) l_gemv_n(Urs, r, k, k, xs, k, xr, r, nv, 1.0);   //     + U_rs x_s
    } else if constexpr (OP == 2) {
      if (k > 0) l_gemv_n(Lsr, k, r, r, xr, r, xs, k, nv, 1.0);   // y_s += L_sr y_r
      __syncthreads();
      l_trmv(LU, r, xr, tp, nv, 1);                                // y_r = L y_r
      l_permute(perm, r, xr, tp, nv, false);                       // y_r = P^T y_r
      if (k > 0) l_gemv_t(T, k, r, r, xs, k, xr, r, nv, 1.0);     // y_r += T^T y_s
    } else if constexpr (!DOWN) {
      if (k > 0) l_gemv_n(T, k, r, r, xr, r, xs, k, nv, 1.0);     // x_s += T x_r
      __syncthreads();
      l_permute(perm, r, xr, tp, nv, true);                        // x_r = P x_r
      l_trmv(LU, r, xr, tp, nv, 2);                                // x_r = L^T x_r
      if (k > 0) l_gemv_t(Lsr, k, r, r, xs, k, xr, r, nv, 1.0);   //     + L_sr^T x_s
    } else {
      if (k > 0) l_gemv_t(Urs, r, k, k, xr, r, xs, k, nv, 1.0);   // y_s += U_rs^T y_r
      __syncthreads();
      l_trmv(LU, r, xr, tp, nv, 3);                                // y_r = U^T y_r
      if (k > 0) l_gemv_t(T, k, r, r, xs, k, xr, r, nv, 1.0);     // y_r += T^T y_s
    }
    __syncthreads();
    for (int e = tid; e < nv * r; e += bs) u[(e / r) * N + rd[e % r]] = xr[e];
    for (int e = tid; e < nv * k; e += bs) u[(e / k) * N + sk[e % k]] = xs[e];
    __syncthreads();
  }
}

// Top block: x = A_L^{-1} x (op 0), A_L^{-T} x (op 1), A_L x (op 2) or
// A_L^T x (op 3) with A_L = P^T L U; n < kTopSplitMin.
__global__ __launch_bounds__(1024) void k_top_lds(const double* LU, const int32_t* perm, int n, const int32_t* idx,
                                                  double* u, int64_t N, int nrhs, int op) {
  __shared__ double sm[2 * kTopSplitMin * kMaxV];
  __shared__ double tri[tri_len(kNbT)];
  const int tid = threadIdx.x, B = blockDim.x;
  for (int v0 = 0; v0 < nrhs; v0 += kMaxV) {
    const int nv = min(kMaxV, nrhs - v0);
    double* x = sm;
    double* tp = sm + nv * n;
    double* uu = u + v0 * N;
    for (int e = tid; e < nv * n; e += B) x[e] = uu[(e / n) * N + idx[e % n]];
    if (op == 0) tri_first<0>(LU, n, tri);
    if (op == 1) tri_first<2>(LU, n, tri);
    __syncthreads();
    if (op == 0) {
      l_permute(perm, n, x, tp, nv, true);
      l_solve<0>(LU, n, x, n, nv, tri);
      tri_first<1>(LU, n, tri);
      __syncthreads();
      l_solve<1>(LU, n, x, n, nv, tri);
    } else if (op == 1) {
      l_solve<2>(LU, n, x, n, nv, tri);
      tri_first<3>(LU, n, tri);
      __syncthreads();
      l_solve<3>(LU, n, x, n, nv, tri);
      l_permute(perm, n, x, tp, nv, false);
    } else if (op == 2) {
      l_trmv(LU, n, x, tp, nv, 0);
      l_trmv(LU, n, x, tp, nv, 1);
      l_permute(perm, n, x, tp, nv, false);
    } else {
      l_permute(perm, n, x, tp, nv, true);
      l_trmv(LU, n, x, tp, nv, 2);
      l_trmv(LU, n, x, tp, nv, 3);
    }
    for (int e = tid; e < nv * n; e += B) uu[(e / n) * N + idx[e % n]] = x[e];
    __syncthreads();
  }
}

// The same for a top block of any size, on the vectors where they stand (two of
// them with the scratch): one workgroup, for handles whose memory cap left no
// room for what the many-workgroup solves keep.
__global__ __launch_bounds__(1024) void k_top(const double* LU, const int32_t* piv, int n, const int32_t* idx, double* u,
                                              double* work, int64_t N, int nrhs, int op) {
  if (op == 0) {
    swaps_fwd(piv, n, idx, u, N, nrhs);
    solve_L(LU, n, idx, u, N, nrhs);
    solve_U(LU, n, idx, u, N, nrhs);
  } else if (op == 1) {
    solve_UT(LU, n, idx, u, N, nrhs);
    solve_LT(LU, n, idx, u, N, nrhs);
    swaps_rev(piv, n, idx, u, N, nrhs);
  } else if (op == 2) {
    tri_mul(LU, n, idx, u, work, N, nrhs, 0);
    tri_mul(LU, n, idx, u, work, N, nrhs, 1);
    swaps_rev(piv, n, idx, u, N, nrhs);
  } else {
    swaps_fwd(piv, n, idx, u, N, nrhs);
    tri_mul(LU, n, idx, u, work, N, nrhs, 2);
    tri_mul(LU, n, idx, u, work, N, nrhs, 3);
  }
}

// Gather form of the row interchanges j <-> piv[j], j = 0..n-1 (in order).
constexpr int kPermLds = 8192;
__device__ void make_perm(const int32_t* piv, int32_t* perm, int n) {
  __shared__ int32_t sp[kPermLds];
  __shared__ int32_t spv[kPermLds];
  if (n <= kPermLds) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
      sp[i] = i;
      spv[i] = piv[i];
    }
    __syncthreads();
    if (threadIdx.x == 0)
      for (int j = 0; j < n; ++j) {
        const int p = spv[j];
        const int t = sp[j];
        sp[j] = sp[p];
        sp[p] = t;
      }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += blockDim.x) perm[i] = sp[i];
  } else {
    for (int i = threadIdx.x; i < n; i += blockDim.x) perm[i] = i;
    __syncthreads();
    if (threadIdx.x == 0)
      for (int j = 0; j < n; ++j) {
        const int p = piv[j];
        const int t = perm[j];
        perm[j] = perm[p];
        perm[p] = t;
      }
  }
}

__global__ __launch_bounds__(64) void k_make_perm(const GroupRec* recs, int32_t* iarena) {
  const GroupRec R = recs[blockIdx.x];
  int32_t* piv = iarena + R.idx + R.r + R.k;
  make_perm(piv, piv + R.r, R.r);
}

__global__ __launch_bounds__(64) void k_make_perm_top(const int32_t* piv, int32_t* perm, int n) {
  make_perm(piv, perm, n);
}

// The top block's solve record: indices, interchanges, gather permutation.
__global__ void k_top_record(const int32_t* idx, const int32_t* piv, const int32_t* perm, int r, int32_t* iarena,
                             GroupRec* rec, int64_t* woff) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) {
    *rec = GroupRec{r, 0, 0, 0};
    *woff = 0;
  }
  if (i >= r) return;
  iarena[i] = idx[i];
  iarena[r + i] = piv[i];
  iarena[2 * r + i] = perm[i];
}

__global__ void k_copy(const double* x, double* y, int64_t n) {
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x)
    y[i] = x[i];
}

// ---------------------------------------------------------------------------
// Solve and transposed solve (op 0, 1) for sub-levels with few, large
// records: each record is spread over many workgroups and all right-hand
// sides go through its factors in one pass (the LDS kernel above holds
// 2r + k entries per right-hand side and so rereads large factors once per
// right-hand side).  Per record, B holds the right-hand sides of the
// triangular solve and X its solution, both [nv][r] at nv * woff in the work
// buffer.  The products with T, L_sr and U_rs are spread over many
// workgroups per record; the triangular solve of every record of the pass is
// one launch of workgroups that hand 64-row blocks of X to each other
// (k_sp_chain).
// ---------------------------------------------------------------------------
struct SpArgs {
  const GroupRec* recs;
  const int32_t* iarena;
  const double* darena;
  const int64_t* woff;
  double* u;  // [nv][N]
  double* B;
  double* X;
  int64_t N;
  int nv;
  const double* dinv;  // diagonal-block inverses (SubLevel::dinv layout)
  int dnb;             // blocks per record in dinv
  // Ticket counter of the chained triangular solve (two of them where a top
  // block's two solves follow each other).
  uint32_t* sync = nullptr;
  int nbm = 0;  // blocks of the largest record
  long long wait_ticks = 0;  // bound on each wait, in ticks of the 100 MHz constant clock
};

struct SpRec {
  int r, k;
  const int32_t *rd, *sk, *perm;
  const double *T, *Lsr, *Urs, *LU;
  double *B, *X;
};

__device__ __forceinline__ SpRec sp_rec(const SpArgs& A, int i) {
  const GroupRec R = A.recs[i];
  SpRec v;
  v.r = R.r;
  v.k = R.k;
  v.rd = A.iarena + R.idx;
  v.sk = v.rd + R.r;
  v.perm = v.sk + R.k + R.r;
  v.T = A.darena + R.off;
  v.Lsr = v.T + int64_t(R.k) * R.r;
  v.Urs = v.Lsr + int64_t(R.k) * R.r;
  v.LU = v.Urs + int64_t(R.r) * R.k;
  v.B = A.B + A.nv * A.woff[i];
  v.X = A.X + A.nv * A.woff[i];
  return v;
}

// The first kernel of a pass readies the chained solve that follows it:
// workgroup (0, 0) clears the ticket counter, and every workgroup marks its
// rows of X pending (rows i0 .. i0 + nrow - 1 of each right-hand side).  The
// next launch on the stream sees both.
constexpr uint64_t kXPending = 0x7FF4A3B2C1D0E0F1ull;  // a signaling NaN: no arithmetic result
__device__ __forceinline__ void sp_ready_chain(const SpArgs& A, const SpRec& R, int i0, int nrow) {
  if (!A.sync) return;
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) A.sync[0] = 0u;
  const int n = min(nrow, R.r - i0);
  uint64_t* X = reinterpret_cast<uint64_t*>(R.X);
  for (int e = threadIdx.x; e < A.nv * n; e += blockDim.x) X[(e / n) * R.r + i0 + e % n] = kXPending;
}

// Where a vector of a record's redundant unknowns is read or written: its X
// or B block of the work buffer, or the right-hand sides themselves through
// the record's indices (u_r, or P u_r with the row interchanges).
enum SpVec { kInX = 0, kInB = 1, kInU = 2, kInPu = 3 };

__device__ __forceinline__ double* sp_at(const SpArgs& A, const SpRec& R, int where, int v, int i) {
  if (where >= kInU) return A.u + v * A.N + R.rd[where == kInPu ? R.perm[i] : i];
  return (where == kInX ? R.X : R.B) + int64_t(v) * R.r + i;
}

constexpr int kSpChunk = 512;  // skeleton entries staged in LDS per pass

// The product of a 64 x 16 tile of a matrix with 16 entries of each right-hand
// side, one wave.  One right-hand side: lane = row, the entries of x broadcast
// through scalar registers (read from LDS, they would cost a broadcast read
// per entry and wave, and the one LDS of a CU bounds its four SIMDs).  Up to
// 8: matrix instructions, 16 of 64 cycles, whose 16 columns hold the
// right-hand sides (columns 8 .. 15 are ignored).  Broadcasts cost 128
// products, 256 lane reads and their wait states, three times as long.
//   m[q]:  entry (row(q), col(q)) of the tile
//   x[s]:  entry col_x(s) of right-hand side rhs()
using d4 = double __attribute__((ext_vector_type(4)));
template <int NV>
struct SpTile {
  static_assert(NV == 1 || NV == kMaxV, "one right-hand side, or a pass of up to kMaxV");
  static constexpr int kNx = NV == 1 ? 1 : 4;
  static constexpr int kLd = 66;  // row of sums or entries in LDS, padded against bank conflicts
  double s = 0.0;
  d4 a[NV == 1 ? 1 : 4] = {};

  static __device__ __forceinline__ int row(int q) {
    return NV == 1 ? int(threadIdx.x & 63) : 16 * (q >> 2) + int(threadIdx.x & 15);
  }
  static __device__ __forceinline__ int col(int q) { return NV == 1 ? q : 4 * (q & 3) + int(threadIdx.x & 63) / 16; }
  static __device__ __forceinline__ int rhs() { return NV == 1 ? 0 : int(threadIdx.x & 15); }
  static __device__ __forceinline__ int col_x(int s) {
    return NV == 1 ? int(threadIdx.x & 15) : 4 * s + int(threadIdx.x & 63) / 16;
  }
  __device__ __forceinline__ void mul(const double (&m)[16], const double (&x)[kNx]) {
    if constexpr (NV == 1) {
#pragma unroll
      for (int q = 0; q < 16; ++q) s += m[q] * lane_value(x[0], q);
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int t = 0; t < 4; ++t) a[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(m[4 * t + k], x[k], a[t], 0, 0, 0);
    }
  }
  // the 64 sums of each right-hand side
  __device__ __forceinline__ void put(double (*dst)[kLd]) const {
    const int lane = threadIdx.x & 63;
    if constexpr (NV == 1) {
      dst[0][lane] = s;
    } else if ((lane & 15) < NV) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) dst[lane & 15][16 * t + 4 * e + lane / 16] = a[t][e];
    }
  }
};

// acc += sum_{j < n} M(j, ib + l) x(v, j) for the 64 columns ib + l of the
// workgroup, clamped to column nc - 1 (M row-major, leading dimension ld): the
// waves take 16 rows j each in turn, 16 coalesced loads in flight per wave and
// no barrier; x(v, j) is read where x stands.  colmap (if given) is the column
// read in place of ib + l.  TRI >= 0 keeps one triangle of a matrix whose row
// 0 is jb: 2 the rows jb + j > ib + l, 3 the rows jb + j <= ib + l.
template <int NV, int TRI = -1, typename X>
__device__ __forceinline__ void sp_cols_acc(const double* M, int64_t ld, int ib, int nc, int n, int nv,
                                            SpTile<NV>& acc, X x, const int32_t* colmap = nullptr, int jb = 0) {
  using T = SpTile<NV>;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  constexpr int kCols = NV == 1 ? 1 : 4;  // columns of a lane
  int c[kCols];
#pragma unroll
  for (int t = 0; t < kCols; ++t) {
    c[t] = min(ib + T::row(4 * t), nc - 1);
    if (colmap) c[t] = colmap[c[t]];
  }
  for (int j0 = wv * 16; j0 < n; j0 += nw * 16) {
    double m[16], xv[T::kNx];
#pragma unroll
    for (int q = 0; q < 16; ++q) m[q] = M[int64_t(min(j0 + T::col(q), n - 1)) * ld + c[NV == 1 ? 0 : q >> 2]];
#pragma unroll
    for (int k = 0; k < T::kNx; ++k) {
      const int j = j0 + T::col_x(k);
      xv[k] = j < n && T::rhs() < nv ? x(T::rhs(), j) : 0.0;
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int j = j0 + T::col(q), i = ib + T::row(q);
      if (j >= n || (TRI == 2 && jb + j <= i) || (TRI == 3 && jb + j > i)) m[q] = 0.0;
    }
    acc.mul(m, xv);
  }
}

// The waves' sums of a workgroup's 64 columns, added in wave order: out(v, l)
// is called with the total of column l of right-hand side v.
constexpr int kSpColWaves = 16;
template <int NV, typename O>
__device__ __forceinline__ void sp_cols_out(const SpTile<NV>& acc, int nv, O out) {
  __shared__ double sred[kSpColWaves][NV][SpTile<NV>::kLd];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  acc.put(sred[wv]);
  __syncthreads();
  for (int v = wv; v < nv; v += kSpColWaves) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kSpColWaves; ++w) t += sred[w][v][lane];
    out(v, lane, t);
  }
}

// The sums over the wave of acc[q][v] (4 rows q of the wave, kMaxV
// right-hand sides) in one reduce-scatter: returns the total of row q =
// lane >> 4, right-hand side v = (lane >> 1) & 7, held by lanes 2c and
// 2c + 1 (c = 8q + v).
__device__ __forceinline__ double sp_rows_sum(const double (&acc)[4][kMaxV]) {
  double p[kRs];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int v = 0; v < kMaxV; ++v) p[q * kMaxV + v] = acc[q][v];
  return wave_rs32(p);
}

// dst[v][e] = src(v, e) for e < n, v < nv, with src(v, e) = base[v ld + idx[e]]
// (idx given) or base[v ld + e]: an entry per thread and step, its index
// loaded once and its right-hand sides' loads issued together before any is
// stored (the caller synchronizes before the block is read).
__device__ __forceinline__ void sp_stage(const double* base, int64_t ld, const int32_t* idx, int n, int nv,
                                         double (*dst)[kSpChunk]) {
  for (int e = threadIdx.x; e < n; e += blockDim.x) {
    const int64_t g = idx ? int64_t(idx[e]) : int64_t(e);
    double t[kMaxV];
#pragma unroll
    for (int v = 0; v < kMaxV; ++v) t[v] = v < nv ? base[v * ld + g] : 0.0;
#pragma unroll
    for (int v = 0; v < kMaxV; ++v)
      if (v < nv) dst[v][e] = t[v];
  }
}

// The same of entries c0 .. c0 + n - 1 of a record's vector.
__device__ __forceinline__ void sp_stage_vec(const SpArgs& A, const SpRec& R, int where, int c0, int n,
                                             double (*dst)[kSpChunk]) {
  if (where == kInX || where == kInB)
    sp_stage((where == kInX ? R.X : R.B) + c0, R.r, nullptr, n, A.nv, dst);
  else
    for (int e = threadIdx.x; e < n; e += blockDim.x) {
      const int64_t g = R.rd[where == kInPu ? R.perm[c0 + e] : c0 + e];
      double t[kMaxV];
#pragma unroll
      for (int v = 0; v < kMaxV; ++v) t[v] = v < A.nv ? A.u[v * A.N + g] : 0.0;
#pragma unroll
      for (int v = 0; v < kMaxV; ++v)
        if (v < A.nv) dst[v][e] = t[v];
    }
}

// acc[q][v] += sum_{c < nc} mr[q][c] s[v][c] for a wave's 4 rows q (mr[q] null
// past the record; its sums are then never used), lane c = lane, lane + 64, ...
// The loads of the 4 rows and of two column steps are issued together before
// any is used; each acc[q][v] still adds its terms in increasing c.  TRI >= 0
// keeps one triangle of rows iq[q] (column c0 + c): 0 the upper one with the
// diagonal, 1 the strictly lower one; the other entries count as zero.
template <int TRI = -1>
__device__ __forceinline__ void sp_rows4_acc(const double* const (&mr)[4], int nc, const double (*s)[kSpChunk], int nv,
                                             double (&acc)[4][kMaxV], int c0 = 0, const int* iq = nullptr) {
  const int lane = threadIdx.x & 63;
  for (int c = lane; c < nc; c += 128) {
    double m[2][4];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int cc = c + 64 * u;
        bool keep = mr[q] && cc < nc;
        if constexpr (TRI == 0) keep = keep && c0 + cc >= iq[q];
        if constexpr (TRI == 1) keep = keep && c0 + cc < iq[q];
        m[u][q] = keep ? mr[q][cc] : 0.0;
      }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int cc = c + 64 * u;
      if (cc < nc)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int v = 0; v < kMaxV; ++v)
            if (v < nv) acc[q][v] += m[u][q] * s[v][cc];
    }
  }
}

// Readies the chained solves of a pass that has no product before them (the
// top block): X and B pending, both ticket counters zero.
__global__ __launch_bounds__(256) void k_sp_ready(SpArgs A) {
  const SpRec R = sp_rec(A, blockIdx.y);
  const int i0 = blockIdx.x * 64;
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < 2) A.sync[threadIdx.x] = 0u;
  const int n = min(64, R.r - i0);
  for (int e = threadIdx.x; e < A.nv * n; e += blockDim.x) {
    const int64_t o = int64_t(e / n) * R.r + i0 + e % n;
    reinterpret_cast<uint64_t*>(R.X)[o] = kXPending;
    reinterpret_cast<uint64_t*>(R.B)[o] = kXPending;
  }
}

// First step of an up pass (and of the transposed solve's down pass), column
// form: B(v, i) = u_r(v, c) - (M^T u_s)(v, c) with c = perm[i] (PERM: the
// row interchanges of the solve, B = P(u_r - T^T u_s)) or c = i, and
// M = T (k x r), or L_sr with LSR.  With ADD instead u_r(v, i) += (M^T u_s)(v, i)
// in place (the last step of the apply sweeps' down pass).  64 rows i per
// workgroup, lane per row, the sum over the skeleton split between its 16
// waves.
template <bool LSR, bool PERM, bool ADD, int NV>
__global__ __launch_bounds__(kSpColWaves * 64) void k_sp_first_cols(SpArgs A) {
  const SpRec R = sp_rec(A, blockIdx.y);
  const int lane = threadIdx.x & 63, ib = blockIdx.x * 64;
  if (!ADD) sp_ready_chain(A, R, ib, 64);
  if (ib >= R.r) return;
  const int i = min(ib + lane, R.r - 1), c = PERM ? R.perm[i] : i;
  SpTile<NV> acc;
  sp_cols_acc<NV>(LSR ? R.Lsr : R.T, R.r, ib, R.r, R.k, A.nv, acc,
                  [&](int v, int j) { return A.u[v * A.N + R.sk[j]]; }, PERM ? R.perm : nullptr);
  sp_cols_out<NV>(acc, A.nv, [&](int v, int l, double t) {
    if (ib + l >= R.r) return;
    double* ur = A.u + v * A.N + R.rd[c];
    if (ADD)
      *ur += t;
    else
      R.B[int64_t(v) * R.r + ib + l] = *ur - t;
  });
}

// Down, first step of the solve: B(v, i) = (u_r - U_rs u_s)(v, i), one wave
// per row i.
__global__ __launch_bounds__(256) void k_sp_down_first(SpArgs A) {
  const SpRec R = sp_rec(A, blockIdx.y);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int i0 = blockIdx.x * 16;  // 16 rows per workgroup, 4 per wave
  sp_ready_chain(A, R, i0, 16);
  if (i0 >= R.r) return;
  const int nv = A.nv;
  __shared__ double sus[kMaxV][kSpChunk];
  double acc[4][kMaxV];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int v = 0; v < kMaxV; ++v) acc[q][v] = 0.0;
  for (int j0 = 0; j0 < R.k; j0 += kSpChunk) {
    const int nj = min(kSpChunk, R.k - j0);
    __syncthreads();
    sp_stage(A.u, A.N, R.sk + j0, nj, nv, sus);
    __syncthreads();
    const double* mr[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = i0 + wv * 4 + q;
      mr[q] = i < R.r ? R.Urs + int64_t(i) * R.k + j0 : nullptr;
    }
    sp_rows4_acc(mr, nj, sus, nv, acc);
  }
  {
    const double t = sp_rows_sum(acc);
    const int i = i0 + wv * 4 + (lane >> 4), v = (lane >> 1) & 7;
    if ((lane & 1) == 0 && i < R.r && v < nv) R.B[v * R.r + i] = A.u[v * A.N + R.rd[i]] - t;
  }
}

// u_s += sgn M x (M = L_sr or T, k x r), one wave per skeleton row; x is X,
// or with GATHER the record's u_r read through its indices; staged in LDS by
// chunks of columns.
template <bool GATHER>
__global__ __launch_bounds__(256) void k_sp_skel_update(SpArgs A, int which, double sgn) {
  const SpRec R = sp_rec(A, blockIdx.y);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int j0 = blockIdx.x * 16;
  if (j0 >= R.k) return;
  const int nv = A.nv;
  const double* M = which ? R.T : R.Lsr;
  __shared__ double sx[kMaxV][kSpChunk];
  double acc[4][kMaxV];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int v = 0; v < kMaxV; ++v) acc[q][v] = 0.0;
  for (int c0 = 0; c0 < R.r; c0 += kSpChunk) {
    const int nc = min(kSpChunk, R.r - c0);
    __syncthreads();
    if (GATHER)
      sp_stage(A.u, A.N, R.rd + c0, nc, nv, sx);
    else
      sp_stage(R.X + c0, R.r, nullptr, nc, nv, sx);
    __syncthreads();
    const double* mr[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int j = j0 + wv * 4 + q;
      mr[q] = j < R.k ? M + int64_t(j) * R.r + c0 : nullptr;
    }
    sp_rows4_acc(mr, nc, sx, nv, acc);
  }
  {
    const double t = sp_rows_sum(acc);
    const int j = j0 + wv * 4 + (lane >> 4), v = (lane >> 1) & 7;
    if ((lane & 1) == 0 && j < R.k && v < nv) A.u[v * A.N + R.sk[j]] += sgn * t;
  }
}

// u_s += sgn U_rs^T x (U_rs r x k), x = X or with GATHER the record's u_r
// read through its indices: lane per skeleton entry j, 64 per workgroup, the
// sum over the rows of U_rs split between its 16 waves.
template <bool GATHER, int NV>
__global__ __launch_bounds__(kSpColWaves * 64) void k_sp_skel_update_T(SpArgs A, double sgn) {
  const SpRec R = sp_rec(A, blockIdx.y);
  const int jb = blockIdx.x * 64;
  if (jb >= R.k) return;
  SpTile<NV> acc;
  sp_cols_acc<NV>(R.Urs, R.k, jb, R.k, R.r, A.nv, acc,
                  [&](int v, int i) { return *sp_at(A, R, GATHER ? kInU : kInX, v, i); });
  sp_cols_out<NV>(acc, A.nv, [&](int v, int l, double t) {
    if (jb + l < R.k) A.u[v * A.N + R.sk[jb + l]] += sgn * t;
  });
}

// B = u_r, or with PERM B = P u_r (B[i] = u_r[perm[i]]).
template <bool PERM>
__global__ __launch_bounds__(256) void k_sp_gather(SpArgs A) {
  const SpRec R = sp_rec(A, blockIdx.y);
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= R.r) return;
  const int d = R.rd[PERM ? R.perm[i] : i];
  for (int v = 0; v < A.nv; ++v) R.B[v * R.r + i] = A.u[v * A.N + d];
}

// The triangular products of the apply sweeps (and the rectangular ones
// beside them), for few large records, from vector src to vector dst of the
// record (not the same one).  Row form: out(v, i) = (M x)(v, i) [+ (U_rs u_s)(v, i)]
// with M the upper U of the record's LU (TRI 0, columns j >= i) or its unit
// lower L (TRI 1, x_i plus the columns j < i); one wave per row i, 16 rows
// per workgroup, x and u_s staged in LDS by chunks.
template <int TRI, bool RECT>
__global__ __launch_bounds__(256) void k_sp_rowmv(SpArgs A, int src, int dst) {
  const SpRec R = sp_rec(A, blockIdx.y);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int i0 = blockIdx.x * 16;
  if (i0 >= R.r) return;
  const int nv = A.nv, r = R.r;
  __shared__ double sx[kMaxV][kSpChunk];
  double acc[4][kMaxV];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int v = 0; v < kMaxV; ++v) acc[q][v] = 0.0;
  // the columns the workgroup's rows reach
  const int cb = TRI == 0 ? i0 : 0, ce = TRI == 0 ? r : min(r, i0 + 16);
  for (int c0 = cb; c0 < ce; c0 += kSpChunk) {
    const int nc = min(kSpChunk, ce - c0);
    __syncthreads();
    sp_stage_vec(A, R, src, c0, nc, sx);
    __syncthreads();
    const double* mr[4];
    int iq[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      iq[q] = i0 + wv * 4 + q;
      mr[q] = iq[q] < r ? R.LU + int64_t(iq[q]) * r + c0 : nullptr;
    }
    sp_rows4_acc<TRI == 0 ? 0 : 1>(mr, nc, sx, nv, acc, c0, iq);
  }
  if (RECT)
    for (int j0 = 0; j0 < R.k; j0 += kSpChunk) {
      const int nj = min(kSpChunk, R.k - j0);
      __syncthreads();
      sp_stage(A.u, A.N, R.sk + j0, nj, nv, sx);
      __syncthreads();
      const double* mr[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = i0 + wv * 4 + q;
        mr[q] = i < r ? R.Urs + int64_t(i) * R.k + j0 : nullptr;
      }
      sp_rows4_acc(mr, nj, sx, nv, acc);
    }
  {
    const double t = sp_rows_sum(acc);
    const int i = i0 + wv * 4 + (lane >> 4), v = (lane >> 1) & 7;
    if ((lane & 1) == 0 && i < r && v < nv)
      *sp_at(A, R, dst, v, i) = t + (TRI == 1 ? *sp_at(A, R, src, v, i) : 0.0);
  }
}

// Column form: out(v, i) = (M^T x)(v, i) [+ (L_sr^T u_s)(v, i)] with M^T the
// unit upper L^T (TRI 2: x_i plus the rows j > i of L) or the lower U^T
// (TRI 3: the rows j <= i of U); lane per i, 64 per workgroup, the sum over
// j split between its 16 waves.
template <int TRI, bool RECT, int NV>
__global__ __launch_bounds__(kSpColWaves * 64) void k_sp_colmv(SpArgs A, int src, int dst) {
  const SpRec R = sp_rec(A, blockIdx.y);
  const int ib = blockIdx.x * 64, r = R.r;
  if (ib >= r) return;
  SpTile<NV> acc;
  // the rows the workgroup's columns reach
  const int jb = TRI == 2 ? ib : 0, je = TRI == 2 ? r : min(r, ib + 64);
  sp_cols_acc<NV, TRI>(R.LU + int64_t(jb) * r, r, ib, r, je - jb, A.nv, acc,
                       [&](int v, int j) { return *sp_at(A, R, src, v, jb + j); }, nullptr, jb);
  if (RECT)
    sp_cols_acc<NV>(R.Lsr, r, ib, r, R.k, A.nv, acc, [&](int v, int j) { return A.u[v * A.N + R.sk[j]]; });
  sp_cols_out<NV>(acc, A.nv, [&](int v, int l, double t) {
    if (ib + l < r) *sp_at(A, R, dst, v, ib + l) = t + (TRI == 2 ? *sp_at(A, R, src, v, ib + l) : 0.0);
  });
}

// Inverses of the diagonal blocks of the records' L (unit lower) and U
// (upper) for the chained solves below: workgroup (b, i) inverts block b of
// record i, wave 0 the block of L and wave 1 that of U, read with rows and
// columns reversed, which makes it lower triangular too.  Lane c builds
// column c by substitution, 16 rows at a time in registers: a row of 16
// entries of the matrix is read from LDS as eight broadcasts for 16 products.
// Rows and columns past a partial last block are the identity.
__global__ __launch_bounds__(128) void k_sp_dinv(SpArgs A, double* dinv) {
  const SpRec R = sp_rec(A, blockIdx.y);
  const int b = blockIdx.x, j0 = b * kNbT;
  if (j0 >= R.r) return;
  const int nb = min(kNbT, R.r - j0), r = R.r, c = threadIdx.x & 63, w = threadIdx.x >> 6;
  __shared__ __align__(16) double sM[2][kNbT][kNbT + 2];  // [j][i]: column j of the lower triangle
  __shared__ double sX[2][kNbT][kNbT + 1];
  for (int a = w; a < kNbT; a += 2) {
    const double m = (a < nb && c < nb) ? R.LU[int64_t(j0 + a) * r + j0 + c] : (a == c ? 1.0 : 0.0);
    const bool low = a > c;
    if (low)
      sM[0][c][a] = m;
    else
      sM[1][kNbT - 1 - c][kNbT - 1 - a] = m;
    if (a == c) sM[0][c][c] = 1.0;
  }
  __syncthreads();
  for (int i0 = 0; i0 < kNbT; i0 += 16) {
    double v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = i0 + i == c ? 1.0 : 0.0;
#pragma unroll 2
    for (int j = 0; j < i0; ++j) {
      const double xj = sX[w][j][c];
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i] -= sM[w][j][i0 + i] * xj;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      double x = v[i];
      if (w) x = x / sM[1][i0 + i][i0 + i];
      if (i0 + i < c) x = 0.0;
      sX[w][i0 + i][c] = x;
#pragma unroll
      for (int q = i + 1; q < 16; ++q) v[q] -= sM[w][i0 + i][i0 + q] * x;
    }
  }
  __syncthreads();
  double* out = dinv + (int64_t(blockIdx.y) * A.dnb + b) * 2 * kNbT * kNbT;
  for (int a = w; a < kNbT; a += 2) {
    out[a * kNbT + c] = sX[0][a][c];
    out[kNbT * kNbT + a * kNbT + c] = sX[1][kNbT - 1 - a][kNbT - 1 - c];
  }
}

// ---------------------------------------------------------------------------
// The blocked triangular solve X = M^{-1} B of every record of a pass in one
// launch.  Workgroup (record, block j) owns rows 64j .. 64j + 63 of X: it
// subtracts the products of its row of 64 x 64 blocks of M with the blocks
// of X it depends on, each as soon as that block is written, multiplies the
// result by the stored inverse of its diagonal block and writes its block of
// X.  The block's values are their own flag: the pass's first kernel marks
// every entry of X pending (a signaling NaN, which no arithmetic produces),
// the owner stores the entries with relaxed device-scope atomic stores, and
// a reader polls them with relaxed device-scope atomic loads, both coherent
// across the chip, until none is pending: one memory round trip per block,
// with no cache write-back or invalidation.  The workgroups draw (record,
// block) from a ticket counter in the order in which the blocks become
// ready, so a workgroup only ever waits on one that has already started, and
// every wait ends however many workgroups are resident at once.  Each wait
// is also bounded in time; past the bound (not expected) the workgroup
// writes NaN in its block, so that the failure shows in the result instead
// of stalling the device.
//   A chain is bound by the time from one block of X to the next, so little
// stands on that path.  Wave 4 polls and nothing else: loads return in order,
// so a wave that also loaded tiles would wait for those on every poll (all
// waves did both before: 2.2 us per block of one right-hand side, 4.5 us of
// eight).  Waves 0 .. 3 each hold 16 columns of a tile of M in registers, the
// next two tiles in flight, and their sums meet once, after the last block.
//   MODE 0: L X = B    (unit lower L of the record's LU; blocks first to last)
//   MODE 1: U X = B    (upper U; last to first)
//   MODE 2: U^T X = B  (first to last; U read by columns)
//   MODE 3: L^T X = B  (last to first; L read by columns)
// B is the record's vector src, X its block `dst` of the work buffer (X or B,
// not the one B is read from), and with put (kInU or kInPu) the entries are
// also written there.  Grid (A.nbm, records), 320 threads; the ticket is zero
// and dst pending at launch.
// ---------------------------------------------------------------------------
constexpr long long kWaitTicks = 20000000;  // 0.2 s of the 100 MHz constant clock (default bound)

// The polling wave: block b0 .. b0 + nbb - 1 of X, every right-hand side,
// into sx (lane = row of the block), polled until no entry is pending.
// Returns false past the time bound (wait ticks of the constant clock).
template <int NV>
__device__ __forceinline__ bool sp_read_block(const double* X, int r, int b0, int nbb, int nv, double (*sx)[66],
                                              long long wait) {
  const int lane = threadIdx.x & 63;
  // every lane reads an entry that exists, and every load of a poll is issued
  // before any is looked at: one load at a time made a poll of 8 right-hand
  // sides take 8 memory round trips
  const uint64_t* X64 = reinterpret_cast<const uint64_t*>(X) + b0 + min(lane, nbb - 1);
  uint64_t got[NV];
  const long long t0 = wall_clock64();
  bool ok = true;
  for (;;) {
#pragma unroll
    for (int v = 0; v < NV; ++v)
      got[v] = __hip_atomic_load(X64 + int64_t(min(v, nv - 1)) * r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    bool ready = true;
#pragma unroll
    for (int v = 0; v < NV; ++v) ready &= got[v] != kXPending;
    if (__all(ready)) break;
    if (wall_clock64() - t0 > wait) {
      ok = false;
      break;
    }
    __builtin_amdgcn_s_sleep(1);
  }
#pragma unroll
  for (int v = 0; v < NV; ++v) sx[v][lane] = v < nv && lane < nbb ? __longlong_as_double((long long)got[v]) : 0.0;
  return ok;
}

template <int MODE, int NV>
__global__ __launch_bounds__(320) void k_sp_chain(SpArgs A, int src, int dst, int put) {
  constexpr bool kFwd = MODE == 0 || MODE == 2;
  constexpr bool kTrans = MODE >= 2;
  constexpr bool kUseU = MODE == 1 || MODE == 2;
  __shared__ unsigned s_ticket;
  __shared__ int s_ok;
  using T = SpTile<NV>;
  __shared__ double sT[4][kTrans ? 1 : kNbT][17];  // a wave's 16 columns of a tile on their way to SpTile's layout
  __shared__ double sx[2][NV][T::kLd];
  __shared__ double sacc[2][4][NV][T::kLd];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (tid == 0) {
    s_ticket = atomicAdd(A.sync, 1u);
    s_ok = 1;
  }
  __syncthreads();
  const unsigned t = s_ticket;
  const int rec = int(t / unsigned(A.nbm)), jj = int(t % unsigned(A.nbm));
  if (unsigned(rec) >= gridDim.y) return;  // sweeps of one handle that overlap on two streams draw from one counter
  const SpRec R = sp_rec(A, rec);
  const int r = R.r, nbk = (r + kNbT - 1) / kNbT;
  if (jj >= nbk) return;
  const int j = kFwd ? jj : nbk - 1 - jj;
  const int j0 = j * kNbT, nb = min(kNbT, r - j0), nv = A.nv;
  const int ndep = kFwd ? j : nbk - 1 - j;
  double* X = dst == kInX ? R.X : R.B;
  // the polling wave; the barrier of step d hands over block d (sx[d & 1] is
  // written again only after the next barrier, when all have read it)
  if (wv == 4) {
    for (int d = 0; d < ndep; ++d) {
      const int b0 = (kFwd ? d : nbk - 1 - d) * kNbT;
      if (!sp_read_block<NV>(X, r, b0, min(kNbT, r - b0), nv, sx[d & 1], A.wait_ticks) && lane == 0) s_ok = 0;
      __syncthreads();
    }
    __syncthreads();
    __syncthreads();
    return;
  }
  // The wave's columns are 16 wv .. 16 wv + 15 of a tile.  A tile of M^T is
  // read in the layout of the product (consecutive lanes, consecutive
  // addresses); a tile of M is read by rows, 16 consecutive entries of 4 rows
  // at a time, and turned through LDS by the wave that owns its columns.
  const int cw = 16 * wv, c4 = cw + (lane & 15), r4 = lane >> 4;
  auto load_tile = [&](int d, double (&p)[16]) {
    const int b0 = (kFwd ? d : nbk - 1 - d) * kNbT, nbb = min(kNbT, r - b0);
    if constexpr (kTrans) {
#pragma unroll
      for (int q = 0; q < 16; ++q)
        p[q] = R.LU[int64_t(b0 + min(cw + T::col(q), nbb - 1)) * r + j0 + min(T::row(q), nb - 1)];
    } else {
      const double* m = R.LU + int64_t(j0) * r + b0 + min(c4, nbb - 1);
#pragma unroll
      for (int q = 0; q < 16; ++q) p[q] = m[int64_t(min(4 * q + r4, nb - 1)) * r];
    }
  };
  auto turn = [&](const double (&p)[16], double (&m)[16]) {
    if constexpr (kTrans) {
#pragma unroll
      for (int q = 0; q < 16; ++q) m[q] = p[q];
    } else {
#pragma unroll
      for (int q = 0; q < 16; ++q) sT[wv][4 * q + r4][lane & 15] = p[q];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int q = 0; q < 16; ++q) m[q] = sT[wv][T::row(q)][T::col(q)];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  };
  {
    // the wave's columns of the stored inverse of the diagonal block
    // (row-major; transposed for U^T, L^T)
    const double* Dg = A.dinv + (int64_t(rec) * A.dnb + j) * 2 * kNbT * kNbT + (kUseU ? kNbT * kNbT : 0);
    double p[16], dm[16], p0[16], p1[16], b[T::kNx], x[T::kNx];
#pragma unroll
    for (int q = 0; q < 16; ++q)
      p[q] = kTrans ? Dg[(cw + T::col(q)) * kNbT + T::row(q)] : Dg[(4 * q + r4) * kNbT + c4];
    if (ndep > 0) load_tile(0, p0);
    if (ndep > 1) load_tile(1, p1);
    const int vx = T::rhs(), vl = NV == 1 ? 0 : vx & (NV - 1);
#pragma unroll
    for (int k = 0; k < T::kNx; ++k) {
      const int c = cw + T::col_x(k);
      b[k] = c < nb && vx < nv ? *sp_at(A, R, src, vx, j0 + c) : 0.0;
    }
    turn(p, dm);
    T acc, y;
    auto step = [&](int d, double (&pd)[16]) {
      double m[16];
      turn(pd, m);
      if (d + 2 < ndep) load_tile(d + 2, pd);
      __syncthreads();
#pragma unroll
      for (int k = 0; k < T::kNx; ++k) x[k] = sx[d & 1][vl][cw + T::col_x(k)];
      acc.mul(m, x);
    };
    for (int d = 0; d < ndep; d += 2) {
      step(d, p0);
      if (d + 1 < ndep) step(d + 1, p1);
    }
    // B - M X of the wave's 16 rows, then its part of X = D^{-1} (B - M X)
    acc.put(sacc[0][wv]);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < T::kNx; ++k) {
      const int c = cw + T::col_x(k);
      if (c < nb)
        b[k] -= (sacc[0][0][vl][c] + sacc[0][1][vl][c]) + (sacc[0][2][vl][c] + sacc[0][3][vl][c]);
    }
    y.mul(dm, b);
    y.put(sacc[1][wv]);
  }
  __syncthreads();
  // each thread its row (lane) of its right-hand sides, entry by entry
  // visible to the readers, and only then u
  const bool ok = s_ok != 0;
  uint64_t* X64 = reinterpret_cast<uint64_t*>(X);
  double x[(NV + 3) / 4];
#pragma unroll
  for (int e = 0; e < (NV + 3) / 4; ++e) {
    const int v = wv + 4 * e;
    if (v >= nv || lane >= nb) continue;
    x[e] = ok ? (sacc[1][0][v][lane] + sacc[1][1][v][lane]) + (sacc[1][2][v][lane] + sacc[1][3][v][lane])
              : __builtin_nan("");
    __hip_atomic_store(X64 + int64_t(v) * r + j0 + lane, (uint64_t)__double_as_longlong(x[e]), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  }
  if (put)
#pragma unroll
    for (int e = 0; e < (NV + 3) / 4; ++e) {
      const int v = wv + 4 * e;
      if (v < nv && lane < nb) *sp_at(A, R, put, v, j0 + lane) = x[e];
    }
}

}  // namespace

void launch_make_perm(const GroupRec* recs, int nrec, int32_t* iarena, int max_r, hipStream_t s) {
  (void)max_r;
  hipLaunchKernelGGL(k_make_perm, dim3(nrec), dim3(64), 0, s, recs, iarena);
  HIF_HIP(hipGetLastError());
}

void launch_make_perm_top(const int32_t* piv, int32_t* perm, int n, hipStream_t s) {
  hipLaunchKernelGGL(k_make_perm_top, dim3(1), dim3(64), 0, s, piv, perm, n);
  HIF_HIP(hipGetLastError());
}

// k_sweep_lds of one sweep (op, down).
using SweepLds = void (*)(SwArgs, int);
static SweepLds sweep_lds_kernel(int op, int down) {
  static constexpr SweepLds k[4][2] = {{k_sweep_lds<0, false>, k_sweep_lds<0, true>},
                                       {k_sweep_lds<1, false>, k_sweep_lds<1, true>},
                                       {k_sweep_lds<2, false>, k_sweep_lds<2, true>},
                                       {k_sweep_lds<3, false>, k_sweep_lds<3, true>}};
  return k[op][down];
}

// Dynamic LDS of the staged sweeps goes up to kCapL doubles (128 KiB) and a
// diagonal block.
static void allow_large_lds() {
  static std::once_flag once;
  std::call_once(once, [] {
    const int bytes = (kCapL + tri_len(kNbT)) * int(sizeof(double));
    for (int op = 0; op < 4; ++op)
      for (int down = 0; down < 2; ++down)
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(sweep_lds_kernel(op, down)),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    (void)hipGetLastError();
  });
}

// Sub-levels whose sweeps run through the multi-workgroup path for nv
// right-hand sides per pass: records too large for LDS with all of them, or
// few records (at most kSplitMaxRecords) of at least kSplitMinR redundant
// unknowns, which one workgroup each would leave most of the chip idle.
#ifndef HIF_SPLIT_MAX_RECORDS
#define HIF_SPLIT_MAX_RECORDS 64
#endif
#ifndef HIF_SPLIT_MIN_R
#define HIF_SPLIT_MIN_R 128
#endif
constexpr int kSplitMaxRecords = HIF_SPLIT_MAX_RECORDS;
constexpr int kSplitMinR = HIF_SPLIT_MIN_R;
static bool split_solve(const SubLevel& sub, int64_t N, int nv) {
  return 2 * sub.sum_r <= N &&
         (int64_t(sub.max_2rk) * nv > kCapL || (sub.nrec <= kSplitMaxRecords && sub.max_r >= kSplitMinR));
}

// A top block of some size is solved like a large record with no skeleton
// through the many-workgroup triangular solves, if its solve record was built.
static bool top_split_solve(const hif_factor_s* H) { return H->top_dinv.p != nullptr; }

// Scratch of a sweep over nrhs right-hand sides, in doubles: what it needs, and
// what it takes where there is that much (two vectors of a top block of more
// than half of the unknowns).
static int64_t sweep_work_min(const hif_factor_s* H, int64_t nrhs) { return std::min<int64_t>(nrhs, kMaxV) * H->n; }
static int64_t sweep_work(const hif_factor_s* H, int64_t nrhs) {
  return std::min<int64_t>(nrhs, kMaxV) * std::max<int64_t>(H->n, top_split_solve(H) ? 2 * H->ntop : 0);
}

// Right-hand sides per pass that the kernels are built for, f(integral
// constant): one, or up to kMaxV.
template <typename F>
static void for_nv(int nv, F f) {
  if (nv == 1)
    f(std::integral_constant<int, 1>{});
  else
    f(std::integral_constant<int, kMaxV>{});
}

// The blocked triangular solve X = M^{-1} B of every record of a pass, one
// launch (k_sp_chain); mode, src, dst and put as there.
static void chain(const SpArgs& P, int mode, unsigned nr, hipStream_t s, int src, int dst, int put) {
  const dim3 g(unsigned(P.nbm), nr);
  for_nv(P.nv, [&](auto nvc) {
    constexpr int NV = decltype(nvc)::value;
    if (mode == 0)
      hipLaunchKernelGGL((k_sp_chain<0, NV>), g, dim3(320), 0, s, P, src, dst, put);
    else if (mode == 1)
      hipLaunchKernelGGL((k_sp_chain<1, NV>), g, dim3(320), 0, s, P, src, dst, put);
    else if (mode == 2)
      hipLaunchKernelGGL((k_sp_chain<2, NV>), g, dim3(320), 0, s, P, src, dst, put);
    else
      hipLaunchKernelGGL((k_sp_chain<3, NV>), g, dim3(320), 0, s, P, src, dst, put);
  });
}

template <bool LSR, bool PERM, bool ADD = false>
static void first_cols(const SpArgs& P, dim3 g, hipStream_t s) {
  for_nv(P.nv, [&](auto nvc) {
    hipLaunchKernelGGL((k_sp_first_cols<LSR, PERM, ADD, decltype(nvc)::value>), g, dim3(kSpColWaves * 64), 0, s, P);
  });
}

template <bool GATHER>
static void skel_update_T(const SpArgs& P, dim3 g, hipStream_t s, double sgn) {
  for_nv(P.nv, [&](auto nvc) {
    hipLaunchKernelGGL((k_sp_skel_update_T<GATHER, decltype(nvc)::value>), g, dim3(kSpColWaves * 64), 0, s, P, sgn);
  });
}

template <int TRI, bool RECT>
static void colmv(const SpArgs& P, dim3 g, hipStream_t s, int src, int dst) {
  for_nv(P.nv, [&](auto nvc) {
    hipLaunchKernelGGL((k_sp_colmv<TRI, RECT, decltype(nvc)::value>), g, dim3(kSpColWaves * 64), 0, s, P, src, dst);
  });
}

// The sweeps proper.  work: wcap >= sweep_work_min doubles of scratch, reused
// by every group of 8 right-hand sides (all launches are ordered on s).
static void sweep_run(hif_factor_s* H, int op, const double* x, double* y, int64_t nrhs, hipStream_t s,
                      double* work, int64_t wcap) {
  const int64_t N = H->n;
  const int64_t tot = N * nrhs;
  if (x != y) {
    int64_t blocks = (tot + 255) / 256;
    if (blocks > (1 << 20)) blocks = 1 << 20;
    hipLaunchKernelGGL(k_copy, dim3(unsigned(blocks)), dim3(256), 0, s, x, y, tot);
    HIF_HIP(hipGetLastError());
  }
  const long long wait_ticks = H->opts.sweep_wait_us > 0 ? 100ll * H->opts.sweep_wait_us : kWaitTicks;
  for (int64_t v0 = 0; v0 < nrhs; v0 += 8) {
    const int nv = int(std::min<int64_t>(8, nrhs - v0));
    double* u = y + v0 * N;
    double* wk = work;
    // solve / solve_T of a sub-level go through LDS when a group fits; the
    // four sweeps of few large records are spread over many workgroups per
    // record:
    //   solve   up:   B = P(u_r - T^T u_s); X = L^{-1} B;   u_s -= L_sr X; u_r = X
    //           down: B = u_r - U_rs u_s;   X = U^{-1} B;   u_s -= T X;    u_r = X
    //   solve_T up:   B = u_r - T^T u_s;    X = U^{-T} B;   u_s -= U_rs^T X; u_r = X
    //           down: B = u_r - L_sr^T u_s; X = L^{-T} B;   u_r = P^T X;   u_s -= T u_r
    //   apply   up:   B = u_r; u_s += T u_r;      X = U B + U_rs u_s;       u_r = X
    //           down: B = u_r; u_s += L_sr u_r;   X = L B; u_r = P^T X;     u_r += T^T u_s
    //   apply_T up:   B = P u_r; u_s += T u_r;    X = L^T B + L_sr^T u_s;   u_r = X
    //           down: B = u_r; u_s += U_rs^T u_r; X = U^T B; u_r = X;       u_r += T^T u_s
    auto sweep = [&](const SubLevel& sub, int down) {
      SwArgs A{sub.rec.p, sub.iarena.p, sub.darena.p, u, wk, N, nv, op};
      if (split_solve(sub, N, nv)) {
        HIF_REQUIRE(sub.dinv.p && H->sync.p, HIF_EDEVICE,
                    "the diagonal-block inverses of a sub-level were not built");
        SpArgs P{sub.rec.p,  sub.iarena.p, sub.darena.p, sub.woff.p, u, wk, wk + nv * sub.sum_r, N, nv,
                 sub.dinv.p, sub.dinv_nb};
        P.sync = H->sync.p;
        P.wait_ticks = wait_ticks;
        P.nbm = (sub.max_r + kNbT - 1) / kNbT;
        const unsigned nr = unsigned(sub.nrec);
        const dim3 gr(unsigned((sub.max_r + 255) / 256), nr), gu(unsigned((sub.max_r + 63) / 64), nr);
        const dim3 gw(unsigned((sub.max_r + 15) / 16), nr);
        const dim3 gs(unsigned((sub.max_k + 15) / 16), nr), gt(unsigned((sub.max_k + 63) / 64), nr);
        const bool sk = sub.max_k > 0;
        if (op == 0 && !down) {
          first_cols<false, true>(P, gu, s);
          chain(P, 0, nr, s, kInB, kInX, kInU);
          if (sk) hipLaunchKernelGGL(k_sp_skel_update<false>, gs, dim3(256), 0, s, P, 0, -1.0);
        } else if (op == 0) {
          hipLaunchKernelGGL(k_sp_down_first, gw, dim3(256), 0, s, P);
          chain(P, 1, nr, s, kInB, kInX, kInU);
          if (sk) hipLaunchKernelGGL(k_sp_skel_update<false>, gs, dim3(256), 0, s, P, 1, -1.0);
        } else if (op == 1 && !down) {
          first_cols<false, false>(P, gu, s);
          chain(P, 2, nr, s, kInB, kInX, kInU);
          if (sk) skel_update_T<false>(P, gt, s, -1.0);
        } else if (op == 1) {
          first_cols<true, false>(P, gu, s);
          chain(P, 3, nr, s, kInB, kInX, kInPu);
          if (sk) hipLaunchKernelGGL(k_sp_skel_update<true>, gs, dim3(256), 0, s, P, 1, -1.0);
        } else if (op == 2 && !down) {
          hipLaunchKernelGGL(k_sp_gather<false>, gr, dim3(256), 0, s, P);
          if (sk) hipLaunchKernelGGL(k_sp_skel_update<true>, gs, dim3(256), 0, s, P, 1, 1.0);
          hipLaunchKernelGGL((k_sp_rowmv<0, true>), gw, dim3(256), 0, s, P, kInB, kInU);
        } else if (op == 2) {
          hipLaunchKernelGGL(k_sp_gather<false>, gr, dim3(256), 0, s, P);
          if (sk) hipLaunchKernelGGL(k_sp_skel_update<true>, gs, dim3(256), 0, s, P, 0, 1.0);
          hipLaunchKernelGGL((k_sp_rowmv<1, false>), gw, dim3(256), 0, s, P, kInB, kInPu);
          if (sk) first_cols<false, false, true>(P, gu, s);
        } else if (!down) {
          hipLaunchKernelGGL(k_sp_gather<true>, gr, dim3(256), 0, s, P);
          if (sk) hipLaunchKernelGGL(k_sp_skel_update<true>, gs, dim3(256), 0, s, P, 1, 1.0);
          colmv<2, true>(P, gu, s, kInB, kInU);
        } else {
          hipLaunchKernelGGL(k_sp_gather<false>, gr, dim3(256), 0, s, P);
          if (sk) skel_update_T<true>(P, gt, s, 1.0);
          colmv<3, false>(P, gu, s, kInB, kInU);
          if (sk) first_cols<false, false, true>(P, gu, s);
        }
        return;
      }
      if (sub.max_2rk <= kCapL) {
        allow_large_lds();
        // LDS for as many right-hand sides per pass as fit (all of them when
        // the records are small); 1024 threads per record when the records
        // are too few to give every CU several workgroups
        const int nvb = std::max(1, std::min(nv, kCapL / sub.max_2rk));
        const int cap = nvb * sub.max_2rk;
        const size_t lds = size_t(cap + (op < 2 ? tri_len(std::min(kNbT, sub.max_r)) : 0)) * sizeof(double);
        const int many = sub.nrec < kManyRecords ? 1024 : tuning().sweep_many_threads;
        const int bs = many == 64 || many == 128 || many == 1024 ? many : 256;
        hipLaunchKernelGGL(sweep_lds_kernel(op, down), dim3(sub.nrec), dim3(bs), lds, s, A, cap);
      } else if (down)
        hipLaunchKernelGGL(k_down, dim3(sub.nrec), dim3(kBlock), 0, s, A);
      else
        hipLaunchKernelGGL(k_up, dim3(sub.nrec), dim3(kBlock), 0, s, A);
    };
    for (auto& sub : H->subs)
      if (sub.nrec > 0) sweep(sub, 0);
    // A top block of some size is swept like a large record with no
    // skeleton (k = 0), through the same chained triangular solves and
    // products: solve X = U^{-1} L^{-1} P u, solve_T X = P^T L^{-T} U^{-T} u,
    // apply X = P^T L U u, apply_T X = U^T L^T P u.
    if (top_split_solve(H) && 2 * int64_t(nv) * H->ntop <= wcap) {
      const int r = int(H->ntop);
      const int nbk = (r + kNbT - 1) / kNbT;
      SpArgs P{H->top_rec.p, H->top_iarena.p, H->top_lu.p,  H->top_woff.p, u, wk, wk + int64_t(nv) * r, N, nv,
               H->top_dinv.p, nbk};
      P.sync = H->sync.p;
      P.wait_ticks = wait_ticks;
      P.nbm = nbk;
      const dim3 gu(unsigned(nbk), 1), gw(unsigned((r + 15) / 16), 1);
      SpArgs P2 = P;
      P2.sync = P.sync + 1;
      if (op == 0) {
        hipLaunchKernelGGL(k_sp_ready, gu, dim3(256), 0, s, P);
        chain(P, 0, 1, s, kInPu, kInX, 0);
        chain(P2, 1, 1, s, kInX, kInB, kInU);
      } else if (op == 1) {
        hipLaunchKernelGGL(k_sp_ready, gu, dim3(256), 0, s, P);
        chain(P, 2, 1, s, kInU, kInX, 0);
        chain(P2, 3, 1, s, kInX, kInB, kInPu);
      } else if (op == 2) {
        hipLaunchKernelGGL((k_sp_rowmv<0, false>), gw, dim3(256), 0, s, P, kInU, kInX);
        hipLaunchKernelGGL((k_sp_rowmv<1, false>), gw, dim3(256), 0, s, P, kInX, kInPu);
      } else {
        colmv<2, false>(P, gu, s, kInPu, kInX);
        colmv<3, false>(P, gu, s, kInX, kInU);
      }
    } else if (H->ntop >= kTopSplitMin) {
      hipLaunchKernelGGL(k_top, dim3(1), dim3(1024), 0, s, H->top_lu.p, H->top_piv.p, int(H->ntop), H->top_idx.p, u, wk,
                         N, nv, op);
    } else if (H->ntop > 0) {
      hipLaunchKernelGGL(k_top_lds, dim3(1), dim3(1024), 0, s, H->top_lu.p, H->top_perm.p, int(H->ntop),
                         H->top_idx.p, u, N, nv, op);
    }
    for (auto it = H->subs.rbegin(); it != H->subs.rend(); ++it)
      if (it->nrec > 0) sweep(*it, 1);
    HIF_HIP(hipGetLastError());
  }
}



// Diagonal-block inverses of the sub-levels (and the top block) whose solve
// can take the multi-workgroup path, for any number of right-hand sides per
// pass (at most kMaxV).
static void build_dinv(hif_factor_s* H, hipStream_t s) {
  for (SubLevel& sub : H->subs) {
    if (sub.nrec == 0 || sub.dinv.p || !split_solve(sub, H->n, kMaxV)) continue;
    sub.dinv_nb = (sub.max_r + kNbT - 1) / kNbT;
    sub.dinv.alloc(size_t(sub.nrec) * sub.dinv_nb * 2 * kNbT * kNbT, &H->mem);
    SpArgs P{sub.rec.p, sub.iarena.p, sub.darena.p, sub.woff.p, nullptr, nullptr, nullptr, H->n, 1,
             nullptr, sub.dinv_nb};
    hipLaunchKernelGGL(k_sp_dinv, dim3(unsigned(sub.dinv_nb), unsigned(sub.nrec)), dim3(128), 0, s, P, sub.dinv.p);
  }
  HIF_HIP(hipGetLastError());
}

void prepare_sweeps(hif_factor_s* H, hipStream_t s) {
  build_dinv(H, s);
  // the top block's solve record, where the memory cap has room for it
  const int r = int(H->ntop), nbk = (r + kNbT - 1) / kNbT;
  if (H->ntop >= kTopSplitMin && !H->top_dinv.p) {
    try {
      H->top_iarena.alloc(size_t(3) * r, &H->mem);
      H->top_rec.alloc(1, &H->mem);
      H->top_woff.alloc(1, &H->mem);
      H->sync.alloc(2, &H->mem);
      H->top_dinv.alloc(size_t(nbk) * 2 * kNbT * kNbT, &H->mem);
    } catch (const Error& e) {
      if (e.status != HIF_ENOMEM) throw;
      H->top_iarena.release();
      H->top_rec.release();
      H->top_woff.release();
      H->sync.release();
    }
  }
  if (top_split_solve(H)) {
    hipLaunchKernelGGL(k_top_record, dim3(unsigned((r + 255) / 256)), dim3(256), 0, s, H->top_idx.p, H->top_piv.p,
                       H->top_perm.p, r, H->top_iarena.p, H->top_rec.p, H->top_woff.p);
    SpArgs P{H->top_rec.p, H->top_iarena.p, H->top_lu.p, H->top_woff.p, nullptr, nullptr, nullptr, H->n, 1,
             nullptr, nbk};
    hipLaunchKernelGGL(k_sp_dinv, dim3(unsigned(nbk), 1), dim3(128), 0, s, P, H->top_dinv.p);
    HIF_HIP(hipGetLastError());
  }
  // the ticket counters of the chained triangular solves
  bool chained = false;
  for (const SubLevel& sub : H->subs) chained = chained || sub.dinv.p != nullptr;
  if (chained && !H->sync.p) H->sync.alloc(2, &H->mem);
}

// The handle's scratch for nrhs right-hand sides (need: its doubles).  A block
// that a recorded solve writes to on every replay is left to it, not released
// to the next allocation.
static double* sweep_scratch(hif_factor_s* H, int64_t nrhs, int64_t& need) {
  auto get = [&](int64_t cnt) {
    if (H->work.use_count() > 1 && int64_t(H->work->n) < cnt) {
      auto w = std::make_shared<DBuf<double>>();
      w->ensure(cnt, &H->mem);
      H->work = std::move(w);
    }
    H->work->ensure(cnt, &H->mem);
    need = cnt;
    return H->work->p;
  };
  const int64_t most = sweep_work(H, nrhs), least = sweep_work_min(H, nrhs);
  if (most > least) {
    try {
      return get(most);
    } catch (const Error& e) {
      if (e.status != HIF_ENOMEM) throw;
    }
  }
  return get(least);
}

void sweep_impl(hif_factor_s* H, int op, const double* x, double* y, int64_t nrhs, hipStream_t s) {
  int64_t need = 0;
  double* work = sweep_scratch(H, nrhs, need);
  sweep_run(H, op, x, y, nrhs, s, work, need);
}

// The launches of one solve u = F^{-1} f recorded into a HIP graph by stream
// capture on a private stream (kernel nodes only), then instantiated.  The
// sweep scratch is allocated before the capture starts.
void graph_solve_impl(hif_factor_s* H, const double* f, double* u, int64_t nrhs, hipStream_t cs,
                      hipGraph_t* graph, hipGraphExec_t* exec) {
  // a block that is outgrown here is released on cs: sweeps queued on other
  // streams have to be done with it
  if (int64_t(H->work->n) < sweep_work(H, nrhs)) wait_uses(H);
  int64_t need = 0;
  double* work = sweep_scratch(H, nrhs, need);
  allow_large_lds();
  HIF_HIP(hipStreamSynchronize(cs));
  HIF_HIP(hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal));
  try {
    sweep_run(H, 0, f, u, nrhs, cs, work, need);
  } catch (...) {
    hipGraph_t g = nullptr;
    (void)hipStreamEndCapture(cs, &g);
    if (g) (void)hipGraphDestroy(g);
    throw;
  }
  HIF_HIP(hipStreamEndCapture(cs, graph));
  const hipError_t e = hipGraphInstantiate(exec, *graph, nullptr, nullptr, 0);
  if (e != hipSuccess) {
    (void)hipGraphDestroy(*graph);
    *graph = nullptr;
    throw Error{HIF_EDEVICE, std::string("hipGraphInstantiate: ") + hipGetErrorString(e)};
  }
}

// ---------------------------------------------------------------------------
// Solve without allocation (hif_solve_noalloc): the sweep scratch is this
// file-scope device array instead of the handle's work buffer.  Each device
// holds its own copy; host code reaches it only through the address that
// hipGetSymbolAddress returns for the current device (the array's name is a
// host-side stand-in).  Calls that overlap on one device share it and race.
// ---------------------------------------------------------------------------
namespace {
__device__ __align__(256) double scratch[kSolveScratchDoubles];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {};

double* scratch_ptr() {
  int dev = 0;
  HIF_HIP(hipGetDevice(&dev));
  HIF_REQUIRE(dev >= 0 && dev < kMaxDevices, HIF_EDEVICE, "device ordinal beyond the scratch table");
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      throw Error{HIF_EDEVICE, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e)};
    g_scratch_ptr[dev] = static_cast<double*>(p);
  }
  return g_scratch_ptr[dev];
}
}  // namespace

void sweep_noalloc_impl(hif_factor_s* H, const double* f, double* u, int64_t nrhs, hipStream_t s) {
  const int64_t need = std::min<int64_t>(nrhs, 8) * H->n;
  HIF_REQUIRE(need <= int64_t(kSolveScratchDoubles), HIF_EINVAL,
              "min(nrhs, 8) * n = " + std::to_string(need) + " exceeds the " +
                  std::to_string(kSolveScratchDoubles) + " doubles of the solve scratch");
  double* work = scratch_ptr();
  sweep_run(H, 0, f, u, nrhs, s, work, int64_t(kSolveScratchDoubles));
}

}  // namespace hif
