// Per-panel batched kernels for the coarse sub-levels, where a few large
// problems would leave most compute units idle if each ran in one workgroup:
// the row compression before the ID (blocked Householder QR) and the partial
// LU of the elimination (and of the top block) are split into a panel kernel
// (one workgroup per problem) and a trailing-update kernel (one workgroup per
// 64-column tile per problem) launched once per panel of 16 columns.  The
// updates run on the matrix cores (v_mfma_f64_16x16x4f64) with operands read
// straight from device memory in the instruction's lane layout.
#include <algorithm>
#include <climits>
#include <vector>

#include "batched.h"
#include "gemm.h"
#include "wave.h"

namespace hif {

namespace {

constexpr int kNb = 16;     // panel width
constexpr int kTileN = 64;  // columns per update workgroup

struct AM {
  double v;
  int i;
};
__device__ __forceinline__ AM am_better(AM a, AM b) {
  if (b.v > a.v || (b.v == a.v && b.i < a.i)) return b;
  return a;
}
__device__ __forceinline__ double pick16(const double (&y)[kNb], int j) {
  double r = 0.0;
#pragma unroll
  for (int c = 0; c < kNb; ++c)
    if (c == j) r = y[c];
  return r;
}

// Block-wide argmax (larger value, ties to the lower index) for up to 1024 threads.
// The caller must pass a barrier between two calls (the slots are
// rewritten by the next call).
__device__ AM block_argmax_n(AM x) {
  __shared__ double sv[16];
  __shared__ int si[16];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    AM y{__shfl_xor(x.v, o, 64), __shfl_xor(x.i, o, 64)};
    x = am_better(x, y);
  }
  if (lane == 0) { sv[wv] = x.v; si[wv] = x.i; }
  __syncthreads();
  AM r{-1.0, INT_MAX};
  for (int k = 0; k < nw; ++k) r = am_better(r, AM{sv[k], si[k]});
  return r;
}

__device__ AM block_argmax256(AM x) {
  __shared__ double sv[4];
  __shared__ int si[4];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    AM y{__shfl_xor(x.v, o, 64), __shfl_xor(x.i, o, 64)};
    x = am_better(x, y);
  }
  if (lane == 0) { sv[wv] = x.v; si[wv] = x.i; }
  __syncthreads();
  AM r{-1.0, INT_MAX};
  for (int k = 0; k < 4; ++k) r = am_better(r, AM{sv[k], si[k]});
  __syncthreads();
  return r;
}

constexpr int kQrThreads = 1024;            // trailing-update workgroup
constexpr int kQrWaves = kQrThreads / 64;
constexpr int kQpThreads = 512;             // panel workgroup (register budget of 256 VGPRs)
constexpr int kQpWaves = kQpThreads / 64;

__device__ __forceinline__ double bsumQ(double v, double* red) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  v = wave_sum(v);
  if (lane == 0) red[wv] = v;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int w = 0; w < kQpWaves; ++w) t += red[w];
  __syncthreads();
  return t;
}

// ---------------------------------------------------------------------------
// Row compression, panel j0 of every problem: Householder vectors of columns
// j0..j0+jb-1 (rows j0..m-1) into V (m x 16, zero above the diagonal), R's
// diagonal into the block, and T of the compact WY form I - V T V^T into Tq.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kQpThreads) void k_qr_panel(QrBatch A, int j0) {
  const int q = blockIdx.x;
  const int m = A.rows[q], n = A.cols[q];
  if (m <= n || j0 >= n) return;
  double* M = A.base + A.moff[q];
  const int ld = A.ld[q];
  double* V = A.scratch + A.soff[q];
  double* Tq = V + int64_t(m) * kNb;
  const int jb = min(kNb, n - j0);
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  __shared__ double red[kQpWaves];
  __shared__ double sred[kQpWaves][kNb + 1];
  __shared__ double sbeta[kNb];
  __shared__ double sG[kQpWaves][kNb * kNb];
  for (int r = j0 + tid; r < m; r += kQpThreads)
#pragma unroll
    for (int c = 0; c < kNb; ++c) V[int64_t(r - j0) * kNb + c] = 0.0;
  double s0 = 0.0;
  for (int r = j0 + tid; r < m; r += kQpThreads) {
    const double y = M[int64_t(r) * ld + j0];
    s0 += y * y;
  }
  double ss = bsumQ(s0, red);
  for (int jj = 0; jj < jb; ++jj) {
    const int j = j0 + jj;
    const int nc = jb - jj - 1;
    const double x0 = M[int64_t(j) * ld + j];
    const double nrm = sqrt(ss);
    const double alpha = nrm > 0.0 ? -copysign(nrm, x0) : 0.0;
    const double v0 = x0 - alpha;
    const double vtv = ss - x0 * x0 + v0 * v0;
    const double beta = vtv > 0.0 ? 2.0 / vtv : 0.0;
    double part[kNb];
#pragma unroll
    for (int c = 0; c < kNb; ++c) part[c] = 0.0;
    for (int r0 = j + tid; r0 < m; r0 += 4 * kQpThreads) {
      double vr[4], y[4][kNb];
#pragma unroll
      for (int qq = 0; qq < 4; ++qq) {
        const int r = r0 + qq * kQpThreads;
        vr[qq] = 0.0;
        if (r < m) vr[qq] = r == j ? v0 : M[int64_t(r) * ld + j];
#pragma unroll
        for (int c = 0; c < kNb; ++c) y[qq][c] = (r < m && c < nc) ? M[int64_t(r) * ld + j + 1 + c] : 0.0;
      }
#pragma unroll
      for (int qq = 0; qq < 4; ++qq) {
        const int r = r0 + qq * kQpThreads;
        if (r < m) V[int64_t(r - j0) * kNb + jj] = vr[qq];
#pragma unroll
        for (int c = 0; c < kNb; ++c) part[c] += vr[qq] * y[qq][c];
      }
    }
#pragma unroll
    for (int c = 0; c < kNb; ++c) {
      if (c >= nc) break;
      const double t = wave_sum(part[c]);
      if (lane == 0) sred[wv][c] = t;
    }
    __syncthreads();
    double wc[kNb];
#pragma unroll
    for (int c = 0; c < kNb; ++c) {
      double t = 0.0;
#pragma unroll
      for (int w = 0; w < kQpWaves; ++w) t += sred[w][c];
      wc[c] = c < nc ? beta * t : 0.0;
    }
    __syncthreads();
    double snext = 0.0;
    for (int r0 = j + tid; r0 < m; r0 += 4 * kQpThreads) {
      double vr[4], y[4][kNb];
#pragma unroll
      for (int qq = 0; qq < 4; ++qq) {
        const int r = r0 + qq * kQpThreads;
        vr[qq] = 0.0;
        if (r < m) vr[qq] = r == j ? v0 : M[int64_t(r) * ld + j];
#pragma unroll
        for (int c = 0; c < kNb; ++c) y[qq][c] = (r < m && c < nc) ? M[int64_t(r) * ld + j + 1 + c] : 0.0;
      }
#pragma unroll
      for (int qq = 0; qq < 4; ++qq) {
        const int r = r0 + qq * kQpThreads;
#pragma unroll
        for (int c = 0; c < kNb; ++c) y[qq][c] -= wc[c] * vr[qq];
        if (r > j && r < m && nc > 0) snext += y[qq][0] * y[qq][0];
        if (r < m) {
#pragma unroll
          for (int c = 0; c < kNb; ++c)
            if (c < nc) M[int64_t(r) * ld + j + 1 + c] = y[qq][c];
        }
      }
    }
    if (tid == 0) sbeta[jj] = beta;
    ss = bsumQ(snext, red);
    if (tid == 0) M[int64_t(j) * ld + j] = alpha;
  }
  // G = V^T V on the matrix cores: every wave sums its own 4-row slices.
  {
    double4_t acc = {0.0, 0.0, 0.0, 0.0};
    const int mp = m - j0;
    const int li = lane & 15, lk = lane >> 4;
    for (int kb = wv * 4; kb < mp; kb += 4 * kQpWaves) {
      const int r = kb + lk;
      const double a = r < mp ? V[int64_t(r) * kNb + li] : 0.0;
      acc = mfma_f64(a, a, acc);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) sG[wv][(4 * v + lk) * kNb + li] = acc[v];
  }
  __syncthreads();
  __shared__ double T[kNb][kNb];
  for (int e = tid; e < kNb * kNb; e += kQpThreads) T[e / kNb][e % kNb] = 0.0;
  __syncthreads();
  if (tid == 0) {
    for (int i = 0; i < jb; ++i) {
      T[i][i] = sbeta[i];
      for (int p = 0; p < i; ++p) {
        double t = 0.0;
        for (int l = p; l < i; ++l) {
          const int e = l * kNb + i;
          double gsum = 0.0;
          for (int w = 0; w < kQpWaves; ++w) gsum += sG[w][e];
          t += T[p][l] * gsum;
        }
        T[p][i] = -sbeta[i] * t;
      }
    }
  }
  __syncthreads();
  for (int e = tid; e < kNb * kNb; e += kQpThreads) Tq[e] = T[e / kNb][e % kNb];
}

// Trailing update of one 64-column tile: W = T^T V^T Y_t (split over the
// waves along the rows), then Y_t -= V W.
__global__ __launch_bounds__(kQrThreads) void k_qr_update(QrBatch A, int j0) {
  const int q = blockIdx.y;
  const int m = A.rows[q], n = A.cols[q];
  if (m <= n || j0 >= n) return;
  const int jb = min(kNb, n - j0);
  const int c0 = j0 + jb + blockIdx.x * kTileN;
  if (c0 >= n) return;
  const int nt = min(kTileN, n - c0);
  double* M = A.base + A.moff[q];
  const int ld = A.ld[q];
  const double* V = A.scratch + A.soff[q];
  const double* Tq = V + int64_t(m) * kNb;
  const int mp = m - j0;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  __shared__ double sW[kQrWaves][kNb][kTileN + 1];
  __shared__ double sW2[kNb][kTileN + 1];
  // 1. partial W per wave over rows kb = 4*wv, 4*wv + 16, ...
  double4_t acc[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) acc[t] = double4_t{0.0, 0.0, 0.0, 0.0};
  for (int kb = wv * 4; kb < mp; kb += 4 * kQrWaves) {
    const int r = kb + lk;
    const bool ok = r < mp;
    const double a = ok ? V[int64_t(r) * kNb + li] : 0.0;
    const double* yr = M + int64_t(j0 + (ok ? r : 0)) * ld + c0;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int col = t * 16 + li;
      const double b = (ok && col < nt) ? yr[col] : 0.0;
      acc[t] = mfma_f64(a, b, acc[t]);
    }
  }
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) sW[wv][4 * v + lk][t * 16 + li] = acc[t][v];
  __syncthreads();
  // 2. W = T^T (sum of the partials), T upper triangular.
  for (int e = tid; e < kNb * kTileN; e += kQrThreads) {
    const int i = e / kTileN, c = e % kTileN;
    double s = 0.0;
    for (int p = 0; p <= i; ++p) {
      double w = 0.0;
#pragma unroll
      for (int q2 = 0; q2 < kQrWaves; ++q2) w += sW[q2][p][c];
      s += Tq[p * kNb + i] * w;
    }
    sW2[i][c] = s;
  }
  __syncthreads();
  // 3. Y_t -= V W, 16-row tiles spread over the waves.
  for (int rt = wv * 16; rt < mp; rt += 16 * kQrWaves) {
    double4_t d[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) d[t] = double4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int ks = 0; ks < kNb; ks += 4) {
      const int r = rt + li;
      const double a = r < mp ? V[int64_t(r) * kNb + ks + lk] : 0.0;
#pragma unroll
      for (int t = 0; t < 4; ++t) d[t] = mfma_f64(a, sW2[ks + lk][t * 16 + li], d[t]);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = rt + 4 * v + lk, col = t * 16 + li;
        if (r < mp && col < nt) M[int64_t(j0 + r) * ld + c0 + col] -= d[t][v];
      }
  }
}

__global__ void k_qr_clear_lower(QrBatch A) {
  const int q = blockIdx.y;
  const int m = A.rows[q], n = A.cols[q];
  if (m <= n) return;
  double* M = A.base + A.moff[q];
  const int ld = A.ld[q];
  for (int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; e < int64_t(n) * n;
       e += int64_t(gridDim.x) * blockDim.x) {
    const int r = int(e / n), c = int(e % n);
    if (c < r) M[int64_t(r) * ld + c] = 0.0;
  }
}

// ---------------------------------------------------------------------------
// Partial LU (Lemma 2.1) of the n x n problems over their first r columns,
// pivoting among rows < r: panel j0 = columns j0..j0+jb-1 with row swaps over
// whole rows, then U12 = L11^{-1} A12 for the panel rows.
// ---------------------------------------------------------------------------
// Register-resident panel for panels of at most kLpRows rows (rows j0..n-1):
// thread t holds rows j0 + t and j0 + t + kLpThreads of the kNb panel
// columns for all kNb elimination steps; the pivot row is exchanged and
// broadcast through LDS.  The row interchanges are then applied in order to
// the columns outside the panel (one thread per column) and U12 is formed.
constexpr int kLpRows = 2048;  // rows of the largest register panel (1024 threads)

template <int kLpThreads>
__global__ __launch_bounds__(kLpThreads) void k_lu_panel_reg(LuBatch A, int j0) {
  const int q = blockIdx.x;
  const int n = A.n[q], r = A.r[q];
  if (j0 >= r) return;
  double* M = A.base + A.moff[q];
  int32_t* piv = A.piv + A.poff[q];
  const int jb = min(kNb, r - j0);
  const int tid = threadIdx.x;
  __shared__ double sA[kNb], sB[kNb];
  __shared__ int spiv[kNb];
  double y[2][kNb];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int R = j0 + tid + u * kLpThreads;
    const double* src = M + int64_t(R < n ? R : j0) * n + j0;
#pragma unroll
    for (int c = 0; c < kNb; ++c) y[u][c] = (R < n && c < jb) ? src[c] : 0.0;
  }
  for (int jj = 0; jj < jb; ++jj) {
    const int j = j0 + jj;
    AM loc{-1.0, INT_MAX};
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int R = j0 + tid + u * kLpThreads;
      if (R >= j && R < r) loc = am_better(loc, AM{fabs(pick16(y[u], jj)), R});
    }
    const AM best = block_argmax_n(loc);
    if (!(best.v > 0.0)) {
      if (tid == 0) atomicOr(A.status, 1);
      return;
    }
    const int p = best.i;
    // rows j (slot 0 of thread jj) and p trade places; everyone reads the new row j
    const int tp = (p - j0) % kLpThreads, up = (p - j0) / kLpThreads;
    if (tid == jj) {
#pragma unroll
      for (int c = 0; c < kNb; ++c) sA[c] = y[0][c];
    }
    if (tid == tp) {
#pragma unroll
      for (int c = 0; c < kNb; ++c) sB[c] = up == 0 ? y[0][c] : y[1][c];
    }
    if (tid == 0) spiv[jj] = p;
    __syncthreads();
    const double* prow = sB;  // the new row j, read from LDS
    if (p != j) {
      if (tid == jj) {
#pragma unroll
        for (int c = 0; c < kNb; ++c) y[0][c] = prow[c];
      }
      if (tid == tp) {
#pragma unroll
        for (int c = 0; c < kNb; ++c) {
          if (up == 0) y[0][c] = sA[c]; else y[1][c] = sA[c];
        }
      }
    }
    const double inv = 1.0 / prow[jj];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int R = j0 + tid + u * kLpThreads;
      if (R > j && R < n) {
        const double l = pick16(y[u], jj) * inv;
#pragma unroll
        for (int c = 0; c < kNb; ++c) {
          if (c == jj) y[u][c] = l;
          else if (c > jj) y[u][c] -= l * prow[c];
        }
      }
    }
    // Two barriers per step: the argmax slots are read before this step's
    // exchange barrier, which every thread passes before the next step
    // writes them; sA / sB are read after that barrier and before the next
    // step's argmax barrier, which precedes their next writes.
  }
  __syncthreads();  // sA / sB of the last step, before the code below
  // panel back to memory
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int R = j0 + tid + u * kLpThreads;
    if (R < n) {
      double* dst = M + int64_t(R) * n + j0;
#pragma unroll
      for (int c = 0; c < kNb; ++c)
        if (c < jb) dst[c] = y[u][c];
    }
  }
  if (tid < jb) piv[j0 + tid] = spiv[tid];
  // interchanges on the columns outside the panel, in order
  for (int col = tid; col < n; col += kLpThreads) {
    if (col >= j0 && col < j0 + jb) continue;
    for (int jj = 0; jj < jb; ++jj) {
      const int pj = spiv[jj];
      if (pj != j0 + jj) {
        const double t = M[int64_t(j0 + jj) * n + col];
        M[int64_t(j0 + jj) * n + col] = M[int64_t(pj) * n + col];
        M[int64_t(pj) * n + col] = t;
      }
    }
  }
  __syncthreads();  // the panel rows and the interchanges are in memory
  // the unit lower L11 of the panel, read once into LDS for every column
  __shared__ double sL11[kNb][kNb];
  for (int e = tid; e < kNb * kNb; e += kLpThreads) {
    const int a = e / kNb, b = e % kNb;
    sL11[a][b] = (a < jb && b < a) ? M[int64_t(j0 + a) * n + j0 + b] : 0.0;
  }
  __syncthreads();
  // U12 = L11^{-1} A12 (rows j0..j0+jb-1, columns j0+jb..n-1)
  for (int c = j0 + jb + tid; c < n; c += kLpThreads) {
    double x[kNb];
#pragma unroll
    for (int i = 0; i < kNb; ++i) x[i] = i < jb ? M[int64_t(j0 + i) * n + c] : 0.0;
#pragma unroll
    for (int i = 1; i < kNb; ++i) {
      if (i >= jb) break;
      double v = x[i];
#pragma unroll
      for (int p2 = 0; p2 < kNb; ++p2)
        if (p2 < i) v -= sL11[i][p2] * x[p2];
      x[i] = v;
    }
#pragma unroll
    for (int i = 1; i < kNb; ++i)
      if (i < jb) M[int64_t(j0 + i) * n + c] = x[i];
  }
}

// ---------------------------------------------------------------------------
// Multi-workgroup panel for panels taller than the register panels (the top
// block and the largest redundant blocks in 3D): rows in blocks of kLmRows
// per workgroup, one launch per column step.  Every workgroup reduces the
// block maxima left by the previous launch to the pivot (largest |a(i, j)|
// over unpivoted candidate rows i < r, ties to the lowest row), eliminates
// column j from its own unpivoted rows and leaves its block maximum of
// column j + 1 (double-buffered by step parity).  The pivot row is flagged,
// not moved, so no workgroup reads a row that another writes in the same
// launch; after the panel the interchanges go to piv in LAPACK order and are
// applied as one permutation, with U12 = L11^{-1} A12.
// ---------------------------------------------------------------------------
constexpr int kLmRows = 256;

struct LuPanelState {
  double* pv;      // [2][nprob][nblk] block maxima
  int32_t* pi;     // [2][nprob][nblk] their rows
  int32_t* flag;   // [nprob][fstride] -1 unpivoted, else the step (rows j0..)
  int32_t* prow;   // [nprob][kNb] pivot row of each step
  int nblk;
  int64_t fstride;
};

__global__ __launch_bounds__(256) void k_lum_init(LuBatch A, LuPanelState P, int j0) {
  const int q = blockIdx.y, blk = blockIdx.x;
  const int n = A.n[q], r = A.r[q];
  if (j0 >= r || j0 + blk * kLmRows >= n) return;
  const double* M = A.base + A.moff[q];
  const int i = j0 + blk * kLmRows + threadIdx.x;
  if (i < n) P.flag[q * P.fstride + (i - j0)] = -1;
  AM loc{-1.0, INT_MAX};
  if (i < r) loc = AM{fabs(M[int64_t(i) * n + j0]), i};
  const AM b = block_argmax256(loc);
  if (threadIdx.x == 0) {
    P.pv[q * P.nblk + blk] = b.v;
    P.pi[q * P.nblk + blk] = b.i;
  }
}

__global__ __launch_bounds__(256) void k_lum_step(LuBatch A, LuPanelState P, int j0, int jj) {
  const int q = blockIdx.y, blk = blockIdx.x;
  const int n = A.n[q], r = A.r[q];
  if (j0 >= r) return;
  const int jb = min(kNb, r - j0);
  const int rb0 = j0 + blk * kLmRows;
  if (jj >= jb || rb0 >= n) return;
  double* M = A.base + A.moff[q];
  const int tid = threadIdx.x;
  const int64_t cur = int64_t(jj & 1) * A.nprob * P.nblk, nxt = int64_t((jj + 1) & 1) * A.nprob * P.nblk;
  const int nbr = (r - j0 + kLmRows - 1) / kLmRows;  // blocks holding candidate rows
  AM loc{-1.0, INT_MAX};
  for (int b = tid; b < nbr; b += 256) loc = am_better(loc, AM{P.pv[cur + q * P.nblk + b], P.pi[cur + q * P.nblk + b]});
  const AM best = block_argmax256(loc);
  if (!(best.v > 0.0)) {
    if (blk == 0 && tid == 0) atomicOr(A.status, 1);
    return;
  }
  const int rp = best.i;
  __shared__ double sp[kNb];
  if (tid < kNb) sp[tid] = tid < jb ? M[int64_t(rp) * n + j0 + tid] : 0.0;
  __syncthreads();
  if (blk == 0 && tid == 0) P.prow[q * kNb + jj] = rp;
  const int i = rb0 + tid;
  AM nx{-1.0, INT_MAX};
  if (i < n && i != rp && P.flag[q * P.fstride + (i - j0)] < 0) {
    double* row = M + int64_t(i) * n + j0;
    double y[kNb];
#pragma unroll
    for (int c = 0; c < kNb; ++c) y[c] = (c >= jj && c < jb) ? row[c] : 0.0;
    const double l = pick16(y, jj) / sp[jj];
#pragma unroll
    for (int c = 0; c < kNb; ++c) {
      if (c == jj) row[c] = l;
      else if (c > jj && c < jb) {
        y[c] -= l * sp[c];
        row[c] = y[c];
      }
    }
    if (jj + 1 < jb && i < r) nx = AM{fabs(pick16(y, jj + 1)), i};
  }
  if (i == rp) P.flag[q * P.fstride + (i - j0)] = jj;
  const AM b2 = block_argmax256(nx);
  if (tid == 0) {
    P.pv[nxt + q * P.nblk + blk] = b2.v;
    P.pi[nxt + q * P.nblk + blk] = b2.i;
  }
}

// The panel's interchanges as a permutation of at most 2 kNb rows (one wave,
// lane a holds entry a: position dst receives physical row src), and piv.
__device__ void lum_perm(const LuPanelState& P, int q, int j0, int jb, int* s_dst, int* s_src, int* s_na,
                         int32_t* piv) {
  const int lane = threadIdx.x & 63;
  if (threadIdx.x >= 64) return;
  int dst = lane < jb ? j0 + lane : -1, src = dst, na = jb;
  for (int jj = 0; jj < jb; ++jj) {
    const int rp = P.prow[q * kNb + jj];
    const unsigned long long hit = __ballot(src == rp);
    int ap;
    if (hit) {
      ap = __ffsll(hit) - 1;
    } else {
      ap = na++;
      if (lane == ap) dst = src = rp;
    }
    const int pos = __shfl(dst, ap, 64);
    if (piv && lane == 0) piv[j0 + jj] = pos;
    const int s_jj = __shfl(src, jj, 64), s_ap = __shfl(src, ap, 64);
    if (lane == jj) src = s_ap;
    if (lane == ap) src = s_jj;
  }
  if (lane < na) {
    s_dst[lane] = dst;
    s_src[lane] = src;
  }
  if (lane == 0) *s_na = na;
}

// Columns outside the panel (mode 0): the interchanges, and right of the
// panel U12 = L11^{-1} A12 with L11 from the pivot rows' panel columns (not
// written here).  Mode 1: the interchanges of the panel columns.
__global__ __launch_bounds__(256) void k_lum_finish(LuBatch A, LuPanelState P, int j0, int mode) {
  const int q = blockIdx.y;
  const int n = A.n[q], r = A.r[q];
  if (j0 >= r) return;
  const int jb = min(kNb, r - j0);
  double* M = A.base + A.moff[q];
  __shared__ int s_dst[2 * kNb], s_src[2 * kNb], s_na;
  __shared__ double sL[kNb][kNb + 1];
  lum_perm(P, q, j0, jb, s_dst, s_src, &s_na, (mode == 0 && blockIdx.x == 0) ? A.piv + A.poff[q] : nullptr);
  __syncthreads();
  const int na = s_na;
  if (mode == 1) {
    const int e = threadIdx.x;  // one thread per panel column
    if (blockIdx.x != 0 || e >= jb) return;
    const int col = j0 + e;
    double v[2 * kNb];
#pragma unroll
    for (int a2 = 0; a2 < 2 * kNb; ++a2) v[a2] = a2 < na ? M[int64_t(s_src[a2]) * n + col] : 0.0;
#pragma unroll
    for (int a2 = 0; a2 < 2 * kNb; ++a2)
      if (a2 < na && s_src[a2] != s_dst[a2]) M[int64_t(s_dst[a2]) * n + col] = v[a2];
    return;
  }
  for (int e = threadIdx.x; e < kNb * kNb; e += 256) {
    const int i = e / kNb, c = e % kNb;
    sL[i][c] = (i < jb && c < jb) ? M[int64_t(s_src[i]) * n + j0 + c] : 0.0;
  }
  bool moved = false;
  for (int a2 = 0; a2 < na; ++a2) moved = moved || s_src[a2] != s_dst[a2];
  __syncthreads();
  const int col = blockIdx.x * 256 + threadIdx.x;
  if (col >= n || (col >= j0 && col < j0 + jb)) return;
  const bool right = col >= j0 + jb;
  if (!right && !moved) return;
  double v[2 * kNb];
#pragma unroll
  for (int a2 = 0; a2 < 2 * kNb; ++a2)
    v[a2] = (a2 < na && ((right && a2 < jb) || s_src[a2] != s_dst[a2])) ? M[int64_t(s_src[a2]) * n + col] : 0.0;
  if (right) {
#pragma unroll
    for (int i = 1; i < kNb; ++i) {
      if (i >= jb) break;
      double t = v[i];
#pragma unroll
      for (int p2 = 0; p2 < kNb; ++p2)
        if (p2 < i) t -= sL[i][p2] * v[p2];
      v[i] = t;
    }
  }
#pragma unroll
  for (int a2 = 0; a2 < 2 * kNb; ++a2)
    if (a2 < na && ((right && a2 < jb) || s_src[a2] != s_dst[a2])) M[int64_t(s_dst[a2]) * n + col] = v[a2];
}

// Trailing update A22 -= L21 U12 of one 64 x 64 tile (K = panel width).
__global__ __launch_bounds__(256) void k_lu_update(LuBatch A, int j0) {
  const int q = blockIdx.z;
  const int n = A.n[q], r = A.r[q];
  if (j0 >= r) return;
  const int jb = min(kNb, r - j0);
  const int s0 = j0 + jb;
  const int rt0 = s0 + blockIdx.y * 64, ct0 = s0 + blockIdx.x * 64;
  if (rt0 >= n || ct0 >= n) return;
  double* M = A.base + A.moff[q];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int wr = wv >> 1, wc = wv & 1;
  if (A.fp32 && rt0 >= r && ct0 >= r) {
    // Schur update of the skeleton block (rows and columns >= r) in FP32
    float4_t d[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) d[a][b] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < kNb; ks += 4) {
      const int k = ks + lk;
      float af[2], bf[2];
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        const int i = rt0 + wr * 32 + a * 16 + li;
        af[a] = (i < n && k < jb) ? float(M[int64_t(i) * n + j0 + k]) : 0.f;
      }
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int c = ct0 + wc * 32 + b * 16 + li;
        bf[b] = (c < n && k < jb) ? float(M[int64_t(j0 + k) * n + c]) : 0.f;
      }
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) d[a][b] = mfma_f32(af[a], bf[b], d[a][b]);
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int i = rt0 + wr * 32 + a * 16 + 4 * lk + v;
          const int c = ct0 + wc * 32 + b * 16 + li;
          if (i < n && c < n) M[int64_t(i) * n + c] -= double(d[a][b][v]);
        }
    return;
  }
  double4_t d[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) d[a][b] = double4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int ks = 0; ks < kNb; ks += 4) {
    const int k = ks + lk;
    double af[2], bf[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const int i = rt0 + wr * 32 + a * 16 + li;
      af[a] = (i < n && k < jb) ? M[int64_t(i) * n + j0 + k] : 0.0;
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int c = ct0 + wc * 32 + b * 16 + li;
      bf[b] = (c < n && k < jb) ? M[int64_t(j0 + k) * n + c] : 0.0;
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) d[a][b] = mfma_f64(af[a], bf[b], d[a][b]);
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = rt0 + wr * 32 + a * 16 + 4 * v + lk;
        const int c = ct0 + wc * 32 + b * 16 + li;
        if (i < n && c < n) M[int64_t(i) * n + c] -= d[a][b][v];
      }
}

// Batched general GEMM, one 64 x 64 tile of C per workgroup:
// C = beta C + alpha op(A) op(B) for every entry of a problem table.
__global__ __launch_bounds__(256) void k_gemm_tiles(const GemmDesc* D, int nd) {
  const int q = blockIdx.z;
  if (q >= nd) return;
  const GemmDesc g = D[q];
  const int tm = blockIdx.y * kGemmTile, tn = blockIdx.x * kGemmTile;
  if (tm >= g.M || tn >= g.N) return;
  __shared__ double lds[kGemmLds];
  const int Mt = min(kGemmTile, g.M - tm), Nt = min(kGemmTile, g.N - tn);
  const double* Ap = g.ta ? g.A + tm : g.A + int64_t(tm) * g.lda;
  const double* Bp = g.tb ? g.B + int64_t(tn) * g.ldb : g.B + tn;
  if (g.fp32)
    wg_gemm_f32(Mt, Nt, g.K, g.alpha, Ap, g.lda, g.ta, Bp, g.ldb, g.tb, g.beta, g.C + int64_t(tm) * g.ldc + tn, g.ldc,
                lds);
  else
    wg_gemm(Mt, Nt, g.K, g.alpha, Ap, g.lda, g.ta, Bp, g.ldb, g.tb, g.beta, g.C + int64_t(tm) * g.ldc + tn, g.ldc,
            lds);
}

}  // namespace

void launch_qr_batched(const QrBatch& A, int max_rows, int max_cols, hipStream_t s) {
  if (A.nprob == 0) return;
  if (max_rows <= kTsqrMaxRows) {
    launch_tsqr(A, max_rows, max_cols, s);
    hipLaunchKernelGGL(k_qr_clear_lower, dim3(64, A.nprob), dim3(256), 0, s, A);
    HIF_HIP(hipGetLastError());
    return;
  }
  // taller problems: one workgroup per problem for the panel
  for (int j0 = 0; j0 < max_cols; j0 += kNb) {
    hipLaunchKernelGGL(k_qr_panel, dim3(A.nprob), dim3(kQpThreads), 0, s, A, j0);
    const int rem = max_cols - j0 - kNb;
    if (rem > 0) {
      const unsigned tiles = unsigned((rem + kTileN - 1) / kTileN);
      hipLaunchKernelGGL(k_qr_update, dim3(tiles, A.nprob), dim3(kQrThreads), 0, s, A, j0);
    }
  }
  hipLaunchKernelGGL(k_qr_clear_lower, dim3(64, A.nprob), dim3(256), 0, s, A);
  HIF_HIP(hipGetLastError());
}

// One rectangle copy per blockIdx.y: dst[r * dld + c] = src[r * sld + c].
struct BlockCopy {
  const double* src;
  double* dst;
  int32_t sld, dld, rows, cols;
};
__global__ void k_copy_blocks(const BlockCopy* d) {
  const BlockCopy c = d[blockIdx.y];
  const int64_t ne = int64_t(c.rows) * c.cols;
  for (int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; e < ne; e += int64_t(gridDim.x) * blockDim.x) {
    const int64_t r = e / c.cols, k = e % c.cols;
    c.dst[r * c.dld + k] = c.src[r * c.sld + k];
  }
}

static void copy_blocks(const std::vector<BlockCopy>& h, MemTracker* mt, hipStream_t s) {
  if (h.empty()) return;
  DBuf<BlockCopy> d;
  d.alloc(h.size(), mt);
  HIF_HIP(hipMemcpyAsync(d.p, h.data(), sizeof(BlockCopy) * h.size(), hipMemcpyHostToDevice, s));
  for (size_t i = 0; i < h.size(); i += 65535) {
    const unsigned cnt = unsigned(std::min<size_t>(65535, h.size() - i));
    hipLaunchKernelGGL(k_copy_blocks, dim3(256, cnt), dim3(256), 0, s, d.p + i);
  }
  HIF_HIP(hipGetLastError());
}

void launch_rowqr_split(double* base, const std::vector<int64_t>& moff, const std::vector<int32_t>& ld,
                        const std::vector<int32_t>& rows, const std::vector<int32_t>& cols, MemTracker* mt,
                        hipStream_t s) {
  // The R factor of [Y_1; ...; Y_b] is that of [R_1; ...; R_b] with
  // Y_i = Q_i R_i (up to row signs, which the ID does not see), and only R
  // is needed.  Blocks of 4096..8192 rows (n <= 2048) shrink the stack at
  // least 2-fold a round; blocks of 16384..32768 rows (n <= 16384) leave a
  // stack of nb n rows, which a round of 2 blocks brings to one block.
  struct Prob {
    int64_t off;
    int32_t ld, rows, cols, orig;
  };
  int maxn = 1;
  std::vector<Prob> cur;
  for (size_t q = 0; q < rows.size(); ++q)
    if (rows[q] > cols[q]) {
      cur.push_back({moff[q], ld[q], rows[q], cols[q], int32_t(q)});
      maxn = std::max(maxn, cols[q]);
    }
  HIF_REQUIRE(maxn <= kTsqrSplitRows / 2, HIF_EUNSUPPORTED, "row compression of more than 16384 columns");
  const int B = maxn <= 2048 ? 8192 : kTsqrSplitRows;
  double* rbase = base;     // buffer of this round's problems
  DBuf<double> stack[2];    // stacks of R factors, alternating by round
  for (int round = 0; !cur.empty(); ++round) {
    std::vector<int64_t> h_off, h_soff;
    std::vector<int32_t> h_ld, h_rows, h_cols;
    std::vector<int32_t> nblk(cur.size());
    int64_t stot = 0, next_tot = 0;
    int maxr = 1, maxc = 1;
    for (size_t i = 0; i < cur.size(); ++i) {
      const Prob& p = cur[i];
      const int nb = p.rows > B ? (p.rows + B - 1) / B : 1;
      nblk[i] = nb;
      for (int b = 0; b < nb; ++b) {
        const int r0 = int(int64_t(p.rows) * b / nb), r1 = int(int64_t(p.rows) * (b + 1) / nb);
        h_off.push_back(p.off + int64_t(r0) * p.ld);
        h_ld.push_back(p.ld);
        h_rows.push_back(r1 - r0);
        h_cols.push_back(p.cols);
        h_soff.push_back(stot);
        stot += rowqr_scratch(r1 - r0, p.cols);
        maxr = std::max(maxr, r1 - r0);
        maxc = std::max(maxc, p.cols);
      }
      if (nb > 1) next_tot += int64_t(nb) * p.cols * p.cols;
    }
    const int np = int(h_off.size());
    DBuf<int64_t> d_off, d_soff;
    DBuf<int32_t> d_ld, d_rows, d_cols;
    DBuf<double> scratch;
    d_off.alloc(np, mt);
    d_soff.alloc(np, mt);
    d_ld.alloc(np, mt);
    d_rows.alloc(np, mt);
    d_cols.alloc(np, mt);
    scratch.alloc(stot + 1, mt);
    HIF_HIP(hipMemcpyAsync(d_off.p, h_off.data(), sizeof(int64_t) * np, hipMemcpyHostToDevice, s));
    HIF_HIP(hipMemcpyAsync(d_soff.p, h_soff.data(), sizeof(int64_t) * np, hipMemcpyHostToDevice, s));
    HIF_HIP(hipMemcpyAsync(d_ld.p, h_ld.data(), sizeof(int32_t) * np, hipMemcpyHostToDevice, s));
    HIF_HIP(hipMemcpyAsync(d_rows.p, h_rows.data(), sizeof(int32_t) * np, hipMemcpyHostToDevice, s));
    HIF_HIP(hipMemcpyAsync(d_cols.p, h_cols.data(), sizeof(int32_t) * np, hipMemcpyHostToDevice, s));
    QrBatch A{};
    A.base = rbase;
    A.moff = d_off.p;
    A.ld = d_ld.p;
    A.rows = d_rows.p;
    A.cols = d_cols.p;
    A.scratch = scratch.p;
    A.soff = d_soff.p;
    A.nprob = np;
    // every block has at most B <= kTsqrSplitRows rows: one TSQR stack
    launch_qr_batched(A, maxr, maxc, s);
    // Unsplit problems are done (copied home if they are stacks); split ones
    // become stacks of their blocks' n x n R factors (lower parts cleared).
    DBuf<double>& nxt = stack[round & 1];
    if (next_tot > 0) nxt.alloc(next_tot, mt);
    std::vector<Prob> next;
    std::vector<BlockCopy> gather, back;
    int64_t noff = 0;
    size_t k = 0;
    for (size_t i = 0; i < cur.size(); ++i) {
      const Prob& p = cur[i];
      const int nb = nblk[i];
      if (nb == 1) {
        if (round > 0)
          back.push_back({rbase + p.off, base + moff[p.orig], p.ld, ld[p.orig], p.cols, p.cols});
        ++k;
        continue;
      }
      for (int b = 0; b < nb; ++b, ++k)
        gather.push_back({rbase + h_off[k], nxt.p + noff + int64_t(b) * p.cols * p.cols, p.ld, p.cols, p.cols,
                          p.cols});
      next.push_back({noff, p.cols, nb * p.cols, p.cols, p.orig});
      noff += int64_t(nb) * p.cols * p.cols;
    }
    // both copies read this round's buffer, which the round after next
    // allocates over (stream-ordered)
    copy_blocks(back, mt, s);
    copy_blocks(gather, mt, s);
    cur.swap(next);
    rbase = nxt.p;
  }
}

void launch_lu_batched(const LuBatch& A, int max_r, int max_n, hipStream_t s) {
  if (A.nprob == 0) return;
  // state of the multi-workgroup panel (panels taller than kLpRows)
  DBuf<double> pv;
  DBuf<int32_t> pi, flag, prow;
  LuPanelState P{};
  if (max_n > kLpRows) {
    P.nblk = (max_n + kLmRows - 1) / kLmRows;
    P.fstride = max_n;
    pv.alloc(size_t(2) * A.nprob * P.nblk, nullptr);
    pi.alloc(size_t(2) * A.nprob * P.nblk, nullptr);
    flag.alloc(size_t(A.nprob) * max_n, nullptr);
    prow.alloc(size_t(A.nprob) * kNb, nullptr);
    P.pv = pv.p;
    P.pi = pi.p;
    P.flag = flag.p;
    P.prow = prow.p;
  }
  const hif_tuning tu = tuning();
  for (int j0 = 0; j0 < max_r; j0 += kNb) {
    if (max_n - j0 > kLpRows) {
      const dim3 g(unsigned((max_n - j0 + kLmRows - 1) / kLmRows), unsigned(A.nprob));
      hipLaunchKernelGGL(k_lum_init, g, dim3(256), 0, s, A, P, j0);
      for (int jj = 0; jj < kNb; ++jj) hipLaunchKernelGGL(k_lum_step, g, dim3(256), 0, s, A, P, j0, jj);
      hipLaunchKernelGGL(k_lum_finish, dim3(unsigned((max_n + 255) / 256), unsigned(A.nprob)), dim3(256), 0, s, A,
                         P, j0, 0);
      hipLaunchKernelGGL(k_lum_finish, dim3(1, unsigned(A.nprob)), dim3(256), 0, s, A, P, j0, 1);
    } else {
      // two rows per thread: at least (panel rows) / 2 threads; within that,
      // the thread count of the launch-shape table for the panel's size
      const int rows = max_n - j0;
      int threads = rows <= kLpRows / 4 ? tu.lu_panel_threads[0] : (rows <= kLpRows / 2 ? tu.lu_panel_threads[1] : 1024);
      if (2 * threads < rows) threads = rows <= kLpRows / 2 ? 512 : 1024;
      if (threads == 256)
        hipLaunchKernelGGL(k_lu_panel_reg<256>, dim3(A.nprob), dim3(256), 0, s, A, j0);
      else if (threads == 512)
        hipLaunchKernelGGL(k_lu_panel_reg<512>, dim3(A.nprob), dim3(512), 0, s, A, j0);
      else
        hipLaunchKernelGGL(k_lu_panel_reg<1024>, dim3(A.nprob), dim3(1024), 0, s, A, j0);
    }
    const int rem = max_n - j0 - 1;
    if (rem > 0) {
      const unsigned tiles = unsigned((rem + 63) / 64);
      hipLaunchKernelGGL(k_lu_update, dim3(tiles, tiles, A.nprob), dim3(256), 0, s, A, j0);
    }
  }
  HIF_HIP(hipGetLastError());
}

void launch_gemm_tiles(const GemmDesc* D, int nd, int max_m, int max_n, hipStream_t s) {
  if (nd == 0 || max_m <= 0 || max_n <= 0) return;
  const unsigned tx = unsigned((max_n + kGemmTile - 1) / kGemmTile), ty = unsigned((max_m + kGemmTile - 1) / kGemmTile);
  hipLaunchKernelGGL(k_gemm_tiles, dim3(tx, ty, nd), dim3(256), 0, s, D, nd);
  HIF_HIP(hipGetLastError());
}

}  // namespace hif
