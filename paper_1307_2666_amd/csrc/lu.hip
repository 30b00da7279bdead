// Partial LU with partial pivoting (Lemma 2.1) of many n x n problems over
// their first r columns, pivots chosen among rows < r: the eliminations of the
// groups and the top block.
//
// Two levels of blocking.  An outer panel of 64 columns is factored 16
// columns at a time (its own columns right of the 16 updated at once); the
// interchanges and U12 of all other columns then follow for the 64 steps
// together, and the trailing block takes one update of depth 64: with 16 it
// was read and written four times as often, which bound the large problems
// (135 of 192 ms of a 9870-unknown top block).
#include <algorithm>
#include <climits>
#include <mutex>

#include "batched.h"
#include "gemm.h"
#include "select.h"

namespace hif {

namespace {

constexpr int kNb = 16;  // columns factored at a time
constexpr int kNo = 64;  // outer panel

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

// Best candidate of a workgroup of 256 threads (NaN is none); lane reductions
// in the vector ALU.
__device__ AM block_argmax256(AM x) {
  __shared__ double sv[4];
  __shared__ int si[4];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const double v = fmax(x.v, -1.0), mx = wave_max(v);
  const int mi = wave_min(v == mx ? x.i : INT_MAX);
  if (lane == 0) {
    sv[wv] = mx;
    si[wv] = mi;
  }
  __syncthreads();
  AM r[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) r[k] = AM{sv[k], si[k]};
  __syncthreads();
  return am_better(am_better(r[0], r[1]), am_better(r[2], r[3]));
}

// ---------------------------------------------------------------------------
// Outer panel of problems with at most 2 NT rows from row J on, one workgroup
// each.  16 columns at a time: thread t holds rows j0 + t and j0 + t + NT of
// them in registers through their elimination steps.  A step has one barrier:
// each wave publishes its best candidate with the whole row (16 entries), so
// that after the barrier every thread knows the pivot and has its row.  Then
// the interchanges of the panel's other columns, U12 of those right of the 16,
// and their update on the matrix cores.  Bound by that chain: about 0.6 us a
// step.
// ---------------------------------------------------------------------------
constexpr int kLpRows = 2048;  // rows of the largest register panel (1024 threads)

template <int NT>
__global__ __launch_bounds__(NT) void k_lu_panel(LuBatch A, int J) {
  constexpr int NW = NT / 64;
  const int q = blockIdx.x;
  const int n = A.n[q], r = A.r[q];
  if (J >= r) return;
  double* M = A.base + A.moff[q];
  int32_t* piv = A.piv + A.poff[q];
  const int Je = min(J + kNo, r);
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  __shared__ double s_val[2][NW];
  __shared__ int s_row[2][NW];
  alignas(16) __shared__ double s_cand[2][NW][kNb], s_top[2][kNb];
  __shared__ double sL[kNb][kNb + 1];
  __shared__ int s_piv[kNb], s_dst[2 * kNb], s_src[2 * kNb], s_na;
  for (int j0 = J; j0 < Je; j0 += kNb) {
    const int jb = min(kNb, Je - j0);
    double y[2][kNb];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int R = j0 + tid + u * NT;
      const double* src = M + int64_t(R < n ? R : j0) * n + j0;
#pragma unroll
      for (int c = 0; c < kNb; ++c) {
        const double t = src[c < jb ? c : 0];
        y[u][c] = (R < n && c < jb) ? t : 0.0;
      }
    }
#pragma unroll
    for (int jj = 0; jj < kNb; ++jj) {
      if (jj < jb) {
        const int j = j0 + jj, b = jj & 1;
        const int R0 = j0 + tid, R1 = j0 + tid + NT;
        const double c0 = (tid >= jj && R0 < r) ? fmax(fabs(y[0][jj]), -1.0) : -1.0;
        const double c1 = R1 < r ? fmax(fabs(y[1][jj]), -1.0) : -1.0;
        const double mx = wave_max(fmax(c0, c1));
        const unsigned long long b0 = __ballot(c0 == mx), b1 = __ballot(c1 == mx);
        const int bl = b0 ? __ffsll(b0) - 1 : __ffsll(b1) - 1;  // lowest row of the wave's best
        if (lane == bl) {
          s_val[b][wv] = mx;
          s_row[b][wv] = b0 ? R0 : R1;
#pragma unroll
          for (int c = 0; c < kNb; c += 2)
            *reinterpret_cast<double2*>(&s_cand[b][wv][c]) =
                b0 ? double2{y[0][c], y[0][c + 1]} : double2{y[1][c], y[1][c + 1]};
        }
        if (tid == jj) {
#pragma unroll
          for (int c = 0; c < kNb; c += 2) *reinterpret_cast<double2*>(&s_top[b][c]) = double2{y[0][c], y[0][c + 1]};
        }
        __syncthreads();
        // the waves' best, compared across lanes; ties to the lowest row
        const double wvl = s_val[b][lane & (NW - 1)];
        const int wrw = s_row[b][lane & (NW - 1)];
        const double bv = group_max<NW>(wvl);
        const int p = __builtin_amdgcn_readfirstlane(group_min<NW>(wvl == bv ? wrw : INT_MAX));
        const int bw = ((p - j0) & (NT - 1)) >> 6;
        if (!(bv > 0.0)) {
          if (tid == 0) atomicOr(A.status, 1);
          if (tid < Je - j0) piv[j0 + tid] = j0 + tid;  // what follows reads them
          return;
        }
        double pr[kNb];  // the new row j
#pragma unroll
        for (int c = 0; c < kNb; c += 2) {
          const double2 t = *reinterpret_cast<const double2*>(&s_cand[b][bw][c]);
          pr[c] = t.x;
          pr[c + 1] = t.y;
        }
        if (tid == 0) s_piv[jj] = p;
        if (p != j) {
          if (tid == jj) {
#pragma unroll
            for (int c = 0; c < kNb; ++c) y[0][c] = pr[c];
          }
          if (R0 == p) {
#pragma unroll
            for (int c = 0; c < kNb; ++c) y[0][c] = s_top[b][c];
          }
          if (R1 == p) {
#pragma unroll
            for (int c = 0; c < kNb; ++c) y[1][c] = s_top[b][c];
          }
        }
        const double inv = 1.0 / pr[jj];
        const double l0 = tid > jj ? y[0][jj] * inv : 0.0, l1 = y[1][jj] * inv;
        if (tid > jj) y[0][jj] = l0;
        y[1][jj] = l1;
#pragma unroll
        for (int c = jj + 1; c < kNb; ++c) {
          y[0][c] -= l0 * pr[c];
          y[1][c] -= l1 * pr[c];
        }
        // the slots of this parity are written again two steps on, past the
        // next step's barrier, which follows every read above
      }
    }
    // the 16 columns back to memory, L11 to LDS
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int R = j0 + tid + u * NT;
      if (R < n) {
        double* dst = M + int64_t(R) * n + j0;
#pragma unroll
        for (int c = 0; c < kNb; ++c)
          if (c < jb) dst[c] = y[u][c];
      }
    }
    if (tid < kNb)
#pragma unroll
      for (int c = 0; c < kNb; ++c) sL[tid][c] = (tid < jb && c < tid) ? y[0][c] : 0.0;
    __syncthreads();
    if (tid < jb) piv[j0 + tid] = s_piv[tid];
    const int nl = j0 - J, nr = Je - j0 - jb;  // the panel's other columns, left and right
    if (nl + nr == 0) break;
    if (wv == 0) compose_swaps(s_piv, j0, jb, n, s_dst, s_src, &s_na);
    __syncthreads();
    {
      const int na = s_na, nc = nl + nr;
      constexpr int kE = (2 * kNb * (kNo - kNb) + NT - 1) / NT;
      double v[kE];
#pragma unroll
      for (int k = 0; k < kE; ++k) {
        const int e = tid + k * NT, a = e / nc, c = e - a * nc;
        const int col = c < nl ? J + c : j0 + jb + (c - nl);
        v[k] = a < na ? M[int64_t(s_src[a]) * n + col] : 0.0;
      }
      __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): every row is read before any is written
      __syncthreads();
#pragma unroll
      for (int k = 0; k < kE; ++k) {
        const int e = tid + k * NT, a = e / nc, c = e - a * nc;
        const int col = c < nl ? J + c : j0 + jb + (c - nl);
        if (a < na) M[int64_t(s_dst[a]) * n + col] = v[k];
      }
    }
    __syncthreads();
    if (nr == 0) break;
    if (tid < nr) {  // U12 = L11^{-1} A12
      double* col = M + int64_t(j0) * n + j0 + jb + tid;
      double x[kNb];
#pragma unroll
      for (int i = 0; i < kNb; ++i) x[i] = col[int64_t(i) * n];  // nr > 0: jb == 16
#pragma unroll
      for (int i = 1; i < kNb; ++i) {
        double t = x[i];
#pragma unroll
        for (int p2 = 0; p2 < kNb; ++p2)
          if (p2 < i) t -= sL[i][p2] * x[p2];
        x[i] = t;
      }
#pragma unroll
      for (int i = 1; i < kNb; ++i) col[int64_t(i) * n] = x[i];
    }
    __syncthreads();
    // update of the panel's columns right of the 16 (at most 48): row tiles of
    // 16 over the waves, up to three column tiles each
    {
      const int cb = j0 + kNb;
      double bf[3][4];
#pragma unroll
      for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int c = 16 * t + li;
          const double v = M[int64_t(j0 + 4 * s + lk) * n + cb + (c < nr ? c : 0)];
          bf[t][s] = c < nr ? -v : 0.0;
        }
      for (int r0 = cb + 16 * wv; r0 < n; r0 += 16 * NW) {
        double af[4];
        const int ra = min(r0 + li, n - 1);
#pragma unroll
        for (int s = 0; s < 4; ++s) af[s] = M[int64_t(ra) * n + j0 + 4 * s + lk];
        double4_t d[3];
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            d[t][v] = M[int64_t(min(r0 + 4 * v + lk, n - 1)) * n + cb + (16 * t + li < nr ? 16 * t + li : 0)];
#pragma unroll
        for (int t = 0; t < 3; ++t) {
#pragma unroll
          for (int s = 0; s < 4; ++s) d[t] = mfma_f64(af[s], bf[t][s], d[t]);
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (16 * t + li < nr && r0 + 4 * v + lk < n) M[int64_t(r0 + 4 * v + lk) * n + cb + 16 * t + li] = d[t][v];
        }
      }
    }
    __syncthreads();
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
// launch; after the 16 columns the interchanges go to piv in LAPACK order and
// are applied to the outer panel's columns as one permutation, with
// U12 = L11^{-1} A12 there.
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
  if (blk == 0 && threadIdx.x < kNb) P.prow[q * kNb + threadIdx.x] = j0 + int(threadIdx.x);
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
  // the block maxima, and the workgroup's rows, on their way while the pivot is
  // found: a 6255-unknown block's LU 51.7 ms when they were read after it and the
  // candidates compared by shuffles, 48.2 so
  const int64_t c0 = cur + q * P.nblk;
  AM loc{P.pv[c0 + min(tid, nbr - 1)], P.pi[c0 + min(tid, nbr - 1)]};
  const int i = rb0 + tid, ic = min(i, n - 1);
  double* row = M + int64_t(ic) * n + j0;
  double y[kNb];
#pragma unroll
  for (int c = 0; c < kNb; ++c) y[c] = (c >= jj && c < jb) ? row[c] : 0.0;
  const int done = P.flag[q * P.fstride + (ic - j0)];
  for (int b = tid + 256; b < nbr; b += 256) loc = am_better(loc, AM{P.pv[c0 + b], P.pi[c0 + b]});
  const AM best = block_argmax256(loc);
  if (!(best.v > 0.0)) {
    // P.prow stays at the step's own row (k_lum_init); the slot the next step
    // reads is undefined memory or an earlier step's until it is written
    if (tid == 0) {
      P.pv[nxt + q * P.nblk + blk] = -1.0;
      P.pi[nxt + q * P.nblk + blk] = INT_MAX;
      if (blk == 0) atomicOr(A.status, 1);
    }
    return;
  }
  const int rp = best.i;
  __shared__ double sp[kNb];
  if (tid < kNb) sp[tid] = tid < jb ? M[int64_t(rp) * n + j0 + tid] : 0.0;
  __syncthreads();
  if (blk == 0 && tid == 0) P.prow[q * kNb + jj] = rp;
  AM nx{-1.0, INT_MAX};
  if (i < n && i != rp && done < 0) {
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
    const int rp = P.prow[q * kNb + jj];  // a row of the panel: every slot k_lum_step reads has been written
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

// The outer panel's columns outside the 16 (mode 0): the interchanges, and
// right of the 16 U12 = L11^{-1} A12 with L11 from the pivot rows' entries in
// the 16 (not written here).  Mode 1: the interchanges of the 16 columns.
__global__ __launch_bounds__(kNo) void k_lum_finish(LuBatch A, LuPanelState P, int J, int j0, int mode) {
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
  for (int e = threadIdx.x; e < kNb * kNb; e += kNo) {
    const int i = e / kNb, c = e % kNb;
    sL[i][c] = (i < jb && c < jb) ? M[int64_t(s_src[i]) * n + j0 + c] : 0.0;
  }
  bool moved = false;
  for (int a2 = 0; a2 < na; ++a2) moved = moved || s_src[a2] != s_dst[a2];
  __syncthreads();
  const int col = J + int(threadIdx.x);
  if (col >= min(J + kNo, r) || (col >= j0 && col < j0 + jb)) return;
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

// Update of the outer panel's columns right of the 16: wave per 16 rows.
__global__ __launch_bounds__(256) void k_lum_update(LuBatch A, int J, int j0) {
  const int q = blockIdx.y;
  const int n = A.n[q], r = A.r[q];
  const int cb = j0 + kNb, nr = min(J + kNo, r) - cb;
  if (nr <= 0) return;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int r0 = cb + 64 * int(blockIdx.x) + 16 * wv;
  if (r0 >= n) return;
  double* M = A.base + A.moff[q];
  double af[4], bf[3][4];
  const int ra = min(r0 + li, n - 1);
#pragma unroll
  for (int s = 0; s < 4; ++s) af[s] = M[int64_t(ra) * n + j0 + 4 * s + lk];
  double4_t d[3];
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    const int c = 16 * t + li < nr ? 16 * t + li : 0;
#pragma unroll
    for (int s = 0; s < 4; ++s) bf[t][s] = -M[int64_t(j0 + 4 * s + lk) * n + cb + c];
#pragma unroll
    for (int v = 0; v < 4; ++v) d[t][v] = M[int64_t(min(r0 + 4 * v + lk, n - 1)) * n + cb + c];
  }
#pragma unroll
  for (int t = 0; t < 3; ++t) {
#pragma unroll
    for (int s = 0; s < 4; ++s) d[t] = mfma_f64(af[s], bf[t][s], d[t]);
#pragma unroll
    for (int v = 0; v < 4; ++v)
      if (16 * t + li < nr && r0 + 4 * v + lk < n) M[int64_t(r0 + 4 * v + lk) * n + cb + 16 * t + li] = d[t][v];
  }
}

// ---------------------------------------------------------------------------
// After an outer panel: the columns outside it, 64 per workgroup.  All rows
// the interchanges move (the panel's and up to 64 others) are read before any
// is written; right of the panel the panel's rows become U12 = L11^{-1} A12 in
// LDS, 16 rows at a time (substitution by a thread per column, the rows below
// on the matrix cores).  LDS for two workgroups a CU.
// ---------------------------------------------------------------------------
constexpr int kSwLd = kNo + 1;
constexpr size_t kSwapLds = size_t(2 * kNo) * kSwLd * sizeof(double);
__global__ __launch_bounds__(256, 2) void k_lu_swap(LuBatch A, int J) {
  const int q = blockIdx.y;
  const int n = A.n[q], r = A.r[q];
  const int ct = int(blockIdx.x) * kNo;
  if (J >= r || ct >= n) return;
  const int Je = min(J + kNo, r), nj = Je - J;
  if (ct == J && Je == min(J + kNo, n)) return;  // the panel itself
  double* M = A.base + A.moff[q];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  extern __shared__ double smem[];
  double* sX = smem;               // [kNo][kSwLd] the panel's rows
  double* sL = smem + kNo * kSwLd;  // [kNo][kSwLd]
  __shared__ int s_dst[2 * kNo], s_src[2 * kNo], s_na;
  if (wv == 0) compose_swaps(A.piv + A.poff[q] + J, J, nj, n, s_dst, s_src, &s_na);
  const bool right = ct + kNo > Je;  // the tile has columns right of the panel
  if (right)
    for (int e = tid; e < kNo * kNo; e += 256) {
      const int i = e >> 6, c = e & 63;
      const double t = M[int64_t(J + (i < nj ? i : 0)) * n + J + (c < nj ? c : 0)];
      sL[i * kSwLd + c] = (i < nj && c < i) ? t : 0.0;
    }
  __syncthreads();
  const int na = s_na;
  if (!right) {  // left of the panel: nothing to do where no row moves
    bool moved = false;
    for (int a = 0; a < na; ++a) moved = moved || s_src[a] != s_dst[a];
    if (!moved) return;
  }
  const int col = ct + lane;
  const bool mine = col < n && (col < J || col >= Je);
  const int lc = mine ? col : (ct < J ? ct : Je);  // a column that may be read (Je < n: the tile has one to its right)
  double vp[16], ve[16];  // rows wv + 4 k of the panel's and of the others
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    vp[k] = M[int64_t(s_src[min(wv + 4 * k, nj - 1)]) * n + lc];
    ve[k] = M[int64_t(s_src[min(nj + wv + 4 * k, na - 1)]) * n + lc];
  }
#pragma unroll
  for (int k = 0; k < 16; ++k) sX[(wv + 4 * k) * kSwLd + lane] = wv + 4 * k < nj ? vp[k] : 0.0;
  __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): every row is read before any is written
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 16; ++k)
    if (mine && nj + wv + 4 * k < na) M[int64_t(s_dst[nj + wv + 4 * k]) * n + col] = ve[k];
  if (right) {
    for (int b = 0; b < nj; b += kNb) {
      if (tid < kNo) {
        double x[kNb];
#pragma unroll
        for (int i = 0; i < kNb; ++i) x[i] = sX[(b + i) * kSwLd + tid];
#pragma unroll
        for (int i = 1; i < kNb; ++i) {
          double t = x[i];
#pragma unroll
          for (int p = 0; p < kNb; ++p)
            if (p < i) t -= sL[(b + i) * kSwLd + b + p] * x[p];
          x[i] = t;
        }
#pragma unroll
        for (int i = 1; i < kNb; ++i) sX[(b + i) * kSwLd + tid] = x[i];
      }
      __syncthreads();
      if (b + kNb < nj) {  // wave w: columns 16 w .. of the rows below
        double bf[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) bf[s] = -sX[(b + 4 * s + lk) * kSwLd + 16 * wv + li];
        for (int rt = b + kNb; rt < kNo; rt += 16) {
          double4_t d;
#pragma unroll
          for (int v = 0; v < 4; ++v) d[v] = sX[(rt + 4 * v + lk) * kSwLd + 16 * wv + li];
#pragma unroll
          for (int s = 0; s < 4; ++s) d = mfma_f64(sL[(rt + li) * kSwLd + b + 4 * s + lk], bf[s], d);
#pragma unroll
          for (int v = 0; v < 4; ++v) sX[(rt + 4 * v + lk) * kSwLd + 16 * wv + li] = d[v];
        }
        __syncthreads();
      }
    }
  }
  if (mine)
    for (int a = wv; a < nj; a += 4)
      if (col >= Je || s_src[a] != J + a) M[int64_t(J + a) * n + col] = sX[a * kSwLd + lane];
}

// ---------------------------------------------------------------------------
// Trailing update A22 -= L21 U12 of one 64 x 64 tile, depth up to 64: both
// operands staged in LDS by one burst of loads, wave (wr, wc) 32 x 32 of it.
// 4096 matrix-core cycles for 64 KB of the block read and written: bound by
// memory (a 9870-unknown block's first update, 1.5 GB, takes 0.52 ms).
// ---------------------------------------------------------------------------
constexpr int kUaLd = 68, kUbLd = 80;  // row strides that spread the fragments over the banks
constexpr size_t kUpdLds = size_t(kNo) * (kUaLd + kUbLd) * sizeof(double);
__global__ __launch_bounds__(256, 2) void k_lu_update(LuBatch A, int J) {
  const int q = blockIdx.z;
  const int n = A.n[q], r = A.r[q];
  if (J >= r) return;
  const int Je = min(J + kNo, r), K = Je - J;
  const int rt0 = Je + int(blockIdx.y) * 64, ct0 = Je + int(blockIdx.x) * 64;
  if (rt0 >= n || ct0 >= n) return;
  double* M = A.base + A.moff[q];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const int wr = wv >> 1, wc = wv & 1;
  extern __shared__ double smem[];
  double* sA = smem;               // [64 rows][kUaLd]
  double* sB = smem + kNo * kUaLd;  // [64 k][kUbLd]
  double4_t d[2][2];
  {
    double a[16], b[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int i = wv + 4 * u;  // a row of either operand, lane = its column
      const double ta = M[int64_t(min(rt0 + i, n - 1)) * n + J + min(lane, K - 1)];
      const double tb = M[int64_t(J + min(i, K - 1)) * n + min(ct0 + lane, n - 1)];
      a[u] = lane < K ? ta : 0.0;
      b[u] = i < K ? -tb : 0.0;
    }
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < 2; ++y)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          d[x][y][v] = M[int64_t(min(rt0 + wr * 32 + x * 16 + 4 * v + lk, n - 1)) * n +
                         min(ct0 + wc * 32 + y * 16 + li, n - 1)];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int i = wv + 4 * u;
      sA[i * kUaLd + lane] = a[u];
      sB[i * kUbLd + lane] = b[u];
    }
  }
  __syncthreads();
  if (A.fp32 && rt0 >= r && ct0 >= r) {
    // Schur update of the skeleton block (rows and columns >= r) on the FP32
    // matrix cores, 16 products at a time summed in FP32, the sums in FP64
    for (int k0 = 0; k0 < K; k0 += kNb) {
      float4_t f[2][2];
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) f[x][y] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < kNb; ks += 4) {
        float af[2], bf[2];
#pragma unroll
        for (int x = 0; x < 2; ++x) af[x] = float(sA[(wr * 32 + x * 16 + li) * kUaLd + k0 + ks + lk]);
#pragma unroll
        for (int y = 0; y < 2; ++y) bf[y] = float(sB[(k0 + ks + lk) * kUbLd + wc * 32 + y * 16 + li]);
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int y = 0; y < 2; ++y) f[x][y] = mfma_f32(af[x], bf[y], f[x][y]);
      }
      // element v of the FP32 layout is row 4 lk + v, of the FP64 one 4 v + lk
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int i = rt0 + wr * 32 + x * 16 + 4 * lk + v, c = ct0 + wc * 32 + y * 16 + li;
            if (i < n && c < n) M[int64_t(i) * n + c] += double(f[x][y][v]);
          }
    }
    return;
  }
  for (int ks = 0; ks < K; ks += 4) {
    double af[2], bf[2];
#pragma unroll
    for (int x = 0; x < 2; ++x) af[x] = sA[(wr * 32 + x * 16 + li) * kUaLd + ks + lk];
#pragma unroll
    for (int y = 0; y < 2; ++y) bf[y] = sB[(ks + lk) * kUbLd + wc * 32 + y * 16 + li];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < 2; ++y) d[x][y] = mfma_f64(af[x], bf[y], d[x][y]);
  }
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = rt0 + wr * 32 + x * 16 + 4 * v + lk, c = ct0 + wc * 32 + y * 16 + li;
        if (i < n && c < n) M[int64_t(i) * n + c] = d[x][y][v];
      }
}

}  // namespace

static void allow_lu_lds() {
  static std::once_flag once;
  std::call_once(once, [] {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_lu_swap), hipFuncAttributeMaxDynamicSharedMemorySize,
                              int(kSwapLds));
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_lu_update), hipFuncAttributeMaxDynamicSharedMemorySize,
                              int(kUpdLds));
    (void)hipGetLastError();
  });
}

void launch_lu_batched(const LuBatch& A, int max_r, int max_n, hipStream_t s) {
  if (A.nprob == 0) return;
  allow_lu_lds();
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
  const unsigned np = unsigned(A.nprob);
  for (int J = 0; J < max_r; J += kNo) {
    const int rows = max_n - J;
    if (rows > kLpRows) {
      for (int j0 = J; j0 < std::min(J + kNo, max_r); j0 += kNb) {
        const dim3 g(unsigned((max_n - j0 + kLmRows - 1) / kLmRows), np);
        hipLaunchKernelGGL(k_lum_init, g, dim3(256), 0, s, A, P, j0);
        for (int jj = 0; jj < kNb; ++jj) hipLaunchKernelGGL(k_lum_step, g, dim3(256), 0, s, A, P, j0, jj);
        hipLaunchKernelGGL(k_lum_finish, dim3(1, np), dim3(kNo), 0, s, A, P, J, j0, 0);
        hipLaunchKernelGGL(k_lum_finish, dim3(1, np), dim3(kNo), 0, s, A, P, J, j0, 1);
        if (j0 + kNb < std::min(J + kNo, max_r))
          hipLaunchKernelGGL(k_lum_update, dim3(unsigned((max_n - j0 - kNb + 63) / 64), np), dim3(256), 0, s, A, J, j0);
      }
    } else {
      // two rows per thread: at least (panel rows) / 2 threads; within that,
      // the thread count of the launch-shape table for the panel's size
      int threads = rows <= kLpRows / 4 ? tu.lu_panel_threads[0] : (rows <= kLpRows / 2 ? tu.lu_panel_threads[1] : 1024);
      if (2 * threads < rows) threads = rows <= kLpRows / 2 ? 512 : 1024;
      if (threads == 256)
        hipLaunchKernelGGL(k_lu_panel<256>, dim3(np), dim3(256), 0, s, A, J);
      else if (threads == 512)
        hipLaunchKernelGGL(k_lu_panel<512>, dim3(np), dim3(512), 0, s, A, J);
      else
        hipLaunchKernelGGL(k_lu_panel<1024>, dim3(np), dim3(1024), 0, s, A, J);
    }
    // every problem has at most max_n columns; whether one has any outside its
    // panel does not follow from the maxima (blocks of 64 and of 20 columns, the
    // second over its first 5: they would be taken for two whole panels)
    const unsigned tiles = unsigned((max_n + kNo - 1) / kNo);
    hipLaunchKernelGGL(k_lu_swap, dim3(tiles, np), dim3(256), kSwapLds, s, A, J);
    const int rem = max_n - J - 1;
    if (rem > 0) {
      const unsigned ut = unsigned((rem + 63) / 64);
      hipLaunchKernelGGL(k_lu_update, dim3(ut, ut, np), dim3(256), kUpdLds, s, A, J);
    }
  }
  HIF_HIP(hipGetLastError());
}

}  // namespace hif
