// Blocked column-pivoted Householder QR of the IDs' large problems (Lemma 2.2,
// Section 2.2: at every step the column of largest remaining norm, stopped at
// the first pivot with |R_ii| <= tol |R_00|), then T = R11^{-1} R12.
//
// The pivots of a block of up to 32 steps are chosen first, from the Gram
// matrix G = Y^T Y of the trailing columns, as the pivoted Cholesky
// factorization of G takes them: its diagonal entries are the squared norms of
// what is left of the columns, so a step costs one row of G instead of a pass
// over all of Y.  Only the choice comes from G.  The chosen columns are moved
// to the front and factored by the Householder panels of the row compression
// (tsqr.hip), which also update the trailing columns, and the rank rule is
// applied to the panel's own R_ii.  G follows by the Cholesky rows; once the
// largest norm has fallen to kPqRefresh of what it was when G was formed, G is
// formed again from Y, so that the norms compared are good to about 1e-10 of
// the largest one.
//
// A step of the delayed-update formulation read the whole trailing block
// (29 us a step for 64 problems of 731 columns, 71 us for 8 of 3298) after a
// pivot search and column update of its own (10-18 us).  IDs of the 512 x 512
// grid 62 -> 33 ms, of the 32^3 grid 305 -> 95 ms.
#include <algorithm>
#include <vector>

#include "batched.h"
#include "gemm.h"
#include "kernels.h"
#include "select.h"

namespace hif {

namespace {

constexpr int kPb = kTsqrNb;            // steps per block
constexpr double kPqRefresh = 1e-6;     // of the squared norm
constexpr int kPqT = 1024;              // threads of the pivot choice
constexpr int kPqRegCols = 16 * kPqT;   // columns whose norms and positions fit in its registers

struct PqCtl {
  int k;      // columns factored
  int nb;     // columns chosen for the open block
  int g0;     // first column of G
  int gram;   // G is to be formed (from column k on)
  int need;   // the choice ended for want of accuracy
  int done;
  unsigned long long left;  // largest squared norm of what is left (its bits), where G is to be formed again
  double gmax;  // largest squared norm when G was formed
  double r00;
};

struct PqState {
  double* G;        // per problem, at goff: upper 64 x 64 tiles, leading dimension ld
  const int64_t* goff;
  double* d;        // [nprob][stride] squared norms, by column of G
  int32_t* pos;     // [nprob][stride] present position of column g of G, -1 once chosen
  double* Rc;       // [nprob][kPb][stride] Cholesky rows of the open block
  int32_t* key;     // [nprob][stride] original column of column g of G (k_pq_select_wide only)
  int32_t* cp;      // [nprob][stride] original column at each position
  int32_t* sw;      // [nprob][4 kPb + 1] dst, src, count of the block's moves
  double* alpha;    // [nprob][stride] R_ii
  PqCtl* ctl;
  int32_t *j0v, *jbv;
  int64_t stride;
};

__global__ __launch_bounds__(256) void k_pq_init(IdArgs A, PqState S) {
  const int q = blockIdx.y;
  const int n = A.cols[q];
  for (int c = blockIdx.x * 256 + threadIdx.x; c < n; c += gridDim.x * 256) S.cp[q * S.stride + c] = c;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    PqCtl c{};
    c.gram = 1;
    S.ctl[q] = c;
    S.jbv[q] = 0;
  }
}

// The largest norm of the trailing columns of problems whose G is to be formed
// again: 64 columns a workgroup, the rows over its waves.  Where it is within the
// tolerance nothing is left to choose, and one pass over the block has saved the
// Gram matrix, which costs all its columns' products (one 4096 x 4096 problem of
// rank 8: 4.7 ms where it is formed for that, 2.8 so).  16 waves: with 4 the
// chain of a wave's rows slowed the factorizations by 1%.
__global__ __launch_bounds__(1024) void k_pq_left(IdArgs A, PqState S) {
  constexpr int NW = 16;
  const int q = blockIdx.y;
  PqCtl* C = S.ctl + q;
  if (C->done || !C->gram || C->k == 0) return;
  const int n = A.cols[q], m = A.rows[q], ld = A.ld[q], c0 = C->k + int(blockIdx.x) * 64;
  if (c0 >= n) return;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const double* Z = A.base + A.moff[q] + min(c0 + lane, n - 1);
  double s0 = 0.0;
  for (int r = C->k + wv; r < m; r += 8 * NW) {
    double y[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) y[u] = Z[int64_t(min(r + NW * u, m - 1)) * ld];
#pragma unroll
    for (int u = 0; u < 8; ++u) s0 = r + NW * u < m ? fma(y[u], y[u], s0) : s0;
  }
  __shared__ double part[NW][64];
  part[wv][lane] = s0;
  __syncthreads();
  if (wv) return;
  double t = 0.0;
#pragma unroll
  for (int w = 0; w < NW; ++w) t += part[w][lane];
  const double mx = wave_max(fmax(t, 0.0));  // a column of NaN is never chosen
  if (lane == 0) atomicMax(&C->left, static_cast<unsigned long long>(__double_as_longlong(mx)));
}
// Such a problem is done if no pivot can pass the rank rule any more (the norms
// are good to far better than the margin).
__global__ void k_pq_end(IdArgs A, PqState S) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= A.nprob) return;
  PqCtl* C = S.ctl + q;
  if (C->done || !C->gram || C->k == 0) return;
  if (sqrt(__longlong_as_double((long long)C->left)) <= A.tol[q] * C->r00 * (1.0 - 1e-10)) {
    C->done = 1;
    A.rank[q] = C->k;
  }
}

// Tile (ta, tb), ta <= tb, of G: formed from the trailing block, or brought up
// to date with the last block's Cholesky rows.
__global__ __launch_bounds__(256) void k_pq_gram(IdArgs A, PqState S) {
  const int q = blockIdx.z, ta = blockIdx.y, tb = blockIdx.x;
  if (ta > tb) return;
  const PqCtl C = S.ctl[q];
  if (C.done) return;
  const int g0 = C.gram ? C.k : C.g0, ng = A.cols[q] - g0;
  const int a0 = ta * 64, b0 = tb * 64;
  if (b0 >= ng) return;
  const int ld = A.ld[q];
  double* G = S.G + S.goff[q] + int64_t(a0) * ld + b0;
  const int Mt = min(64, ng - a0), Nt = min(64, ng - b0);
  __shared__ double lds[kGemmLds];
  if (C.gram) {
    const double* Z = A.base + A.moff[q] + int64_t(g0) * ld + g0;
    wg_gemm(Mt, Nt, A.rows[q] - g0, 1.0, Z + a0, ld, true, Z + b0, ld, false, 0.0, G, ld, lds);
  } else if (C.nb > 0) {
    const double* R = S.Rc + q * kPb * S.stride;
    wg_gemm(Mt, Nt, C.nb, -1.0, R + a0, int(S.stride), true, R + b0, int(S.stride), false, 1.0, G, ld, lds);
  }
}

// The moves that bring the nb chosen columns to the front, and what the block's
// other kernels read; the first wave of the pivot choice.
__device__ __forceinline__ void pq_close(const PqState& S, int q, int k, int n, int nb, int g0, int need, double gmax,
                                         const int* s_swap) {
  const int lane = threadIdx.x & 63;
  PqCtl* C = S.ctl + q;
  int32_t* sw = S.sw + q * (4 * kPb + 1);
  __shared__ int s_dst[2 * kPb], s_src[2 * kPb], s_na;
  compose_swaps(s_swap, k, nb, n, s_dst, s_src, &s_na);
  __builtin_amdgcn_wave_barrier();
  if (lane < 2 * kPb && lane < s_na) {
    sw[lane] = s_dst[lane];
    sw[2 * kPb + lane] = s_src[lane];
  }
  if (lane == 0) {
    sw[4 * kPb] = s_na;
    C->nb = nb;
    C->g0 = g0;
    C->gram = 0;
    C->need = need;
    C->gmax = gmax;
    S.j0v[q] = k;
    S.jbv[q] = nb;
  }
}

// The pivots of the next block of problem blockIdx.x.  Thread t owns columns
// t + 1024 u of G (u < U): their squared norms and positions and, with U = 1,
// their Cholesky rows in registers (in memory otherwise).  One barrier a step:
// each wave publishes its best column with its Cholesky entries.  Bound by the
// chain of a step (search, row of G from memory, dot product with the chosen
// column's entries): 3.3 us with U = 1, 17 us with U = 4 (3298 columns).
template <int U>
__global__ __launch_bounds__(kPqT) void k_pq_select(IdArgs A, PqState S) {
  constexpr int NW = kPqT / 64;
  const int q = blockIdx.x;
  const PqCtl* C = S.ctl + q;
  if (C->done) {
    if (threadIdx.x == 0) S.jbv[q] = 0;
    return;
  }
  const int n = A.cols[q], m = A.rows[q], ld = A.ld[q];
  const int k = C->k, fresh = C->gram;
  const int g0 = fresh ? k : C->g0, ng = n - g0;
  const double tol = A.tol[q], r00 = C->r00;
  const int nmax = min(kPb, min(m, n) - k);
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const double* G = S.G + S.goff[q];
  double* dq = S.d + q * S.stride;
  int32_t* posq = S.pos + q * S.stride;
  double* Rc = S.Rc + q * kPb * S.stride;
  __shared__ double s_val[2][NW];
  __shared__ int s_key[2][NW], s_g[2][NW], s_pos[2][NW], s_occ[kPb], s_swap[kPb];
  alignas(16) __shared__ double s_r[2][NW][kPb];
  double d[U];
  int pos[U], key[U];  // key: the original column (ties go to the lowest)
  double r[U == 1 ? kPb : 1];
#pragma unroll
  for (int l = 0; l < (U == 1 ? kPb : 1); ++l) r[l] = 0.0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int g = tid + u * kPqT;
    d[u] = -1.0;
    pos[u] = -1;
    key[u] = INT_MAX;
    if (g < ng) {
      pos[u] = fresh ? g0 + g : posq[g];
      if (pos[u] >= 0) {
        d[u] = fresh ? G[int64_t(g) * ld + g] : dq[g];
        key[u] = S.cp[q * S.stride + pos[u]];
        if (pos[u] < k + kPb) s_occ[pos[u] - k] = g;
      }
    }
  }
  double gmax = C->gmax;
  int nb = 0, need = 0;
  for (int i = 0; i < nmax; ++i) {
    const int b = i & 1;
    double bv = -1.0;
    int bk = INT_MAX, bu = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const double v = pos[u] >= 0 ? fmax(d[u], -1.0) : -1.0;  // NaN is never chosen
      if (v > bv || (v == bv && pos[u] >= 0 && key[u] < bk)) {
        bv = v;
        bk = pos[u] >= 0 ? key[u] : INT_MAX;
        bu = u;
      }
    }
    const double wm = wave_max(bv);
    const int wk = wave_min(bv == wm ? bk : INT_MAX);
    if (bv == wm && bk == wk && (wk != INT_MAX || lane == 0)) {
      const int g = tid + bu * kPqT;
      s_val[b][wv] = wk == INT_MAX ? -1.0 : wm;
      s_key[b][wv] = wk;
      s_g[b][wv] = g;
      int p = pos[0];
#pragma unroll
      for (int u = 1; u < U; ++u) p = bu == u ? pos[u] : p;
      s_pos[b][wv] = p;
      if constexpr (U == 1) {
#pragma unroll
        for (int l = 0; l < kPb; l += 2) *reinterpret_cast<double2*>(&s_r[b][wv][l]) = double2{r[l], r[l + 1]};
      } else {
#pragma unroll 8
        for (int l = 0; l < i; ++l) s_r[b][wv][l] = Rc[l * S.stride + g];
      }
    }
    __syncthreads();
    const double wvl = s_val[b][lane & (NW - 1)];
    const int wkl = s_key[b][lane & (NW - 1)];
    const double dp = group_max<NW>(wvl);
    const int kp = group_min<NW>(wvl == dp ? wkl : INT_MAX);
    if (i == 0 && fresh) gmax = dp;
    const bool first = i == 0 && fresh;
    if (!(dp > 0.0) || (!first && dp <= kPqRefresh * gmax)) {
      need = !first;  // at the limit of G's accuracy: form it again
      break;
    }
    if (sqrt(dp) <= 0.5 * tol * r00) break;  // past the rank
    const int w = __ffsll(__ballot(wvl == dp && wkl == kp)) - 1;
    const int p = s_g[b][w], ppos = s_pos[b][w];
    const int other = s_occ[i];  // trades places with the chosen column
    const double inv = 1.0 / sqrt(dp);
    const int pt = p >> 6;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int g = tid + u * kPqT;
      if (U > 1 && u * kPqT >= ng) break;
      const int gc = g < ng ? g : 0;
      // upper tiles: entry (a, b) is stored where a / 64 <= b / 64
      double x = (gc >> 6) >= pt ? G[int64_t(p) * ld + gc] : G[int64_t(gc) * ld + p];
      if constexpr (U == 1) {
        double x2 = 0.0;
#pragma unroll
        for (int l = 0; l < kPb; l += 2) {  // entries past the step are zero
          const double2 t = *reinterpret_cast<const double2*>(&s_r[b][w][l]);
          x -= r[l] * t.x;
          x2 -= r[l + 1] * t.y;
        }
        x = (x + x2) * inv;
#pragma unroll
        for (int l = 0; l < kPb; ++l) r[l] = l == i ? x : r[l];
      } else {
#pragma unroll 8
        for (int l = 0; l < i; ++l) x -= Rc[l * S.stride + gc] * s_r[b][w][l];
        x *= inv;
      }
      if (g < ng) {
        Rc[i * S.stride + g] = x;
        d[u] = fmax(d[u] - x * x, 0.0);
        if (g == p) {
          pos[u] = -1;
        } else if (g == other) {
          pos[u] = ppos;
          if (ppos < k + kPb) s_occ[ppos - k] = g;
        }
      }
    }
    if (tid == 0) s_swap[i] = ppos;
    nb = i + 1;
    // the slots of this parity are written again two steps on, past the next
    // step's barrier, which follows every read above
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int g = tid + u * kPqT;
    if (g < ng) {
      dq[g] = d[u];
      posq[g] = pos[u];
    }
  }
  __syncthreads();
  if (wv == 0) pq_close(S, q, k, n, nb, g0, need, gmax, s_swap);
}

// The same choice for any number of columns, their norms, positions and Cholesky
// rows in memory: one pass over them a step, which also finds the best column of
// the next step.
__global__ __launch_bounds__(kPqT) void k_pq_select_wide(IdArgs A, PqState S) {
  constexpr int NW = kPqT / 64;
  const int q = blockIdx.x;
  const PqCtl* C = S.ctl + q;
  if (C->done) {
    if (threadIdx.x == 0) S.jbv[q] = 0;
    return;
  }
  const int n = A.cols[q], m = A.rows[q], ld = A.ld[q];
  const int k = C->k, fresh = C->gram;
  const int g0 = fresh ? k : C->g0, ng = n - g0;
  const double tol = A.tol[q], r00 = C->r00;
  const int nmax = min(kPb, min(m, n) - k);
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const double* G = S.G + S.goff[q];
  double* dq = S.d + q * S.stride;
  int32_t *posq = S.pos + q * S.stride, *keyq = S.key + q * S.stride;
  double* Rc = S.Rc + q * kPb * S.stride;
  __shared__ double s_val[2][NW], s_r[2][NW][kPb];
  __shared__ int s_key[2][NW], s_g[2][NW], s_pos[2][NW], s_occ[kPb], s_swap[kPb];
  double bv = -1.0;  // this thread's best column
  int bk = INT_MAX, bg = 0, bp = -1;
  auto offer = [&](double d, int key, int g, int pos) {
    const double v = fmax(d, -1.0);  // NaN is never chosen
    if (v > bv || (v == bv && key < bk)) {
      bv = v;
      bk = key;
      bg = g;
      bp = pos;
    }
  };
  for (int g = tid; g < ng; g += kPqT) {
    const int pos = fresh ? g0 + g : posq[g];
    if (fresh) posq[g] = pos;
    if (pos < 0) continue;
    const double d = fresh ? G[int64_t(g) * ld + g] : dq[g];
    const int key = S.cp[q * S.stride + pos];
    dq[g] = d;
    keyq[g] = key;
    if (pos < k + kPb) s_occ[pos - k] = g;
    offer(d, key, g, pos);
  }
  double gmax = C->gmax;
  int nb = 0, need = 0;
  for (int i = 0; i < nmax; ++i) {
    const int b = i & 1;
    const double wm = wave_max(bv);
    const int wk = wave_min(bv == wm ? bk : INT_MAX);
    if (bv == wm && bk == wk && (wk != INT_MAX || lane == 0)) {
      s_val[b][wv] = wk == INT_MAX ? -1.0 : wm;
      s_key[b][wv] = wk;
      s_g[b][wv] = bg;
      s_pos[b][wv] = bp;
#pragma unroll 8
      for (int l = 0; l < i; ++l) s_r[b][wv][l] = Rc[l * S.stride + bg];
    }
    __syncthreads();
    const double wvl = s_val[b][lane & (NW - 1)];
    const int wkl = s_key[b][lane & (NW - 1)];
    const double dp = group_max<NW>(wvl);
    const int kp = group_min<NW>(wvl == dp ? wkl : INT_MAX);
    const bool first = i == 0 && fresh;
    if (first) gmax = dp;
    if (!(dp > 0.0) || (!first && dp <= kPqRefresh * gmax)) {
      need = !first;
      break;
    }
    if (sqrt(dp) <= 0.5 * tol * r00) break;
    const int w = __ffsll(__ballot(wvl == dp && wkl == kp)) - 1;
    const int p = s_g[b][w], ppos = s_pos[b][w], other = s_occ[i], pt = p >> 6;
    const double inv = 1.0 / sqrt(dp);
    bv = -1.0;
    bk = INT_MAX;
    for (int g = tid; g < ng; g += kPqT) {
      double x = (g >> 6) >= pt ? G[int64_t(p) * ld + g] : G[int64_t(g) * ld + p];
#pragma unroll 8
      for (int l = 0; l < i; ++l) x -= Rc[l * S.stride + g] * s_r[b][w][l];
      x *= inv;
      Rc[i * S.stride + g] = x;
      int pos = posq[g];
      if (g == p) {
        pos = posq[g] = -1;
      } else if (g == other) {
        pos = posq[g] = ppos;
        if (ppos < k + kPb) s_occ[ppos - k] = g;
      }
      if (pos < 0) continue;
      const double d = fmax(dq[g] - x * x, 0.0);
      dq[g] = d;
      offer(d, keyq[g], g, pos);
    }
    if (tid == 0) s_swap[i] = ppos;
    nb = i + 1;
  }
  __syncthreads();
  if (wv == 0) pq_close(S, q, k, n, nb, g0, need, gmax, s_swap);
}

// Moves the chosen columns to the front of the trailing ones, in all rows: a
// wave takes 8 rows, lane e the e-th of the (at most 64) moved columns.
__global__ __launch_bounds__(256) void k_pq_swap(IdArgs A, PqState S) {
  const int q = blockIdx.y;
  if (S.jbv[q] <= 0) return;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int m = A.rows[q], r0 = (int(blockIdx.x) * 4 + wv) * 8;
  const int32_t* sw = S.sw + q * (4 * kPb + 1);
  const int na = sw[4 * kPb];
  const bool on = lane < na;
  const int dst = on ? sw[lane] : 0, src = on ? sw[2 * kPb + lane] : 0;
  if (blockIdx.x == 0 && wv == 0 && on) {
    int32_t* cp = S.cp + q * S.stride;
    const int c = cp[src];
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): all lanes read before any writes
    cp[dst] = c;
  }
  if (r0 >= m) return;
  const int ld = A.ld[q];
  double* Z = A.base + A.moff[q];
  double v[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) v[u] = Z[int64_t(min(r0 + u, m - 1)) * ld + src];
  __builtin_amdgcn_s_waitcnt(0x0f70);
#pragma unroll
  for (int u = 0; u < 8; ++u)
    if (on && dst != src && r0 + u < m) Z[int64_t(r0 + u) * ld + dst] = v[u];
}

// The rank rule on the factored panel's R_ii, and what comes next.
__global__ __launch_bounds__(64) void k_pq_rank(IdArgs A, PqState S) {
  const int q = blockIdx.x, lane = threadIdx.x;
  PqCtl* C = S.ctl + q;
  if (C->done) return;
  const int n = A.cols[q], m = A.rows[q], k = C->k, nb = C->nb, ld = A.ld[q];
  const double* Z = A.base + A.moff[q];
  double x = 0.0;
  if (lane < nb) {
    x = Z[int64_t(k + lane) * ld + k + lane];
    S.alpha[q * S.stride + k + lane] = x;
  }
  const double r00 = k > 0 ? C->r00 : fabs(__shfl(x, 0, 64));
  const double ax = fabs(x);
  const unsigned long long bad = __ballot(lane < nb && !(ax > 0.0 && ax > A.tol[q] * r00));
  if (lane == 0) {
    int kn = k + nb, done = 0;
    if (bad) {
      kn = k + __ffsll(bad) - 1;
      done = 1;
    } else if (kn >= min(m, n) || (nb < kPb && !C->need)) {
      done = 1;  // nothing left, or nothing left above the tolerance
    }
    C->k = kn;
    C->r00 = r00;
    C->done = done;
    C->gram = !done && C->need;
    C->left = 0;
    if (done) A.rank[q] = kn;
  }
}

// perm (the pivots in order, then the redundant columns ascending) and the
// position of every original column.
__global__ __launch_bounds__(1024) void k_pq_perm(IdArgs A, PqState S) {
  const int q = blockIdx.x;
  const int n = A.cols[q], k = A.rank[q];
  const int32_t* cp = S.cp + q * S.stride;
  int32_t* pos = S.pos + q * S.stride;
  int32_t* perm = A.perm + A.poff[q];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  __shared__ int s_cnt[16];
  for (int c = tid; c < n; c += 1024) {
    const int o = cp[c];
    pos[o] = c;
    if (c < k) perm[c] = o;
  }
  __syncthreads();
  int base = k;
  for (int c0 = 0; c0 < n; c0 += 1024) {
    const int c = c0 + tid;
    const bool red = c < n && pos[c] >= k;
    const unsigned long long bal = __ballot(red);
    if (lane == 0) s_cnt[wv] = __popcll(bal);
    __syncthreads();
    int off = base, tot = 0;
    for (int w = 0; w < 16; ++w) {
      if (w < wv) off += s_cnt[w];
      tot += s_cnt[w];
    }
    if (red) perm[off + __popcll(bal & ((1ull << lane) - 1ull))] = c;
    base += tot;
    __syncthreads();
  }
}

// Problems into the working copy: rows from column c / 16 line-aligned.
__global__ __launch_bounds__(256) void k_pq_copy(IdArgs src, IdArgs dst) {
  const int q = blockIdx.y;
  const int n = src.cols[q], rows = src.rows[q];
  const double* S0 = src.base + src.moff[q];
  double* D0 = dst.base + dst.moff[q];
  const int lds = src.ld[q], ldd = dst.ld[q];
  for (int r = blockIdx.x * 8; r < min(rows, int(blockIdx.x) * 8 + 8); ++r)
    for (int c = threadIdx.x; c < n; c += 256) D0[int64_t(r) * ldd + c] = S0[int64_t(r) * lds + c];
}

// Rows 0..rank-1 back, every column to its original place.
__global__ __launch_bounds__(256) void k_pq_out(IdArgs src, IdArgs dst, PqState S) {
  const int q = blockIdx.y;
  const int n = src.cols[q], rows = dst.rank[q];
  const double* S0 = src.base + src.moff[q];
  double* D0 = dst.base + dst.moff[q];
  const int32_t* pos = S.pos + q * S.stride;
  const int lds = src.ld[q], ldd = dst.ld[q];
  for (int r = blockIdx.x * 8; r < min(rows, int(blockIdx.x) * 8 + 8); ++r)
    for (int c = threadIdx.x; c < n; c += 256) D0[int64_t(r) * ldd + c] = S0[int64_t(r) * lds + pos[c]];
}

__global__ void k_pq_iota(int32_t* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = i;
}

}  // namespace

// All problems of A0 together.  Every allocation comes before the first output.
static void id_blocked(const IdArgs& A0, int max_rows, int max_cols, hipStream_t s) {
  // The problems move to a copy whose rows start on 128-byte lines (row stride
  // padded to 16 doubles); only rows 0..k-1 (R11 and T) are copied back.
  const int np = A0.nprob;
  std::vector<int32_t> hr(np), hcl(np);
  HIF_HIP(hipMemcpyAsync(hr.data(), A0.rows, sizeof(int32_t) * np, hipMemcpyDeviceToHost, s));
  HIF_HIP(hipMemcpyAsync(hcl.data(), A0.cols, sizeof(int32_t) * np, hipMemcpyDeviceToHost, s));
  HIF_HIP(hipStreamSynchronize(s));
  // Problems with more rows than columns and than the row compression's tree
  // takes: the R factor has the same ID.  What is then left to the panels of the
  // pivoted QR has at most kTsqrPanelRows rows.
  const bool tall = max_rows > kTsqrMaxRows;
  std::vector<int64_t> off(size_t(5) * np);   // offsets of Z, G, the panels' and the tall problems' scratch, and zeros
  std::vector<int32_t> num(size_t(2) * np);   // leading dimensions and rows
  int64_t zt = 0, gt = 0, st = 0, qt = 0;
  for (int q = 0; q < np; ++q) {
    const int ld = (hcl[q] + 15) & ~15, rows = tall ? std::min(hr[q], hcl[q]) : hr[q];
    num[q] = ld;
    num[np + q] = rows;
    off[q] = zt;
    off[np + q] = gt;
    off[2 * np + q] = st;
    off[3 * np + q] = qt;
    off[4 * np + q] = 0;
    if (tall && hr[q] > hcl[q]) qt += rowqr_scratch(hr[q], hcl[q]);
    zt += int64_t(hr[q]) * ld;
    gt += int64_t(hcl[q]) * ld;
    st += tsqr_layout(rows).total;
  }
  IdArgs A = A0;
  DBuf<double> Z, Gm, scratch, vec, qr;
  DBuf<int64_t> doff;
  DBuf<int32_t> dnum, ints;
  DBuf<PqCtl> ctl;
  Z.alloc(zt + 16, nullptr);
  doff.alloc(off.size(), nullptr);
  dnum.alloc(num.size(), nullptr);
  HIF_HIP(hipMemcpyAsync(doff.p, off.data(), sizeof(int64_t) * off.size(), hipMemcpyHostToDevice, s));
  HIF_HIP(hipMemcpyAsync(dnum.p, num.data(), sizeof(int32_t) * num.size(), hipMemcpyHostToDevice, s));
  A.base = Z.p;
  A.moff = doff.p;
  A.ld = dnum.p;
  hipLaunchKernelGGL(k_pq_copy, dim3(unsigned((max_rows + 7) / 8), unsigned(np)), dim3(256), 0, s, A0, A);
  A.rows = dnum.p + np;
  if (tall) {
    if (rowqr_split_fits(max_rows, max_cols)) {
      launch_rowqr_split(Z.p, std::vector<int64_t>(off.begin(), off.begin() + np),
                         std::vector<int32_t>(num.begin(), num.begin() + np), hr, hcl, nullptr, s);
    } else if (qt > 0) {  // over 16384 columns
      qr.alloc(qt, nullptr);
      QrBatch T{};
      T.base = Z.p;
      T.moff = A.moff;
      T.ld = A.ld;
      T.rows = A0.rows;
      T.cols = A.cols;
      T.scratch = qr.p;
      T.soff = doff.p + 3 * np;
      T.nprob = np;
      launch_qr_batched(T, max_rows, max_cols, s);
    }
    max_rows = *std::max_element(num.begin() + np, num.end());
  }
  HIF_REQUIRE(max_rows <= kTsqrPanelRows, HIF_EUNSUPPORTED, "ID problem with more than 65536 rows and columns");
  const int64_t stride = (max_cols + 15) & ~15, tot = stride * np;
  Gm.alloc(gt + 16, nullptr);
  scratch.alloc(st + 1, nullptr);
  vec.alloc(size_t(tot) * (kPb + 2), nullptr);
  ints.alloc(size_t(tot) * 3 + size_t(np) * (4 * kPb + 3), nullptr);
  ctl.alloc(np, nullptr);
  PqState S{};
  S.G = Gm.p;
  S.goff = doff.p + np;
  S.d = vec.p;
  S.alpha = vec.p + tot;
  S.Rc = vec.p + 2 * tot;
  S.pos = ints.p;
  S.cp = ints.p + tot;
  S.key = ints.p + 2 * tot;
  S.sw = ints.p + 3 * tot;
  S.j0v = S.sw + size_t(np) * (4 * kPb + 1);
  S.jbv = S.j0v + np;
  S.ctl = ctl.p;
  S.stride = stride;
  QrBatch Q{};
  Q.base = Z.p;
  Q.moff = A.moff;
  Q.ld = A.ld;
  Q.rows = A.rows;
  Q.cols = A.cols;
  Q.scratch = scratch.p;
  Q.soff = doff.p + 2 * np;
  Q.nprob = np;
  Q.j0v = S.j0v;
  Q.jbv = S.jbv;
  const unsigned up = unsigned(np);
  hipLaunchKernelGGL(k_pq_init, dim3(unsigned((max_cols + 255) / 256), up), dim3(256), 0, s, A, S);
  std::vector<PqCtl> hc(np);
  int kmin = 0, gcols = max_cols, trail = max_cols;  // what is left of the widest problem
  bool all = false, again = false;  // again: a Gram matrix is to be formed once more
  // a block takes a step of each unfinished problem, or the next one does
  for (int blk = 0; blk <= 2 * max_cols + 2 && !all; ++blk) {
    if (again) {
      hipLaunchKernelGGL(k_pq_left, dim3(unsigned((trail + 63) / 64), up), dim3(1024), 0, s, A, S);
      hipLaunchKernelGGL(k_pq_end, dim3(unsigned((np + 63) / 64)), dim3(64), 0, s, A, S);
    }
    const unsigned gt64 = unsigned((gcols + 63) / 64);
    hipLaunchKernelGGL(k_pq_gram, dim3(gt64, gt64, up), dim3(256), 0, s, A, S);
    if (max_cols <= kPqT)
      hipLaunchKernelGGL(k_pq_select<1>, dim3(up), dim3(kPqT), 0, s, A, S);
    else if (max_cols <= 4 * kPqT)
      hipLaunchKernelGGL(k_pq_select<4>, dim3(up), dim3(kPqT), 0, s, A, S);
    else if (max_cols <= kPqRegCols)
      hipLaunchKernelGGL(k_pq_select<16>, dim3(up), dim3(kPqT), 0, s, A, S);
    else
      hipLaunchKernelGGL(k_pq_select_wide, dim3(up), dim3(kPqT), 0, s, A, S);
    hipLaunchKernelGGL(k_pq_swap, dim3(unsigned((max_rows + 31) / 32), up), dim3(256), 0, s, A, S);
    launch_tsqr_panel(Q, std::max(1, max_rows - kmin), trail, s);
    hipLaunchKernelGGL(k_pq_rank, dim3(up), dim3(64), 0, s, A, S);
    HIF_HIP(hipMemcpyAsync(hc.data(), ctl.p, sizeof(PqCtl) * np, hipMemcpyDeviceToHost, s));
    HIF_HIP(hipStreamSynchronize(s));
    all = true;
    again = false;
    kmin = max_cols;
    gcols = trail = 1;
    for (int q = 0; q < np; ++q) {
      if (hc[q].done) continue;
      all = false;
      again = again || (hc[q].gram && hc[q].k > 0);
      kmin = std::min(kmin, hc[q].k);
      gcols = std::max(gcols, hcl[q] - (hc[q].gram ? hc[q].k : hc[q].g0));
      trail = std::max(trail, hcl[q] - hc[q].k);
    }
  }
  if (!all) throw Error{HIF_EDEVICE, "blocked pivoted QR did not finish"};
  hipLaunchKernelGGL(k_pq_perm, dim3(up), dim3(1024), 0, s, A, S);
  int kmax = 0;
  for (const PqCtl& c : hc) kmax = std::max(kmax, c.k);
  // T on the permuted copy, whose columns are in place already
  IdArgs AT = A;
  hipLaunchKernelGGL(k_pq_iota, dim3(unsigned((max_cols + 255) / 256)), dim3(256), 0, s, S.cp, max_cols);
  AT.perm = S.cp;
  AT.poff = doff.p + 4 * np;
  launch_id_T(AT, S.alpha, stride, kmax, max_cols, s);
  hipLaunchKernelGGL(k_pq_out, dim3(unsigned((kmax + 7) / 8 + 1), up), dim3(256), 0, s, A, A0, S);
  launch_id_Tcopy(A0, max_cols, s);
  HIF_HIP(hipGetLastError());
  HIF_HIP(hipStreamSynchronize(s));  // the working copy is released on return
}

void launch_id_blocked(const IdArgs& A, int max_rows, int max_cols, hipStream_t s) {
  if (A.nprob == 0) return;
  // A Gram matrix takes n x n doubles beside the copy of the problem: where the
  // device does not hold those of all problems, half of them at a time.
  try {
    id_blocked(A, max_rows, max_cols, s);
    return;
  } catch (const Error& e) {
    if (e.status != HIF_ENOMEM || A.nprob == 1) throw;
  }
  const int h = A.nprob / 2;
  for (int q0 : {0, h}) {
    IdArgs P = A;
    P.moff += q0;
    P.ld += q0;
    P.rows += q0;
    P.cols += q0;
    P.tol += q0;
    P.rank += q0;
    P.poff += q0;
    if (P.toff) P.toff += q0;
    P.nprob = q0 ? A.nprob - h : h;
    launch_id_blocked(P, max_rows, max_cols, s);
  }
}

bool id_blocked_fits(int nprob, int max_rows, int max_cols) {
  // many small problems go to the one-workgroup ID after row compression
  (void)max_rows;
  return nprob <= 512 && max_cols >= 128;
}

}  // namespace hif
