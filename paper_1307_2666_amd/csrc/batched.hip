// Batched kernels for the coarse sub-levels, where a few large problems would
// leave most compute units idle if each ran in one workgroup: the dispatch of
// the row compression before the ID (the tree of tsqr.hip; above 32768 rows row
// blocks, or panels of 16 columns by one workgroup per problem with a
// trailing-update kernel of one workgroup per 64 columns), and general products
// by 64 x 64 tiles.  The updates run on the matrix cores (v_mfma_f64_16x16x4f64)
// with operands read straight from device memory in the instruction's lane layout.
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
    const bool live = ss >= kReflectorMin;
    const double alpha = live ? -copysign(nrm, x0) : 0.0;
    const double v0 = x0 - alpha;
    const double vtv = ss - x0 * x0 + v0 * v0;
    const double beta = live ? 2.0 / vtv : 0.0;
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

void launch_gemm_tiles(const GemmDesc* D, int nd, int max_m, int max_n, hipStream_t s) {
  if (nd == 0 || max_m <= 0 || max_n <= 0) return;
  const unsigned tx = unsigned((max_n + kGemmTile - 1) / kGemmTile), ty = unsigned((max_m + kGemmTile - 1) / kGemmTile);
  hipLaunchKernelGGL(k_gemm_tiles, dim3(tx, ty, nd), dim3(256), 0, s, D, nd);
  HIF_HIP(hipGetLastError());
}

}  // namespace hif
