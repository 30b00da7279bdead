// Per-panel batched kernels (batched.hip) for sub-levels with few large
// problems.  Internal, not part of the ABI.
#pragma once

#include <vector>

#include "kernels.h"

namespace hif {

// Row compression problems (same fields as RowQrArgs).
using QrBatch = RowQrArgs;
// Few large problems: max_rows/max_cols bound rows/cols over the batch.
void launch_qr_batched(const QrBatch& A, int max_rows, int max_cols, hipStream_t s);

// Row compression of problems taller than one TSQR stack holds (more than
// kTsqrSplitRows rows), from host copies of the problems' offsets (from
// base), leading dimensions, rows and columns: each is cut into row blocks
// factored as problems of their own, whose R factors are stacked and factored
// again.  Leaves R0 in the leading n x n block of every problem with m > n,
// as launch_qr_batched does.
// Blocks have at least half kTsqrSplitRows rows, and at least twice the
// columns for up to 16384 columns, so each round shrinks the stack.
constexpr int kTsqrSplitRows = 32768;
inline bool rowqr_split_fits(int max_rows, int max_cols) {
  return max_rows > kTsqrSplitRows && max_cols <= kTsqrSplitRows / 2;
}
void launch_rowqr_split(double* base, const std::vector<int64_t>& moff, const std::vector<int32_t>& ld,
                        const std::vector<int32_t>& rows, const std::vector<int32_t>& cols, MemTracker* mt,
                        hipStream_t s);

// Householder reflectors of the row compression: a column whose squared norm is
// below this is taken as zero.  2 / v^T v (and T, about that of two reflectors)
// of a smaller one leaves the range of a double, and the block becomes NaN.  Such
// columns arise from ordinary data: a chunk of a panel with fewer nonzero rows
// than columns is left with rounding errors, then with the rounding errors of
// these, 16 digits lower at every turn.
constexpr double kReflectorMin = 0x1p-1000;

// Communication-avoiding panels of the row compression (tsqr.hip): panel
// width, rows per chunk, chunk factors per group, the tallest problem, and the
// tallest panel its three tree levels take.
constexpr int kTsqrNb = 32;
constexpr int kTsqrRows = 256;
constexpr int kTsqrFan = 16;
constexpr int kTsqrMaxRows = 32768;
constexpr int kTsqrPanelRows = kTsqrRows * kTsqrFan * kTsqrFan;
static_assert(kTsqrMaxRows <= kTsqrPanelRows, "three tree levels");
__host__ __device__ inline int tsqr_chunks(int mp) { return (mp + kTsqrRows - 1) / kTsqrRows; }
__host__ __device__ inline int tsqr_groups(int nck) { return (nck + kTsqrFan - 1) / kTsqrFan; }
// Problems of at most kTsqrMaxRows rows.
void launch_tsqr(const QrBatch& A, int max_rows, int max_cols, hipStream_t s);
// One panel of every problem, from A.j0v and A.jbv, and its update of all
// columns right of it (at most max_trail of any problem).
void launch_tsqr_panel(const QrBatch& A, int max_rows, int max_trail, hipStream_t s);
// Scratch of one problem with m rows (doubles): V of the chunks (m x nb) | T
// per chunk | stacked chunk R, replaced by V of the groups | T per group |
// with several groups, their stacked R, replaced by V of the root, and its T.
struct TsqrLayout {
  int64_t V, Tc, S, T1, S2, T2, total;
};
__host__ __device__ inline TsqrLayout tsqr_layout(int m) {
  const int64_t nm = tsqr_chunks(m), ng = tsqr_groups(int(nm)), b2 = int64_t(kTsqrNb) * kTsqrNb;
  TsqrLayout L;
  L.V = 0;
  L.Tc = int64_t(m) * kTsqrNb;
  L.S = L.Tc + nm * b2;
  L.T1 = L.S + nm * b2;
  L.S2 = L.T1 + ng * b2;
  L.T2 = L.S2 + (ng > 1 ? ng * b2 : 0);
  L.total = L.T2 + (ng > 1 ? b2 : 0);
  return L;
}
// Scratch doubles every row-compression path needs for an m x n problem
// (m > n); the TSQR panels alternate between two copies of the layout.
inline int64_t rowqr_scratch(int64_t m, int64_t n) {
  const int64_t fused = m * 16 + 16 * n + 256;
  const int64_t tsqr = 2 * tsqr_layout(int(m)).total;
  return fused > tsqr ? fused : tsqr;
}

// Partial LU problems: n x n row-major blocks (leading dimension n) factored
// over their first r columns with pivots among rows < r.
struct LuBatch {
  double* base;
  const int64_t* moff;
  const int32_t* n;
  const int32_t* r;
  int32_t* piv;           // pivots of problem q at piv + poff[q]
  const int64_t* poff;
  int32_t* status;
  int nprob = 0;
  int fp32 = 0;  // mixed precision: trailing tiles inside the skeleton block on FP32 matrix cores
};
void launch_lu_batched(const LuBatch& A, int max_r, int max_n, hipStream_t s);

// One entry of a batched GEMM: C = beta C + alpha op(A) op(B).
struct GemmDesc {
  int M, N, K;
  int ta, tb;
  int lda, ldb, ldc;
  double alpha, beta;
  const double* A;
  const double* B;
  double* C;
  int fp32 = 0;  // mixed precision: FP32 matrix cores, FP32 accumulation
};
void launch_gemm_tiles(const GemmDesc* D, int nd, int max_m, int max_n, hipStream_t s);

}  // namespace hif
