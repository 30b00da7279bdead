// Row compression of the blocks the IDs run on: communication-avoiding QR
// (TSQR panels) of many problems at once.  Only R is kept.
//
// Panel j0 (columns j0..j0+jb-1, jb <= 32, rows j0..m-1) is cut into balanced
// chunks of at most 256 rows, each factored by one workgroup; the chunk R
// factors are stacked, up to 16 to a group (512 rows), and every group
// factored the same way; with more than one group (m > 4096) the groups' R
// factors are stacked and factored once more.  Every node leaves V and T of
// its compact WY form I - V T V^T.  The columns right of the panel are then
// updated chunk by chunk, and the chunks' (groups') top 32 rows with the
// upper nodes' reflectors.
#include <algorithm>
#include <map>
#include <mutex>

#include "batched.h"
#include "gemm.h"
#include "wave.h"

namespace hif {

namespace {

constexpr int kTb = kTsqrNb;
static_assert(kTb == 32, "the lane layout below holds two column groups of 16");

// The tree over the rows of one panel: nck chunks, ng groups of chunks (0
// with one chunk).
struct PanelGeom {
  int mp, jb, nck, ng;
};
// The panel of problem q: the one at the given j0 where that is a panel of its
// row compression, or the one the pivoted QR has chosen (j0 is set to its
// first column).  false: none.
__device__ __forceinline__ bool panel_geom(const QrBatch& A, int q, int& j0, PanelGeom& g) {
  const int m = A.rows[q], n = A.cols[q];
  if (A.j0v) {
    j0 = A.j0v[q];
    g.jb = A.jbv[q];
    if (g.jb <= 0) return false;
  } else {
    if (m <= n || j0 >= n) return false;
    g.jb = min(kTb, n - j0);
  }
  g.mp = m - j0;
  g.nck = tsqr_chunks(g.mp);
  g.ng = g.nck > 1 ? tsqr_groups(g.nck) : 0;
  return true;
}
__device__ __forceinline__ int part_lo(int i, int total, int parts) {
  return int(unsigned(i) * unsigned(total) / unsigned(parts));  // total <= 65536 rows, i <= parts <= 256
}

// LDS of a panel factorization by NW waves.
template <int NW>
struct FactLds {
  double red[2][NW][kTb];
  double row[2][kTb];
  double v0[kTb], beta[kTb];
  double G[kTb][kTb + 1];
  double T[kTb][kTb + 1];
  alignas(16) double col[NW][4][18];  // the pivot column, by wave and lane row
};

// Householder QR of a block of 64 NW rows and jb <= 32 columns in registers.
// Wave w holds rows 64 w .. 64 w + 63, lane (li, lk) = (lane % 16, lane / 16)
// rows 4 s + lk of columns li and 16 + li in y[s][0], y[s][1] (the layout of
// the 16x16x4 matrix instruction's operands): the products of the pivot column
// with all columns then need only two steps across the lanes, and each lane
// finds the update coefficients of its own two columns.  One barrier per
// column: every lane reads the waves' partial products and forms the reflector
// for itself.  What bounds it is that chain (column broadcast through LDS,
// products, cross-lane sum, LDS round trip, square root and division, update).
// On return rows below the diagonal hold the Householder vectors, rows < jb
// the upper triangle of R; v0 (their diagonal entries), beta = 2 / v^T v and
// the upper part of G = V^T V (zero elsewhere) are in LDS.
template <int NW>
__device__ __forceinline__ void block_qr(double (&y)[16][2], int jb, FactLds<NW>& L) {
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const bool top = wv == 0;  // the wave that holds rows 0..31
  for (int e = tid; e < kTb * (kTb + 1); e += 64 * NW) (&L.G[0][0])[e] = 0.0;
  if (tid < kTb && tid >= jb) {  // columns past a partial panel: no reflector
    L.v0[tid] = 0.0;
    L.beta[tid] = 0.0;
  }
  __syncthreads();
  // columns 4 s0 + l: their diagonal entries are in y[s0][s0 / 4] of lane row l
#pragma unroll
  for (int s0 = 0; s0 < 8; ++s0) {
    const int gj = s0 >> 2;
#pragma nounroll
    for (int l = 0; l < 4; ++l) {
      const int jj = 4 * s0 + l;
      if (jj >= jb) break;
      const int b = l & 1;
      double v[16];
      {
        double* col = L.col[wv][lk];
        if (li == (jj & 15)) {
#pragma unroll
          for (int s = 0; s < 16; s += 2) *reinterpret_cast<double2*>(col + s) = double2{y[s][gj], y[s + 1][gj]};
        }
        // the same wave reads what it wrote: no barrier, only the LDS order
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int s = 0; s < 16; s += 2) {
          const double2 t = *reinterpret_cast<const double2*>(col + s);
          v[s] = t.x;
          v[s + 1] = t.y;
        }
      }
      if (top) {  // rows <= jj are finished; row jj enters through L.row
#pragma unroll
        for (int s = 0; s < s0; ++s) v[s] = 0.0;
        v[s0] = lk <= l ? 0.0 : v[s0];
        if (lk == l) {
          L.row[b][li] = y[s0][0];
          L.row[b][16 + li] = y[s0][1];
        }
      }
      double a0 = 0.0, a1 = 0.0, b0 = 0.0, b1 = 0.0;
#pragma unroll
      for (int s = 0; s < 16; s += 2) {
        a0 += v[s] * y[s][0];
        a1 += v[s] * y[s][1];
        b0 += v[s + 1] * y[s + 1][0];
        b1 += v[s + 1] * y[s + 1][1];
      }
      double t = swap_pair_sum<16>(a0 + b0, a1 + b1);  // lanes < 32: column li, others: column 16 + li
      t = swap_pair_sum<8>(t, t);
      if ((lane & 16) == 0) L.red[b][wv][(lane >> 5) * 16 + li] = t;
      __syncthreads();
      double sj = 0.0, t0 = 0.0, t1 = 0.0;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        sj += L.red[b][w][jj];
        t0 += L.red[b][w][li];
        t1 += L.red[b][w][16 + li];
      }
      const double x0 = L.row[b][jj], r0 = L.row[b][li], r1 = L.row[b][16 + li];
      const double ss = sj + x0 * x0;
      const double nrm = sqrt(ss);
      const bool live = ss >= kReflectorMin;
      const double alpha = live ? -copysign(nrm, x0) : 0.0;
      const double v0 = x0 - alpha;
      const double vtv = sj + v0 * v0;
      const double beta = live ? 2.0 / vtv : 0.0;
      const double g0 = v0 * r0 + t0, g1 = v0 * r1 + t1;
      const double c0 = (li > jj && li < jb) ? beta * g0 : 0.0;
      const double c1 = (16 + li > jj && 16 + li < jb) ? beta * g1 : 0.0;
      if (top) v[s0] = lk == l ? v0 : v[s0];
      if (s0 < 4) {
#pragma unroll
        for (int s = 0; s < 16; ++s) y[s][0] -= c0 * v[s];
      }
#pragma unroll
      for (int s = 0; s < 16; ++s) y[s][1] -= c1 * v[s];
      if (top) {
        if (lk == l && li == (jj & 15)) y[s0][gj] = alpha;
        // column jj of G above the diagonal: column c < jj holds its reflector
        if (lk == 0 && li < jj) L.G[li][jj] = g0;
        if (lk == 1 && 16 + li < jj) L.G[16 + li][jj] = g1;
        if (lane == 0) {
          L.v0[jj] = v0;
          L.beta[jj] = beta;
        }
      }
      // L.red[b] and L.row[b] are written again two columns on, after the next
      // column's barrier, which every wave reaches past its reads above.
    }
  }
  __syncthreads();
}

// T of the compact WY form I - V T V^T (T upper triangular) from beta and the
// upper part of G = V^T V: the two diagonal 16 x 16 blocks by the recurrence
// T(p, i) = -beta_i sum_{l < i} T(p, l) G(l, i), T(i, i) = beta_i, one wave
// each (lane p keeps row p), and T12 = -T11 (G12 T22) on the matrix cores:
// half the serial chain of the recurrence over 32 columns.  All waves call it.
template <int NW>
__device__ __forceinline__ void build_T(FactLds<NW>& L, double* Tout) {
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  if (wv < 2) {
    const int o = 16 * wv;
    double trow[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const double b = L.beta[o + i];
      double acc = 0.0;
#pragma unroll
      for (int l = 0; l < i; ++l) acc += trow[l] * L.G[o + l][o + i];
      trow[i] = li == i ? b : (li < i ? -b * acc : 0.0);
    }
    if (lk == 0) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        L.T[o + li][o + i] = trow[i];
        Tout[(o + li) * kTb + o + i] = trow[i];
      }
    }
  }
  __syncthreads();
  if (wv == 0) {
    double4_t x = {0.0, 0.0, 0.0, 0.0}, d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < 4; ++s) x = mfma_f64(L.G[li][16 + 4 * s + lk], L.T[16 + 4 * s + lk][16 + li], x);
#pragma unroll
    for (int s = 0; s < 4; ++s) d = mfma_f64(L.T[li][4 * s + lk], x[s], d);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      Tout[(4 * v + lk) * kTb + 16 + li] = -d[v];
      Tout[(16 + 4 * v + lk) * kTb + li] = 0.0;
    }
  }
}

// Node x of tree level LEVEL (0: chunks of the panel, 1: groups of stacked
// chunk factors, 2: the stacked group factors): factors its rows, leaves V
// and T, and R in the next level's stack or, at the root, in the block.
// V of levels 1 and 2 replaces the stacked R factors (each wave writes the
// rows it has read).
template <int NW, int LEVEL>
__global__ __launch_bounds__(64 * NW) void k_tsqr_fact(QrBatch A, int j0, int half) {
  const int q = blockIdx.y, x = blockIdx.x;
  PanelGeom g;
  if (!panel_geom(A, q, j0, g)) return;
  const TsqrLayout L = tsqr_layout(A.rows[q]);
  double* S0 = A.scratch + A.soff[q] + half * L.total;
  const int ld = A.ld[q];
  double* Mj = A.base + A.moff[q] + int64_t(j0) * ld + j0;
  int rows, lds_src;
  const double* src;
  double *V, *T, *Rdst;
  bool root;
  if constexpr (LEVEL == 0) {
    if (x >= g.nck) return;
    const int lo = part_lo(x, g.mp, g.nck);
    rows = part_lo(x + 1, g.mp, g.nck) - lo;
    src = Mj + int64_t(lo) * ld;
    lds_src = ld;
    V = S0 + L.V + int64_t(lo) * kTb;
    T = S0 + L.Tc + int64_t(x) * kTb * kTb;
    Rdst = S0 + L.S + int64_t(x) * kTb * kTb;
    root = g.nck == 1;
  } else if constexpr (LEVEL == 1) {
    if (x >= g.ng) return;
    const int lo = part_lo(x, g.nck, g.ng);
    rows = (part_lo(x + 1, g.nck, g.ng) - lo) * kTb;
    V = S0 + L.S + int64_t(lo) * kTb * kTb;
    src = V;
    lds_src = kTb;
    T = S0 + L.T1 + int64_t(x) * kTb * kTb;
    Rdst = S0 + L.S2 + int64_t(x) * kTb * kTb;
    root = g.ng == 1;
  } else {
    if (x > 0 || g.ng < 2) return;
    rows = g.ng * kTb;
    V = S0 + L.S2;
    src = V;
    lds_src = kTb;
    T = S0 + L.T2;
    Rdst = nullptr;
    root = true;
  }
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const bool ok0 = li < g.jb, ok1 = 16 + li < g.jb;
  double y[16][2];
#pragma unroll
  for (int s = 0; s < 16; ++s) {
    const int r = 64 * wv + 4 * s + lk;
    const double* p = src + int64_t(r < rows ? r : 0) * lds_src;
    const double u0 = p[ok0 ? li : 0], u1 = p[ok1 ? 16 + li : 0];
    y[s][0] = (r < rows && ok0) ? u0 : 0.0;
    y[s][1] = (r < rows && ok1) ? u1 : 0.0;
  }
  __shared__ FactLds<NW> F;
  block_qr<NW>(y, g.jb, F);
  if (wv == 0) {  // R: rows < jb, upper triangle
    const int ldr = root ? ld : kTb;
    double* dst = root ? Mj : Rdst;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int r = 4 * s + lk;
      if (!root || (r < g.jb && li < g.jb)) dst[int64_t(r) * ldr + li] = (r < g.jb && li >= r) ? y[s][0] : 0.0;
      if (!root || (r < g.jb && 16 + li < g.jb))
        dst[int64_t(r) * ldr + 16 + li] = (r < g.jb && 16 + li >= r) ? y[s][1] : 0.0;
    }
    const double v0a = F.v0[li], v0b = F.v0[16 + li];
#pragma unroll
    for (int s = 0; s < 8; ++s) {  // V: unit of the reflectors on the diagonal, zero above
      const int r = 4 * s + lk;
      y[s][0] = r > li ? y[s][0] : (r == li ? v0a : 0.0);
      y[s][1] = r > 16 + li ? y[s][1] : (r == 16 + li ? v0b : 0.0);
    }
  }
#pragma unroll
  for (int s = 0; s < 16; ++s) {
    const int r = 64 * wv + 4 * s + lk;
    if (r < rows) {
      V[int64_t(r) * kTb + li] = ok0 ? y[s][0] : 0.0;
      V[int64_t(r) * kTb + 16 + li] = ok1 ? y[s][1] : 0.0;
    }
  }
  build_T<NW>(F, T);
}

// Y <- (I - V T V^T)^T Y = Y - (V T^T) V^T Y of one node's rows, columns
// cbeg + 16 tpw x .. (tpw tiles of 16 columns per workgroup).  Wave w owns
// rows 64 w .. 64 w + 63 and keeps its slices of V and V T^T in registers for
// all tiles; per tile it forms its share of P = V^T Y, the waves add their
// shares through LDS (double-buffered: one barrier per tile), and Y -= (V T^T) P.
// In the 16x16x4 FP64 layout, element v of an accumulator tile holds rows
// 4 v + lane / 16 of column lane % 16, which is the B operand of K-step v: P
// needs no shuffle, and neither does V T^T, formed transposed as T V^T.
// Each tile moves 16 KB per wave for 64 matrix instructions (4096 cycles of
// its SIMD): bound by memory on large problems.  64 problems of 3160 x 731:
// 2.16 GB in 0.71 ms for the first panel's update, the whole compression 12.0 ms
// against 16.6 ms when a workgroup read its 256 x 128 tile, multiplied and
// wrote it one after the other.
template <int NW, int LEVEL>
__global__ __launch_bounds__(64 * NW, 2) void k_tsqr_apply(QrBatch A, int j0, int half, int cbeg, int cend, int tpw) {
  const int q = blockIdx.z, x = blockIdx.y;
  PanelGeom g;
  if (!panel_geom(A, q, j0, g)) return;
  if (A.j0v) {
    cbeg = j0 + g.jb;
    cend = A.cols[q];
  }
  const int c0 = cbeg + int(blockIdx.x) * 16 * tpw, ce = min(min(A.cols[q], cend), c0 + 16 * tpw);
  if (c0 >= ce) return;
  const TsqrLayout L = tsqr_layout(A.rows[q]);
  const double* S0 = A.scratch + A.soff[q] + half * L.total;
  const int ld = A.ld[q];
  double* Mj = A.base + A.moff[q] + int64_t(j0) * ld;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  int rows;
  const double *V, *T;
  int rb[4];  // first row of each 16-row tile of the wave, from the panel's top
  if constexpr (LEVEL == 0) {
    if (x >= g.nck) return;
    const int lo = part_lo(x, g.mp, g.nck);
    rows = part_lo(x + 1, g.mp, g.nck) - lo;
    V = S0 + L.V + int64_t(lo) * kTb;
    T = S0 + L.Tc + int64_t(x) * kTb * kTb;
#pragma unroll
    for (int t = 0; t < 4; ++t) rb[t] = lo + 64 * wv + 16 * t;
  } else if constexpr (LEVEL == 1) {
    if (x >= g.ng) return;
    const int lo = part_lo(x, g.nck, g.ng), hi = part_lo(x + 1, g.nck, g.ng);
    rows = (hi - lo) * kTb;
    V = S0 + L.S + int64_t(lo) * kTb * kTb;
    T = S0 + L.T1 + int64_t(x) * kTb * kTb;
#pragma unroll
    for (int t = 0; t < 4; ++t) rb[t] = part_lo(min(lo + 2 * wv + t / 2, g.nck), g.mp, g.nck) + 16 * (t & 1);
  } else {
    if (x > 0 || g.ng < 2) return;
    rows = g.ng * kTb;
    V = S0 + L.S2;
    T = S0 + L.T2;
#pragma unroll
    for (int t = 0; t < 4; ++t)
      rb[t] = part_lo(part_lo(min(2 * wv + t / 2, g.ng), g.nck, g.ng), g.mp, g.nck) + 16 * (t & 1);
  }
  // Rows past the node are not masked but read from a row of the block that
  // exists: their rows of V are zero here, and they are not written.
  const int nv = rows - 64 * wv;  // rows of this wave (may be <= 0)
#pragma unroll
  for (int t = 0; t < 4; ++t)
    if (16 * t >= nv) rb[t] = 0;
  double va0[16], va1[16], vp[4][8];  // V (two column groups), -V T^T
  {
    double ta[8], tb[4];  // -T, rows 0..15 (all columns) and 16..31 (columns 16..31: T is upper triangular)
#pragma unroll
    for (int s = 0; s < 8; ++s) ta[s] = -T[li * kTb + 4 * s + lk];
#pragma unroll
    for (int s = 0; s < 4; ++s) tb[s] = -T[(16 + li) * kTb + 16 + 4 * s + lk];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const bool in = 16 * t + li < nv;
      const double* p = V + (in ? 64 * wv + 16 * t + li : 0) * kTb + lk;
      double4_t d0 = {0.0, 0.0, 0.0, 0.0}, d1 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const double u = p[4 * s];
        const double vt = in ? u : 0.0;
        d0 = mfma_f64(ta[s], vt, d0);
        if (s >= 4) d1 = mfma_f64(tb[s - 4], vt, d1);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        vp[t][v] = d0[v];
        vp[t][4 + v] = d1[v];
      }
    }
  }
  __builtin_amdgcn_sched_barrier(0);  // the fragments of V below come after T's are dead
#pragma unroll
  for (int s = 0; s < 16; ++s) {
    const bool in = 4 * s + lk < nv;
    const double* p = V + (in ? 64 * wv + 4 * s + lk : 0) * kTb + li;
    const double u0 = p[0], u1 = p[16];
    va0[s] = in ? u0 : 0.0;
    va1[s] = in ? u1 : 0.0;
  }
  __shared__ double sP[2][NW][8][64], sS[2][8][64];
  // the next tile is read before the present one is worked on
  double y[4][4], yn[4][4];
  auto load = [&](int c) {
    const int lc = c + li < ce ? li : 0;  // columns past the range: the tile's first
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const double* p = Mj + (int64_t(rb[t]) * ld + c);
#pragma unroll
      for (int v = 0; v < 4; ++v) yn[t][v] = p[(16 * t + 4 * v + lk < nv ? (4 * v + lk) * ld : 0) + lc];
    }
  };
  load(c0);
  int b = 0;
  for (int c = c0; c < ce; c += 16, b ^= 1) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) y[t][v] = yn[t][v];
    if (c + 16 < ce) load(c + 16);
    __builtin_amdgcn_sched_barrier(0);
    double4_t p0 = {0.0, 0.0, 0.0, 0.0}, p1 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        p0 = mfma_f64(va0[4 * t + v], y[t][v], p0);
        p1 = mfma_f64(va1[4 * t + v], y[t][v], p1);
      }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      sP[b][wv][e][lane] = p0[e];
      sP[b][wv][4 + e][lane] = p1[e];
    }
    __syncthreads();
    // every wave sums 8 / NW of the entries over the waves
#pragma unroll
    for (int e = 0; e < 8 / NW; ++e) {
      const int ee = wv * (8 / NW) + e;
      double s = 0.0;
#pragma unroll
      for (int w = 0; w < NW; ++w) s += sP[b][w][ee][lane];
      sS[b][ee][lane] = s;
    }
    __syncthreads();
    double p[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) p[e] = sS[b][e][lane];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      double4_t d = {y[t][0], y[t][1], y[t][2], y[t][3]};
#pragma unroll
      for (int s = 0; s < 8; ++s) d = mfma_f64(vp[t][s], p[s], d);
#pragma unroll
      for (int v = 0; v < 4; ++v) y[t][v] = d[v];
    }
    // The next tile's loads are waited for here, ahead of the (masked) stores:
    // a wait past them would have to count the stores too.
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
    __builtin_amdgcn_sched_barrier(0);
    const bool ok = c + li < ce;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      double* p2 = Mj + (int64_t(rb[t]) * ld + c);
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (ok && 16 * t + 4 * v + lk < nv) p2[(4 * v + lk) * ld + li] = y[t][v];
    }
  }
}

}  // namespace

// Second stream of the row compression's look-ahead, one per host thread and
// device, with the three events that order it against the caller's stream;
// created on first use and kept for the life of the thread (creating and
// destroying them per call costs a host wait on their work each time, and
// an event must not be destroyed while a stream still waits on it), or
// until release_thread_streams.
struct AuxStream {
  hipStream_t s2 = nullptr;
  hipEvent_t ev_chunk = nullptr, ev_fact = nullptr, ev_rest = nullptr;
};

static std::map<int, AuxStream>& aux_streams() {
  thread_local std::map<int, AuxStream> streams;
  return streams;
}

static void destroy_aux(const AuxStream& a) {
  for (hipEvent_t e : {a.ev_chunk, a.ev_fact, a.ev_rest})
    if (e) (void)hipEventDestroy(e);
  (void)hipStreamDestroy(a.s2);
}

static const AuxStream& aux_stream() {
  std::map<int, AuxStream>& streams = aux_streams();
  int dev = 0;
  HIF_HIP(hipGetDevice(&dev));
  auto it = streams.find(dev);
  if (it != streams.end()) return it->second;
  AuxStream a;
  HIF_HIP(hipStreamCreateWithFlags(&a.s2, hipStreamNonBlocking));
  for (hipEvent_t* e : {&a.ev_chunk, &a.ev_fact, &a.ev_rest})
    if (hipEventCreateWithFlags(e, hipEventDisableTiming) != hipSuccess) {
      *e = nullptr;
      destroy_aux(a);
      throw Error{HIF_EDEVICE, "creating the look-ahead events failed"};
    }
  return streams[dev] = a;
}

void release_thread_streams() {
  std::map<int, AuxStream>& streams = aux_streams();
  int cur = 0;
  (void)hipGetDevice(&cur);
  for (auto& kv : streams) {
    (void)hipSetDevice(kv.first);
    (void)hipStreamSynchronize(kv.second.s2);
    dbuf_retire_stream(kv.second.s2);
    destroy_aux(kv.second);
  }
  streams.clear();
  (void)hipSetDevice(cur);
}

// Updates of the columns [cbeg, cend) with the reflectors of one tree level.
// A workgroup pays for V, T and V T^T once, about what one tile costs, so it
// takes as many tiles as leave kApplyWaves waves in the launch: two rounds of
// the 8 waves a CU holds, which even out problems of unequal height.
constexpr int kApplyWaves = 4096;
template <int NW, int LEVEL>
static void launch_apply(const QrBatch& A, int j0, int half, int cbeg, int cend, int nodes, hipStream_t s) {
  const int tiles = (cend - cbeg + 15) / 16;
  const int64_t base = int64_t(nodes) * A.nprob;
  const int splits = int(std::min<int64_t>(tiles, std::max<int64_t>(1, (kApplyWaves / NW + base - 1) / base)));
  const int tpw = (tiles + splits - 1) / splits;
  hipLaunchKernelGGL((k_tsqr_apply<NW, LEVEL>), dim3(unsigned((tiles + tpw - 1) / tpw), unsigned(nodes), A.nprob),
                     dim3(64 * NW), 0, s, A, j0, half, cbeg, cend, tpw);
}

// Waves of a tree node, 64 rows each, for nodes of at most this many rows.
// Waves with no row would take part in every barrier, sum and product: a stack
// of 3 chunk factors by 8 waves took 42 us a panel, where a whole chunk of 256
// rows by 4 took 30.
template <typename F>
static void node_waves(int rows, int most, F f) {
  if (rows <= 128)
    f(std::integral_constant<int, 2>{});
  else if (rows <= 256 || most == 4)
    f(std::integral_constant<int, 4>{});
  else
    f(std::integral_constant<int, 8>{});
}

// The rows of the nodes of each tree level, of a batch whose tallest panel has
// mp rows: with more than one group of chunks in the tallest, a shorter one may
// still have a full group.
struct TreeRows {
  int nck, ng, rows[3];
  explicit TreeRows(int mp) : nck(std::max(1, tsqr_chunks(mp))), ng(tsqr_groups(nck)) {
    rows[0] = std::min(mp, kTsqrRows);
    rows[1] = std::min(nck, kTsqrFan) * kTb;
    rows[2] = ng * kTb;
  }
  int nodes(int level) const { return level == 0 ? nck : level == 1 ? ng : 1; }
  bool has(int level) const { return level == 0 || (level == 1 ? nck > 1 : ng > 1); }
};

template <int LEVEL>
static void launch_fact(const QrBatch& A, const TreeRows& t, int j0, int half, hipStream_t s) {
  if (!t.has(LEVEL)) return;
  node_waves(t.rows[LEVEL], LEVEL == 0 ? 4 : 8, [&](auto nw) {
    constexpr int NW = decltype(nw)::value;
    if constexpr (LEVEL > 0 || NW <= 4)
      hipLaunchKernelGGL((k_tsqr_fact<NW, LEVEL>), dim3(unsigned(t.nodes(LEVEL)), unsigned(A.nprob)), dim3(64 * NW), 0,
                         s, A, j0, half);
  });
}

template <int LEVEL>
static void launch_apply(const QrBatch& A, const TreeRows& t, int j0, int half, int cbeg, int cend, hipStream_t s) {
  if (!t.has(LEVEL)) return;
  node_waves(t.rows[LEVEL], LEVEL == 0 ? 4 : 8, [&](auto nw) {
    constexpr int NW = decltype(nw)::value;
    if constexpr (LEVEL > 0 || NW <= 4) launch_apply<NW, LEVEL>(A, j0, half, cbeg, cend, t.nodes(LEVEL), s);
  });
}

void launch_tsqr(const QrBatch& A, int max_rows, int max_cols, hipStream_t s) {
  // Look-ahead: panel p is factored on s; its update of the next panel's
  // 32 columns also runs on s, and that of the remaining columns on a
  // second stream, overlapping the factorization of panel p + 1.  Panels
  // alternate between two scratch halves (p & 1), so that panel p + 1
  // never overwrites the V and T that the update of panel p still reads.
  // Orders: the update of panel p on any column follows that of panel
  // p - 1 (s waits for the remaining-columns update of p - 1 before its
  // own updates of panel p), the remaining columns' chunk update of p
  // follows the chunks' factorization of p and their update by the upper
  // tree levels that of those levels (events recorded after each).
  const AuxStream& aux = aux_stream();
  hipStream_t s2 = aux.s2;
  bool rest_pending = false;
  for (int j0 = 0, p = 0; j0 < max_cols; j0 += kTb, ++p) {
    const int half = p & 1;
    const TreeRows t(max_rows - j0);
    const int nb0 = j0 + kTb, nb1 = j0 + 2 * kTb;  // next panel: columns [nb0, nb1)
    const bool rest = nb1 < max_cols;
    launch_fact<0>(A, t, j0, half, s);
    if (rest) HIF_HIP(hipEventRecord(aux.ev_chunk, s));
    launch_fact<1>(A, t, j0, half, s);
    launch_fact<2>(A, t, j0, half, s);
    if (nb0 >= max_cols) break;
    if (rest) HIF_HIP(hipEventRecord(aux.ev_fact, s));
    if (rest_pending) HIF_HIP(hipStreamWaitEvent(s, aux.ev_rest, 0));  // remaining-columns update of p - 1
    rest_pending = false;
    if (rest) {
      HIF_HIP(hipStreamWaitEvent(s2, aux.ev_chunk, 0));
      launch_apply<0>(A, t, j0, half, nb1, max_cols, s2);
      HIF_HIP(hipStreamWaitEvent(s2, aux.ev_fact, 0));
      launch_apply<1>(A, t, j0, half, nb1, max_cols, s2);
      launch_apply<2>(A, t, j0, half, nb1, max_cols, s2);
      HIF_HIP(hipEventRecord(aux.ev_rest, s2));
      rest_pending = true;
    }
    const int ne = std::min(nb1, max_cols);
    launch_apply<0>(A, t, j0, half, nb0, ne, s);
    launch_apply<1>(A, t, j0, half, nb0, ne, s);
    launch_apply<2>(A, t, j0, half, nb0, ne, s);
  }
  if (rest_pending) HIF_HIP(hipStreamWaitEvent(s, aux.ev_rest, 0));
  HIF_HIP(hipGetLastError());
}

void launch_tsqr_panel(const QrBatch& A, int max_rows, int max_trail, hipStream_t s) {
  const TreeRows t(max_rows);
  launch_fact<0>(A, t, 0, 0, s);
  launch_fact<1>(A, t, 0, 0, s);
  launch_fact<2>(A, t, 0, 0, s);
  if (max_trail > 0) {
    // the columns themselves come from each problem's panel; max_trail sizes the grid
    launch_apply<0>(A, t, 0, 0, 0, max_trail, s);
    launch_apply<1>(A, t, 0, 0, 0, max_trail, s);
    launch_apply<2>(A, t, 0, 0, 0, max_trail, s);
  }
  HIF_HIP(hipGetLastError());
}

}  // namespace hif
