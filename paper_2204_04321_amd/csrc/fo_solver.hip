// Linear-algebra kernels behind fo_newton_solve: SpMV over the Jacobian layout with FP64 or FP32 values,
// the vertical-column block preconditioner, and the fused Krylov vector kernels.
//
// Preconditioner.  Each vertex column of the extruded mesh couples its own 2(L+1)
// dofs through a block-tridiagonal matrix (2x2 blocks, one per level).  Extracting
// that block from J and factoring it by block LU without pivoting, one vertical line
// per thread, follows the batched per-line solve the paper uses inside its
// semicoarsening multigrid (arXiv:2204.04321 Sec. 4.4); here it is used directly as
// a block-Jacobi preconditioner for GMRES (Sec. 3.1 names GMRES as the Krylov method).
#include <hip/hip_runtime.h>

#include "fo_internal.h"
#include "fo_solver.h"

namespace fo {
namespace {

__device__ __forceinline__ int nlev(int k, int L) { return (k == 0 || k == L) ? 2 : 3; }
__device__ __forceinline__ int cumlev(int k) { return k == 0 ? 0 : 3 * k - 1; }

constexpr int SPMV_LANES = 8;   // lanes per node (pair of rows); a wave per column with its neighbours' x and the
                                // products in LDS reads the values as one run but is slower (198 -> 214 us)
constexpr int APPLY_COLS = 64;          // most columns of a preconditioner-apply block
constexpr int APPLY_THREADS = 256;      // its threads: all stage and copy, one per column sweeps

template <class JT> struct Pair2;
template <> struct Pair2<double> { using T = double2; };
template <> struct Pair2<float> { using T = float2; };

// y = J x over the Jacobian's own layout, without the CSR column indices.  The two rows of
// node (v, k) (components u and v) share one column list and follow each other: the row
// block starts at colptr[v] + 4 D cumlev(k), row c at + c 2 nl D, and entry (r, lev, d)
// at + r 2 nl + 2 lev + d couples neighbour r of v (sorted list), level klo + lev,
// component d.  Each lane takes whole (u, v) column pairs: one 16-byte x load and one
// two-value load per row.
template <class JT>
__global__ __launch_bounds__(256) void spmv_kernel(int V, int L, const int64_t *__restrict__ colptr,
                                                   const int32_t *__restrict__ nbr_ptr,
                                                   const int32_t *__restrict__ nbr_idx,
                                                   const JT *__restrict__ vals, const double *__restrict__ x,
                                                   double *__restrict__ y) {
  using T2 = typename Pair2<JT>::T;
  const int64_t gid = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t node = gid / SPMV_LANES;
  const int sub = int(gid % SPMV_LANES);
  const int64_t n_nodes = int64_t(V) * (L + 1);
  double a0 = 0.0, a1 = 0.0;
  if (node < n_nodes) {
    const int v = int(node / (L + 1)), k = int(node - int64_t(v) * (L + 1));
    const int nb = nbr_ptr[v], D = nbr_ptr[v + 1] - nb;
    const int nl = nlev(k, L);
    const int klo = k > 0 ? k - 1 : 0;
    const JT *row = vals + colptr[v] + int64_t(4) * D * cumlev(k);
    const int len = 2 * nl * D;
    if constexpr (sizeof(JT) == 4) {
      // FP32 values: two column pairs per lane, one 16-byte load per row (the second row
      // starts 2 nl D entries later, so its loads are only 8-byte aligned)
      for (int q = 2 * sub; q + 1 < nl * D; q += 2 * SPMV_LANES) {
        const int r0 = nl == 3 ? (q * 43691) >> 17 : q >> 1, r1 = nl == 3 ? ((q + 1) * 43691) >> 17 : (q + 1) >> 1;
        const int64_t c0 = 2 * (int64_t(nbr_idx[nb + r0]) * (L + 1) + klo + (q - r0 * nl));
        const int64_t c1 = 2 * (int64_t(nbr_idx[nb + r1]) * (L + 1) + klo + (q + 1 - r1 * nl));
        const double2 x0 = *reinterpret_cast<const double2 *>(x + c0);
        const double2 x1 = *reinterpret_cast<const double2 *>(x + c1);
        float4 v0, v1;
        __builtin_memcpy(&v0, row + 2 * q, sizeof v0);
        __builtin_memcpy(&v1, row + len + 2 * q, sizeof v1);
        a0 = fma(double(v0.x), x0.x, fma(double(v0.y), x0.y, a0));
        a0 = fma(double(v0.z), x1.x, fma(double(v0.w), x1.y, a0));
        a1 = fma(double(v1.x), x0.x, fma(double(v1.y), x0.y, a1));
        a1 = fma(double(v1.z), x1.x, fma(double(v1.w), x1.y, a1));
      }
      if ((nl * D) & 1) {   // the last column pair of an odd count
        const int q = nl * D - 1;
        if (sub == (q >> 1) % SPMV_LANES) {
          const int r = nl == 3 ? (q * 43691) >> 17 : q >> 1;
          const int64_t col = 2 * (int64_t(nbr_idx[nb + r]) * (L + 1) + klo + (q - r * nl));
          const double2 xv = *reinterpret_cast<const double2 *>(x + col);
          const T2 v0 = *reinterpret_cast<const T2 *>(row + 2 * q), v1 = *reinterpret_cast<const T2 *>(row + len + 2 * q);
          a0 = fma(double(v0.x), xv.x, fma(double(v0.y), xv.y, a0));
          a1 = fma(double(v1.x), xv.x, fma(double(v1.y), xv.y, a1));
        }
      }
    } else
    for (int q = sub; q < nl * D; q += SPMV_LANES) {
      const int r = nl == 3 ? (q * 43691) >> 17 : q >> 1;   // q / nl, exact for q < 65536
      const int lev = q - r * nl;
      const int64_t col = 2 * (int64_t(nbr_idx[nb + r]) * (L + 1) + klo + lev);
      const double2 xv = *reinterpret_cast<const double2 *>(x + col);
      const T2 v0 = *reinterpret_cast<const T2 *>(row + 2 * q), v1 = *reinterpret_cast<const T2 *>(row + len + 2 * q);
      a0 = fma(double(v0.x), xv.x, fma(double(v0.y), xv.y, a0));
      a1 = fma(double(v1.x), xv.x, fma(double(v1.y), xv.y, a1));
    }
  }
#pragma unroll
  for (int off = SPMV_LANES / 2; off > 0; off >>= 1) {
    a0 += __shfl_xor(a0, off, SPMV_LANES);
    a1 += __shfl_xor(a1, off, SPMV_LANES);
  }
  if (node < n_nodes && sub == 0) {
    y[2 * node] = a0;
    y[2 * node + 1] = a1;
  }
}

// A level's three 2x2 blocks of a vertical line, by row: coupling to level k - 1, diagonal, coupling
// to level k + 1 (zero where there is none).  The pairs may lie on any boundary of their type.
template <class JT>
struct LineRows {
  typedef JT V2 __attribute__((ext_vector_type(2), aligned(alignof(JT))));
  V2 lo[2], di[2], up[2];
  __device__ __forceinline__ void load(const JT *__restrict__ vals, int D, int sr, int k, int L) {
    const int nl = nlev(k, L);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const V2 *p = reinterpret_cast<const V2 *>(vals + int64_t(4) * D * cumlev(k) + c * 2 * nl * D + sr * 2 * nl);
      lo[c] = V2{0, 0};
      up[c] = V2{0, 0};
      if (k > 0) lo[c] = *p++;
      di[c] = p[0];
      if (k < L) up[c] = p[1];
    }
  }
};

// 2x2 product, [2 r + c]
__device__ __forceinline__ void mul22(const double *a, const double *b, double *o) {
  o[0] = a[0] * b[0] + a[1] * b[2];
  o[1] = a[0] * b[1] + a[1] * b[3];
  o[2] = a[2] * b[0] + a[3] * b[2];
  o[3] = a[2] * b[1] + a[3] * b[3];
}

// Block-tridiagonal factor of one vertical line (a column per thread): per level k the inverse
// of the Schur complement S_k = D_k - Lo_k G_{k-1} (2x2), the coupling to level k-1 (Lo_k) and
// G_k = S_k^{-1} Up_k (Up_k: the coupling to level k+1), which is all the backward sweep needs.
// The recursion runs in FP64; the stored factors are FP32 (half the bytes for every
// preconditioner apply), which defines a fixed linear M^{-1} as right preconditioning needs.
//
// WEIGHTS also forms the collapse weights of the two-level preconditioner from the same values:
// forward Y_k = S_k^-1 (I - Lo_k Y_{k-1}) for the two right-hand sides e_u, e_v at once (rows the
// level's components, columns the right-hand sides), backward Z_k = Y_k - G_k Z_{k+1}, then each
// right-hand side's solution is divided by the mean of its own component over the levels (e_c
// itself where that is not usable).  The block's columns (4 (L+1) values each, Y/Z and G) live in
// LDS and leave with coalesced stores, in FP64 and rounded to FP32.
//
// Bound by memory latency: a column's rows lie apart in J and its levels follow from each other, so
// the rows are loaded two levels ahead (125,000 columns of 10 layers, FP64: 120 us without the
// weights, and 123 us for a kernel of their own that read the same rows again; together 144 us, of
// which the ~300 MB of 64-byte pieces the rows touch take 60; 2,000 columns, alone: 17 -> 12 us).
template <class JT, bool WEIGHTS>
__global__ __launch_bounds__(64) void colblock_factor_kernel(MeshView m, const int32_t *__restrict__ self_rank,
                                                             const JT *__restrict__ vals, float *__restrict__ fac,
                                                             double *__restrict__ W, float *__restrict__ W32) {
  extern __shared__ double wsh[];   // [2][blockDim.x][4 (L + 1)]: Z then G
  const int L = m.L, nw = 4 * (L + 1);
  const int64_t V = m.V, v0 = int64_t(blockIdx.x) * blockDim.x;
  const int nv = int(V - v0 < int64_t(blockDim.x) ? V - v0 : int64_t(blockDim.x));
  if (int(threadIdx.x) < nv) {
    const int64_t v = v0 + threadIdx.x;
    const int D = m.deg[v], sr = self_rank[v];
    const JT *line = vals + m.colptr[v];
    double *Wv = wsh + threadIdx.x * nw, *Gv = wsh + (blockDim.x + threadIdx.x) * nw;
    double G[4] = {0, 0, 0, 0}, Y[4] = {0, 0, 0, 0};
    LineRows<JT> cur, n1, n2;
    n1.load(line, D, sr, 0, L);
    n2.load(line, D, sr, 1, L);
    for (int k = 0; k <= L; ++k) {
      cur = n1;
      n1 = n2;
      if (k + 2 <= L) n2.load(line, D, sr, k + 2, L);
      const double Lo[4] = {double(cur.lo[0].x), double(cur.lo[0].y), double(cur.lo[1].x), double(cur.lo[1].y)};
      const double Up[4] = {double(cur.up[0].x), double(cur.up[0].y), double(cur.up[1].x), double(cur.up[1].y)};
      double S[4] = {double(cur.di[0].x), double(cur.di[0].y), double(cur.di[1].x), double(cur.di[1].y)};
      double t[4];
      mul22(Lo, G, t);
      for (int i = 0; i < 4; ++i) S[i] -= t[i];
      const double det = S[0] * S[3] - S[1] * S[2];
      const double Si[4] = {S[3] / det, -S[1] / det, -S[2] / det, S[0] / det};
      mul22(Si, Up, G);
      float *Fk = fac + int64_t(k) * 12 * V + v;   // field f of level k at Fk[f V]
      for (int i = 0; i < 4; ++i) {
        Fk[i * V] = float(Si[i]);
        Fk[(4 + i) * V] = float(Lo[i]);
        Fk[(8 + i) * V] = float(G[i]);
      }
      if constexpr (WEIGHTS) {
        double T[4] = {1, 0, 0, 1};
        mul22(Lo, Y, t);
        for (int i = 0; i < 4; ++i) T[i] -= t[i];
        mul22(Si, T, Y);
        for (int i = 0; i < 4; ++i) {
          Gv[4 * k + i] = G[i];
          Wv[4 * k + i] = Y[i];
        }
      }
    }
    if constexpr (WEIGHTS) {
      double Z[4] = {Y[0], Y[1], Y[2], Y[3]};
      double sum[2] = {Y[0], Y[3]};
      bool finite[2] = {isfinite(Y[0]) && isfinite(Y[2]), isfinite(Y[1]) && isfinite(Y[3])};
      for (int k = L - 1; k >= 0; --k) {
        double t[4];
        mul22(Gv + 4 * k, Z, t);
        for (int i = 0; i < 4; ++i) {
          Z[i] = Wv[4 * k + i] - t[i];
          Wv[4 * k + i] = Z[i];
        }
        for (int c = 0; c < 2; ++c) {
          sum[c] += Z[3 * c];
          finite[c] = finite[c] && isfinite(Z[c]) && isfinite(Z[2 + c]);
        }
      }
      for (int c = 0; c < 2; ++c) {
        const double mean = sum[c] / double(L + 1);
        const bool ok = finite[c] && isfinite(mean) && mean > 0.0;
        for (int k = 0; k <= L; ++k)
          for (int cp = 0; cp < 2; ++cp)
            Wv[4 * k + 2 * cp + c] = ok ? Wv[4 * k + 2 * cp + c] / mean : (cp == c ? 1.0 : 0.0);
      }
    }
  }
  if constexpr (WEIGHTS) {
    __syncthreads();
    for (int e = threadIdx.x; e < nv * nw; e += blockDim.x) {
      const double w = wsh[e];
      W[v0 * nw + e] = w;
      W32[v0 * nw + e] = float(w);
    }
  }
}

// Forward then backward block substitution of one vertical line, in place on its 2 (L+1)
// values zv (r in, z = M^{-1} r out).  F(f, k) is factor field f of level k; the next level's are
// taken one level ahead.
template <class F>
__device__ __forceinline__ void column_sweep(int L, double *zv, F fac) {
  // forward: y_k = r_k - Lo_k S_{k-1}^{-1} y_{k-1}; keep w_k = S_k^{-1} y_k
  double f[8], fn[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) fn[i] = double(fac(i, 0));
  double w0 = 0, w1 = 0;
  for (int k = 0; k <= L; ++k) {
#pragma unroll
    for (int i = 0; i < 8; ++i) f[i] = fn[i];
    double y0 = zv[2 * k], y1 = zv[2 * k + 1];
    if (k < L) {
#pragma unroll
      for (int i = 0; i < 8; ++i) fn[i] = double(fac(i, k + 1));
    }
    if (k > 0) {
      y0 -= f[4] * w0 + f[5] * w1;
      y1 -= f[6] * w0 + f[7] * w1;
    }
    w0 = f[0] * y0 + f[1] * y1;
    w1 = f[2] * y0 + f[3] * y1;
    zv[2 * k] = w0;
    zv[2 * k + 1] = w1;
  }
  // backward: z_k = w_k - G_k z_{k+1}, G_k = S_k^{-1} Up_k
  double z0 = zv[2 * L], z1 = zv[2 * L + 1];
  double g[4], gn[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) gn[i] = double(fac(8 + i, L - 1 >= 0 ? L - 1 : 0));
  for (int k = L - 1; k >= 0; --k) {
#pragma unroll
    for (int i = 0; i < 4; ++i) g[i] = gn[i];
    if (k > 0) {
#pragma unroll
      for (int i = 0; i < 4; ++i) gn[i] = double(fac(8 + i, k - 1));
    }
    const double n0 = zv[2 * k] - (g[0] * z0 + g[1] * z1);
    const double n1 = zv[2 * k + 1] - (g[2] * z0 + g[3] * z1);
    z0 = n0;
    z1 = n1;
    zv[2 * k] = z0;
    zv[2 * k + 1] = z1;
  }
}

// The sweeps of a block's nv columns (v0 on), whose values lie in col [nv][2 (L+1)].  STAGED: all
// threads first copied the columns' factors to LDS (stage_factors), so the 2 (L+1) dependent
// steps wait for LDS and not for memory; otherwise a thread reads its column's from memory (a
// wave's loads of one field are contiguous, the vertex index being fastest).
template <bool STAGED>
__device__ __forceinline__ void sweep_columns(int V, int L, int64_t v0, int nv, const float *__restrict__ fac,
                                              double *col, const float *fsh) {
  const int t = threadIdx.x;
  if (t >= nv) return;
  if constexpr (STAGED) {
    const float *mine = fsh + t * 12 * (L + 1);
    column_sweep(L, col + t * 2 * (L + 1), [&](int f, int k) { return mine[12 * k + f]; });
  } else {
    const int64_t Vl = V, v = v0 + t;
    column_sweep(L, col + t * 2 * (L + 1), [&](int f, int k) { return fac[(int64_t(k) * 12 + f) * Vl + v]; });
  }
}

// fsh [cols][12 (L+1)] = the factors of columns v0 .. v0 + nv - 1
__device__ __forceinline__ void stage_factors(int V, int L, int cols, int64_t v0, int nv,
                                              const float *__restrict__ fac, float *fsh) {
  const int rows = 12 * (L + 1), shift = 31 - __clz(cols);     // cols is a power of two
#pragma unroll 4
  for (int e = threadIdx.x; e < rows * cols; e += blockDim.x) {
    const int row = e >> shift, c = e & (cols - 1);
    if (c < nv) fsh[c * rows + row] = fac[int64_t(row) * V + v0 + c];
  }
}

// z = M^{-1} r for every vertical line.  A block's `cols` columns are contiguous in r and z
// (2 (L+1) values each): all its threads copy them, and if STAGED their factors, to LDS with
// coalesced loads, and one thread per column runs the column's two sweeps in place there
// (apply_shape: which launch takes which form).
template <bool STAGED>
__global__ __launch_bounds__(APPLY_THREADS) void colblock_apply_kernel(int V, int L, int cols,
                                                                       const float *__restrict__ fac,
                                                                       const double *__restrict__ r,
                                                                       double *__restrict__ z) {
  extern __shared__ double col_sh[];   // [cols][2 (L + 1)], then the factors
  const int n = 2 * (L + 1);
  float *fsh = reinterpret_cast<float *>(col_sh + size_t(cols) * n);
  const int64_t v0 = int64_t(blockIdx.x) * cols;
  const int nv = int(V - v0 < int64_t(cols) ? V - v0 : int64_t(cols));
  for (int e = threadIdx.x; e < nv * n; e += blockDim.x) col_sh[e] = r[v0 * n + e];
  if constexpr (STAGED) stage_factors(V, L, cols, v0, nv, fac, fsh);
  __syncthreads();
  sweep_columns<STAGED>(V, L, v0, nv, fac, col_sh, fsh);
  __syncthreads();
  for (int e = threadIdx.x; e < nv * n; e += blockDim.x) z[v0 * n + e] = col_sh[e];
}

// The last step of the two-level preconditioner: z = P0 y + M^{-1} (r - (J P0) y).  While the
// block's columns are staged in LDS each row subtracts its row of J P0 against the plane vector
// y (J P0 in FP32, column v's block starting at 4 (L+1) nbr_ptr[v] and holding entry (r, d) of
// row q at (2 r + d) 2 (L+1) + q, so consecutive rows of a column are consecutive for each
// entry); after the sweeps each row adds its prolongation sum_c W[v][k][c'][c] y[(v, c)] (FP32
// weights, the two c of a row next to each other).
// A thread takes both rows of a node, so its loads are 8 bytes of J P0 and 16 of the others, and four
// blocks' loads are in flight (125,000 columns of 10 layers: 81 -> 70 us; the 290 MB take 57).
template <bool STAGED>
__global__ __launch_bounds__(APPLY_THREADS) void colblock_correction_kernel(
    int V, int L, int cols, const int32_t *__restrict__ nbr_ptr, const int32_t *__restrict__ nbr_idx,
    const float *__restrict__ fac, const float *__restrict__ W32, const float *__restrict__ JP,
    const double *__restrict__ y, const double *__restrict__ r, double *__restrict__ z) {
  extern __shared__ double col_sh[];   // [cols][2 (L + 1)], then the factors
  const int n = 2 * (L + 1);
  float *fsh = reinterpret_cast<float *>(col_sh + size_t(cols) * n);
  const int64_t v0 = int64_t(blockIdx.x) * cols;
  const int nv = int(V - v0 < int64_t(cols) ? V - v0 : int64_t(cols));
  const double2 *y2 = reinterpret_cast<const double2 *>(y);
  if constexpr (STAGED) stage_factors(V, L, cols, v0, nv, fac, fsh);
  const int64_t first = v0 * (L + 1);   // a thread takes both rows of a node
  for (int e = threadIdx.x; e < nv * (L + 1); e += blockDim.x) {
    const int c = e / (L + 1), k = e - c * (L + 1);
    const int64_t v = v0 + c;
    const int p0 = nbr_ptr[v], D = nbr_ptr[v + 1] - p0;
    const float2 *jp = reinterpret_cast<const float2 *>(JP + int64_t(2 * n) * p0) + k;
    double2 s = reinterpret_cast<const double2 *>(r)[first + e];
    for (int i0 = 0; i0 < D; i0 += 4) {   // four blocks' loads in flight; past the last block zeros
      float2 ja[4], jb[4];
      double2 yw[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = i0 + u < D ? i0 + u : D - 1;
        yw[u] = y2[nbr_idx[p0 + i]];
        ja[u] = jp[(2 * i) * (L + 1)];
        jb[u] = jp[(2 * i + 1) * (L + 1)];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const bool in = i0 + u < D;
        s.x -= double(in ? ja[u].x : 0.0f) * yw[u].x + double(in ? jb[u].x : 0.0f) * yw[u].y;
        s.y -= double(in ? ja[u].y : 0.0f) * yw[u].x + double(in ? jb[u].y : 0.0f) * yw[u].y;
      }
    }
    reinterpret_cast<double2 *>(col_sh)[e] = s;
  }
  __syncthreads();
  sweep_columns<STAGED>(V, L, v0, nv, fac, col_sh, fsh);
  __syncthreads();
  const float4 *W4 = reinterpret_cast<const float4 *>(W32);
  for (int e = threadIdx.x; e < nv * (L + 1); e += blockDim.x) {
    const float4 w = W4[first + e];
    const double2 yv = y2[v0 + e / (L + 1)], c = reinterpret_cast<const double2 *>(col_sh)[e];
    reinterpret_cast<double2 *>(z)[first + e] = make_double2(c.x + (double(w.x) * yv.x + double(w.y) * yv.y),
                                                             c.y + (double(w.z) * yv.x + double(w.w) * yv.y));
  }
}

constexpr int RED_BLOCK = 256;

constexpr int MD_GROUP = 24;   // dot products per pass over a block's chunk

// Sums of MD_GROUP values over a wave's 64 lanes: three exchanges halve the values a lane holds
// (24 -> 12 -> 6 -> 3) while they add over half the lanes each, then the last three add over eight
// lanes: 30 exchanges instead of 6 for each value.  Lane l ends with the sums of values
// 3 (l >> 3) .. 3 (l >> 3) + 2, bit order 5, 4, 3.
__device__ __forceinline__ void wave_sums(double (&s)[MD_GROUP], double (&out)[3]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int half = MD_GROUP / 2, bit = 32; half >= 3; half /= 2, bit /= 2) {
    const bool hi = (lane & bit) != 0;
#pragma unroll
    for (int i = 0; i < half; ++i) {
      const double keep = hi ? s[half + i] : s[i], send = hi ? s[i] : s[half + i];
      s[i] = keep + __shfl_xor(send, bit);
    }
  }
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    double t = s[i];
    for (int bit = 4; bit > 0; bit >>= 1) t += __shfl_xor(t, bit);
    out[i] = t;
  }
}

// One pass of multidot_kernel: G vectors at a time, all their loads in flight at once (a test per
// vector would make every load wait for the one before).  Past the last vector w itself is read,
// which is in the cache, and its sum dropped.
template <int G>
__device__ __forceinline__ void dot_pass(int64_t n2, const double *__restrict__ V, int64_t ld, int nv,
                                         const double *__restrict__ w, int i0, double (&s)[MD_GROUP]) {
  const int64_t stride = int64_t(gridDim.x) * RED_BLOCK;
  const double2 *w2 = reinterpret_cast<const double2 *>(w);
  auto vec = [&](int q) { return reinterpret_cast<const double2 *>(i0 + q < nv ? V + int64_t(i0 + q) * ld : w); };
  int64_t p = int64_t(blockIdx.x) * RED_BLOCK + threadIdx.x;
  for (; p + stride < n2; p += 2 * stride) {
    const double2 wp = w2[p], wq = w2[p + stride];
#pragma unroll
    for (int q = 0; q < G; ++q) {
      const double2 *Vi = vec(q);
      const double2 a = Vi[p], b = Vi[p + stride];
      s[q] = fma(a.x, wp.x, fma(a.y, wp.y, fma(b.x, wq.x, fma(b.y, wq.y, s[q]))));
    }
  }
  if (p < n2) {     // no second place: its products are left out, not multiplied by zero (infinite entries)
    const double2 wp = w2[p];
#pragma unroll
    for (int q = 0; q < G; ++q) {
      const double2 a = vec(q)[p];
      s[q] = fma(a.x, wp.x, fma(a.y, wp.y, s[q]));
    }
  }
}

// partial[i gridDim + b] = sum over block b's rows of V_i . w (i < nv), and w . w (i = nv).
// Vectors are taken MD_GROUP at a time, so each pass loads w once for all of them: each lane takes
// two consecutive entries (16-byte loads; n and ld are even) at two places a grid stride apart.
// Blocks stride through the vectors together, so at any time the grid reads one window of each
// vector (DRAM page locality); the summation order is fixed.
__global__ __launch_bounds__(RED_BLOCK) void multidot_kernel(int64_t n2, const double *__restrict__ V, int64_t ld,
                                                             int nv, const double *__restrict__ w,
                                                             double *__restrict__ partial) {
  __shared__ double red[MD_GROUP][RED_BLOCK / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int i0 = 0; i0 <= nv; i0 += MD_GROUP) {
    const int g = nv + 1 - i0 < MD_GROUP ? nv + 1 - i0 : MD_GROUP;
    double s[MD_GROUP];
#pragma unroll
    for (int q = 0; q < MD_GROUP; ++q) s[q] = 0.0;
    if (g <= 2) dot_pass<2>(n2, V, ld, nv, w, i0, s);
    else if (g <= 6) dot_pass<6>(n2, V, ld, nv, w, i0, s);
    else if (g <= 12) dot_pass<12>(n2, V, ld, nv, w, i0, s);
    else if (g <= 18) dot_pass<18>(n2, V, ld, nv, w, i0, s);
    else dot_pass<24>(n2, V, ld, nv, w, i0, s);
    double t[3];
    wave_sums(s, t);
    if ((lane & 7) == 0) {
#pragma unroll
      for (int i = 0; i < 3; ++i) red[3 * (lane >> 3) + i][wave] = t[i];
    }
    __syncthreads();
    if (threadIdx.x < g) {
      double u = 0.0;
      for (int q = 0; q < RED_BLOCK / 64; ++q) u += red[threadIdx.x][q];
      partial[int64_t(i0 + threadIdx.x) * gridDim.x + blockIdx.x] = u;
    }
    __syncthreads();
  }
}

// One block: out[i] = sum_b partial[i nb + b] (i <= nv) in a fixed order, one wave per i, and
// out[nv + 1], the factor that brings w - V h to unit length: 1 / sqrt(w . w - |h|^2), or 1 where
// that difference has lost too much to cancellation (not above drop w . w; the caller then
// projects once more) and 0 where it is not positive.  With `host` (pinned, coherent) the same
// values go there as well, and after them `seq` to host[kDotsFlag]: the host reads them as soon as they
// are there, while later kernels of the stream run.
__global__ __launch_bounds__(1024) void reduce_dots_kernel(int nb, int nv, const double *__restrict__ partial,
                                                           double drop, double *__restrict__ out, double *host,
                                                           uint64_t seq) {
  __shared__ double sum[kDotsMax], h2[16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double mine = 0.0;
  for (int i = wave; i <= nv; i += 16) {
    const double *row = partial + int64_t(i) * nb;
    double s = 0.0;
#pragma unroll 8
    for (int b = lane; b < nb; b += 64) s += row[b];
    for (int bit = 32; bit > 0; bit >>= 1) s += __shfl_xor(s, bit);
    if (lane == 0) {
      sum[i] = s;
      if (i < nv) mine += s * s;
    }
  }
  if (lane == 0) h2[wave] = mine;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int q = 0; q < 16; ++q) t += h2[q];
    const double left = sum[nv] - t;
    sum[nv + 1] = left > drop * sum[nv] ? 1.0 / sqrt(left) : drop > 0.0 ? 1.0 : 0.0;
  }
  __syncthreads();
  if (wave == 0) {      // one wave writes everything, so its release orders all of it before the flag
    for (int i = lane; i <= nv + 1; i += 64) {
      out[i] = sum[i];
      if (host) host[i] = sum[i];
    }
    if (host) {
      __threadfence_system();
      if (lane == 0)
        __hip_atomic_store(reinterpret_cast<uint64_t *>(host + kDotsFlag), seq, __ATOMIC_RELEASE,
                           __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }
}

// partial[2 b] = sum over block b's entries of a . w, partial[2 b + 1] of w . w; two
// consecutive entries per lane, grid-stride
__global__ __launch_bounds__(RED_BLOCK) void dot2_kernel(int64_t n2, const double *__restrict__ a,
                                                         const double *__restrict__ w,
                                                         double *__restrict__ partial) {
  __shared__ double red[2][RED_BLOCK / 64];
  const int64_t stride = int64_t(gridDim.x) * RED_BLOCK;
  const double2 *a2 = reinterpret_cast<const double2 *>(a);
  const double2 *w2 = reinterpret_cast<const double2 *>(w);
  double s0 = 0.0, s1 = 0.0;
  for (int64_t p = int64_t(blockIdx.x) * RED_BLOCK + threadIdx.x; p < n2; p += stride) {
    const double2 x = a2[p], y = w2[p];
    s0 = fma(x.x, y.x, fma(x.y, y.y, s0));
    s1 = fma(y.x, y.x, fma(y.y, y.y, s1));
  }
  for (int off = 32; off > 0; off >>= 1) {
    s0 += __shfl_xor(s0, off);
    s1 += __shfl_xor(s1, off);
  }
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = s0;
    red[1][threadIdx.x >> 6] = s1;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    double t = 0.0;
    for (int q = 0; q < RED_BLOCK / 64; ++q) t += red[threadIdx.x][q];
    partial[2 * int64_t(blockIdx.x) + threadIdx.x] = t;
  }
}

// out[i] = sum_b partial[b * stride + i], fixed order
__global__ void reduce_partials_kernel(int nb, int stride, const double *__restrict__ partial,
                                       double *__restrict__ out) {
  const int i = blockIdx.x;
  __shared__ double red[256 / 64];
  double s = 0.0;
  for (int b = threadIdx.x; b < nb; b += blockDim.x) s += partial[int64_t(b) * stride + i];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int q = 0; q < 4; ++q) t += red[q];
    out[i] = t;
  }
}

// out = scale (w + sign sum_i h_i V_i) (h, and scale where not NULL, on the device; w may be NULL
// for zero, or out), two consecutive entries per lane.  Walking the vectors from their ends, where
// the dot products before have just been, is no faster (90 against 86 us for 21 vectors of 2.75M).
__global__ __launch_bounds__(256) void multiaxpy_kernel(int64_t n2, const double *__restrict__ V, int64_t ld,
                                                        int nv, const double *__restrict__ h,
                                                        const double *__restrict__ scale, const double *w,
                                                        double *out, double sign) {
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  const double2 *w2 = reinterpret_cast<const double2 *>(w);
  double2 *o2 = reinterpret_cast<double2 *>(out);
  const double c = scale ? scale[0] : 1.0;
  for (int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; p < n2; p += stride) {
    double ax = 0.0, ay = 0.0;
#pragma unroll 8
    for (int i = 0; i < nv; ++i) {
      const double2 a = reinterpret_cast<const double2 *>(V + int64_t(i) * ld)[p];
      ax += h[i] * a.x;
      ay += h[i] * a.y;
    }
    const double2 t = w ? w2[p] : make_double2(0.0, 0.0);
    o2[p] = make_double2(c * (t.x + sign * ax), c * (t.y + sign * ay));
  }
}

// conjugate-gradient step with the step length formed on the device:
// alpha = num[0] / den[0], x += alpha p, r -= alpha q
__global__ __launch_bounds__(256) void cg_step_kernel(int64_t n, const double *__restrict__ num,
                                                      const double *__restrict__ den,
                                                      const double *__restrict__ p,
                                                      const double *__restrict__ q, double *__restrict__ x,
                                                      double *__restrict__ r) {
  const double alpha = num[0] / den[0];
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) {
    x[i] += alpha * p[i];
    r[i] -= alpha * q[i];
  }
}

// y = a x + b y
__global__ __launch_bounds__(256) void axpby_kernel(int64_t n, double a, const double *__restrict__ x, double b,
                                                    double *__restrict__ y) {
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; p < n; p += stride)
    y[p] = (b == 0.0 ? 0.0 : b * y[p]) + a * x[p];
}

// z = x + a y
__global__ __launch_bounds__(256) void xpay_kernel(int64_t n, const double *__restrict__ x, double a,
                                                   const double *__restrict__ y, double *__restrict__ z) {
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; p < n; p += stride)
    z[p] = x[p] + a * y[p];
}

// Shape of an apply launch.  Many columns: 64 a block, each thread reading its column's factors from
// memory, bound by the bytes (125,000 columns of 11 levels 24 us; staged in LDS, in pieces of a
// few columns' width, 46 us).  Too few for a block of 64 on each of 256 compute units: the
// latency of the 2 (L+1) dependent steps counts, so the factors are staged with the columns
// (2000 columns 11.5 -> 7.2 us) and the columns spread over up to 512 blocks of at least four.  Both
// (64 bytes a column and level) have to fit 64 KB of LDS for four columns.
struct ApplyShape {
  int cols;
  bool staged;
  size_t lds;
  unsigned blocks;
};
ApplyShape apply_shape(int V, int L) {
  const size_t col = size_t(2) * (L + 1) * sizeof(double), fct = size_t(12) * (L + 1) * sizeof(float);
  ApplyShape a{};
  a.staged = V < 256 * APPLY_COLS && 4 * (col + fct) <= 65536;
  const size_t per = col + (a.staged ? fct : 0);
  a.cols = APPLY_COLS;
  while (a.cols > 1 && a.cols * per > 65536) a.cols /= 2;
  if (a.staged)
    while (a.cols > 4 && (V + a.cols - 1) / a.cols < 512) a.cols /= 2;
  a.lds = a.cols * per;
  a.blocks = unsigned((V + a.cols - 1) / a.cols);
  return a;
}

unsigned grid_for(int64_t n, int block) {
  const int64_t g = (n + block - 1) / block;
  return unsigned(g < 4096 ? (g > 0 ? g : 1) : 4096);
}

}  // namespace

fo_status spmv(const fo_mesh *mesh, const void *vals, int dtype, const double *x, double *y, hipStream_t s) {
  const MeshView &m = mesh->view;
  const int64_t threads = (m.n_dofs / 2) * SPMV_LANES;
  const unsigned blocks = unsigned((threads + 255) / 256);
  if (dtype == FO_F32)
    hipLaunchKernelGGL(spmv_kernel<float>, dim3(blocks), dim3(256), 0, s, m.V, m.L, m.colptr, mesh->nbr_ptr,
                       mesh->nbr_idx, static_cast<const float *>(vals), x, y);
  else
    hipLaunchKernelGGL(spmv_kernel<double>, dim3(blocks), dim3(256), 0, s, m.V, m.L, m.colptr, mesh->nbr_ptr,
                       mesh->nbr_idx, static_cast<const double *>(vals), x, y);
  FO_LAUNCH_CHECK("spmv_kernel");
  return FO_OK;
}

fo_status colblock_factor(const fo_mesh *mesh, const void *vals, int dtype, float *fac, hipStream_t s) {
  const MeshView &m = mesh->view;
  const unsigned blocks = unsigned((m.V + 63) / 64);
  if (dtype == FO_F32)
    hipLaunchKernelGGL((colblock_factor_kernel<float, false>), dim3(blocks), dim3(64), 0, s, m, mesh->self_rank,
                       static_cast<const float *>(vals), fac, nullptr, nullptr);
  else
    hipLaunchKernelGGL((colblock_factor_kernel<double, false>), dim3(blocks), dim3(64), 0, s, m, mesh->self_rank,
                       static_cast<const double *>(vals), fac, nullptr, nullptr);
  FO_LAUNCH_CHECK("colblock_factor_kernel");
  return FO_OK;
}

fo_status colblock_factor_weights(const fo_mesh *mesh, const void *vals, int dtype, float *fac, double *W, float *W32,
                                  hipStream_t s) {
  const MeshView &m = mesh->view;
  // columns per block: their weights and couplings (8 (L+1) doubles per column) within 64 KB of LDS
  const size_t col_bytes = size_t(8) * (m.L + 1) * sizeof(double);
  int cols = 64;
  while (cols > 1 && cols * col_bytes > 65536) cols /= 2;
  const unsigned blocks = unsigned((m.V + cols - 1) / cols);
  if (dtype == FO_F32)
    hipLaunchKernelGGL((colblock_factor_kernel<float, true>), dim3(blocks), dim3(cols), cols * col_bytes, s, m,
                       mesh->self_rank, static_cast<const float *>(vals), fac, W, W32);
  else
    hipLaunchKernelGGL((colblock_factor_kernel<double, true>), dim3(blocks), dim3(cols), cols * col_bytes, s, m,
                       mesh->self_rank, static_cast<const double *>(vals), fac, W, W32);
  FO_LAUNCH_CHECK("colblock_factor_kernel");
  return FO_OK;
}

fo_status colblock_apply(const fo_mesh *mesh, const float *fac, const double *r, double *z, hipStream_t s) {
  const MeshView &m = mesh->view;
  const ApplyShape a = apply_shape(m.V, m.L);
  hipLaunchKernelGGL(a.staged ? colblock_apply_kernel<true> : colblock_apply_kernel<false>, dim3(a.blocks),
                     dim3(APPLY_THREADS), a.lds, s, m.V, m.L, a.cols, fac, r, z);
  FO_LAUNCH_CHECK("colblock_apply_kernel");
  return FO_OK;
}

fo_status colblock_apply_correction(const fo_mesh *mesh, const float *fac, const float *W32, const float *JP,
                                    const double *y, const double *r, double *z, hipStream_t s) {
  const MeshView &m = mesh->view;
  const ApplyShape a = apply_shape(m.V, m.L);
  hipLaunchKernelGGL(a.staged ? colblock_correction_kernel<true> : colblock_correction_kernel<false>, dim3(a.blocks),
                     dim3(APPLY_THREADS), a.lds, s, m.V, m.L, a.cols, mesh->nbr_ptr, mesh->nbr_idx, fac, W32, JP, y, r,
                     z);
  FO_LAUNCH_CHECK("colblock_correction_kernel");
  return FO_OK;
}

// One pair of entries per thread up to 512 blocks (registers leave one wave per SIMD, so those are two
// rounds of the 256 compute units): a solve of 44,000 dofs took 27 us with a block per 4096 entries
// (11 blocks), 6 us with 86.  2.75M dofs: 102 us before, 85 us with all loads of a pass in flight, which
// is 5.7 TB/s.
int multidot_blocks(int64_t n) {
  const int64_t g = (n / 2 + RED_BLOCK - 1) / RED_BLOCK;
  return int(g < 512 ? (g > 0 ? g : 1) : 512);
}

fo_status multidot(int64_t n, const double *V, int64_t ld, int nv, const double *w, double *partial,
                   double *out, double drop, double *host, uint64_t seq, hipStream_t s) {
  if ((n | ld) & 1) return fail(FO_EINVAL, "multidot: vector length and stride must be even");
  if (nv + 2 > kDotsMax) return fail(FO_EINVAL, "multidot: too many vectors");
  const int nb = multidot_blocks(n);
  hipLaunchKernelGGL(multidot_kernel, dim3(nb), dim3(RED_BLOCK), 0, s, n / 2, V, ld, nv, w, partial);
  FO_LAUNCH_CHECK("multidot_kernel");
  hipLaunchKernelGGL(reduce_dots_kernel, dim3(1), dim3(1024), 0, s, nb, nv, partial, drop, out, host, seq);
  FO_LAUNCH_CHECK("reduce_dots_kernel");
  return FO_OK;
}

int dot2_blocks(int64_t n) {
  const int64_t g = (n / 2 + 4 * RED_BLOCK - 1) / (4 * RED_BLOCK);
  return int(g < 2048 ? (g > 0 ? g : 1) : 2048);
}

fo_status dot2(int64_t n, const double *a, const double *w, double *partial, double *out, hipStream_t s) {
  if (n & 1) return fail(FO_EINVAL, "dot2: vector length must be even");
  const int nb = dot2_blocks(n);
  hipLaunchKernelGGL(dot2_kernel, dim3(nb), dim3(RED_BLOCK), 0, s, n / 2, a, w, partial);
  FO_LAUNCH_CHECK("dot2_kernel");
  hipLaunchKernelGGL(reduce_partials_kernel, dim3(2), dim3(256), 0, s, nb, 2, partial, out);
  FO_LAUNCH_CHECK("reduce_partials_kernel");
  return FO_OK;
}

fo_status multiaxpy(int64_t n, const double *V, int64_t ld, int nv, const double *h, const double *scale,
                    const double *w, double *out, double sign, hipStream_t s) {
  if ((n | ld) & 1) return fail(FO_EINVAL, "multiaxpy: vector length and stride must be even");
  const int64_t g = (n / 2 + 255) / 256;
  hipLaunchKernelGGL(multiaxpy_kernel, dim3(unsigned(g < 2048 ? (g > 0 ? g : 1) : 2048)), dim3(256), 0, s, n / 2, V,
                     ld, nv, h, scale, w, out, sign);
  FO_LAUNCH_CHECK("multiaxpy_kernel");
  return FO_OK;
}

fo_status cg_step(int64_t n, const double *num, const double *den, const double *p, const double *q, double *x,
                  double *r, hipStream_t s) {
  hipLaunchKernelGGL(cg_step_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, n, num, den, p, q, x, r);
  FO_LAUNCH_CHECK("cg_step_kernel");
  return FO_OK;
}

fo_status axpby(int64_t n, double a, const double *x, double b, double *y, hipStream_t s) {
  hipLaunchKernelGGL(axpby_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, n, a, x, b, y);
  FO_LAUNCH_CHECK("axpby_kernel");
  return FO_OK;
}

fo_status xpay(int64_t n, const double *x, double a, const double *y, double *z, hipStream_t s) {
  hipLaunchKernelGGL(xpay_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, n, x, a, y, z);
  FO_LAUNCH_CHECK("xpay_kernel");
  return FO_OK;
}

}  // namespace fo
