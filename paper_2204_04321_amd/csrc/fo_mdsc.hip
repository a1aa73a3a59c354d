// Two-level column semicoarsening preconditioner on the device (arXiv:2204.04321 Sec. 3.3:
// vertical coarsening to a single layer with a matrix-dependent prolongator, then aggregation
// AMG on the plane; Sec. 4.4: the prolongator built line by line by LU without pivoting of each
// vertical line's block-tridiagonal system, Chebyshev smoothing on GPUs).
//
// Setup (per Jacobian): the column preconditioner's factors and, in the same kernel, the collapse
// weights W of every column by an FP64 block-tridiagonal solve with two right-hand sides, then
// one pass over J that forms J P0 and the plane operator P0^T J P0 block by block, the plane
// levels' diagonal inverses and Gershgorin bounds, Galerkin sums through precomputed gather
// lists (fixed order, no atomics) and the coarsest inverse in one workgroup's registers.
// Application: restrict with W, a V-cycle over the plane levels (Chebyshev before and after
// each coarse correction, degree 2 on the first plane level and 1 below it, each step one
// kernel that forms the residual it needs), then the column smoother on r - J P0 y fused with
// the prolongation P0 y.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>
#include <vector>

#include "fo_mdsc.h"
#include "fo_solver.h"

namespace fo {
namespace {

constexpr int NC_MAX = 2 * kMdscCoarsestMax;   // most coarsest dofs
constexpr double CHEB_RATIO = 30.0;
enum { FLAG_DIAG = 0, FLAG_COARSE = 1, N_FLAGS = 4 };
// the flags, then the levels' bounds and smoothing coefficients: zeroed together before a setup
constexpr size_t STATUS_BYTES = sizeof(int32_t) * N_FLAGS + sizeof(PlaneCheb) * kMdscMaxLevels;

__device__ __forceinline__ int nlev(int k, int L) { return (k == 0 || k == L) ? 2 : 3; }
__device__ __forceinline__ int cumlev(int k) { return k == 0 ? 0 : 3 * k - 1; }

// 2x2 helpers, [2 r + c]
__device__ __forceinline__ void mul22(const double *a, const double *b, double *o) {
  o[0] = a[0] * b[0] + a[1] * b[2];
  o[1] = a[0] * b[1] + a[1] * b[3];
  o[2] = a[2] * b[0] + a[3] * b[2];
  o[3] = a[2] * b[1] + a[3] * b[3];
}

// One thread per plane block e = (v, neighbour r = w): the rows of J P0 of column v against
// column w, T[(k, c')][d] = sum over the levels l of J_{(v,k,c'),(w,l,d')} W_w[l][d'][d], and
// the block A_0[v][w][c][d] = sum_k sum_c' W_v[k][c'][c] T[(k, c')][d] from the FP64 values.
// J P0 is stored in FP32 by block: entry d of row q of block e at (2 e + d) 2 (L+1) + q (for a
// column, entry (r, d) of row q at (2 (nbr_ptr[v] + r) + d) 2 (L+1) + q), so a workgroup's
// blocks own one contiguous range, staged in LDS and written with coalesced stores.
//
// Its floor is one pass over J.  A thread's rows lie apart, so the next level's values and weights
// are loaded while this level's are used, and the three levels of weights a row meets are kept from
// level to level (875,000 blocks of 10 layers, FP64: 454 -> 244 us; the 0.87 GB of J and 0.2 GB
// written take 213 at the rate of a large copy).
template <class JT>
__global__ __launch_bounds__(256) void plane_kernel(MeshView m, const int32_t *__restrict__ nbr_ptr,
                                                    const int32_t *__restrict__ nbr_idx,
                                                    const int32_t *__restrict__ blk_row, int32_t nnzb,
                                                    const JT *__restrict__ J, const double *__restrict__ W,
                                                    float *__restrict__ JP, double *__restrict__ A0) {
  extern __shared__ float jsh[];   // [blockDim.x][2][2 (L + 1)]
  typedef JT V2 __attribute__((ext_vector_type(2), aligned(alignof(JT))));   // rows start on any value
  const int L = m.L, nb = 2 * (L + 1);
  const int e0 = int(blockIdx.x) * blockDim.x, e = e0 + threadIdx.x;
  const int ne = nnzb - e0 < int(blockDim.x) ? nnzb - e0 : int(blockDim.x);
  if (e < nnzb) {
    const int v = blk_row[e], nb0 = nbr_ptr[v], r = e - nb0, D = nbr_ptr[v + 1] - nb0, w = nbr_idx[e];
    const JT *Jv = J + m.colptr[v];
    const double4 *Wv = reinterpret_cast<const double4 *>(W) + int64_t(v) * (L + 1);
    const double4 *Ww = reinterpret_cast<const double4 *>(W) + int64_t(w) * (L + 1);
    float2 *J0 = reinterpret_cast<float2 *>(jsh + threadIdx.x * 2 * nb), *J1 = J0 + L + 1;
    // a level's two rows against levels k - 1, k, k + 1 of w (zero where there is none)
    auto rows = [&](int k, V2 (&j)[2][3]) {
      const int nl = nlev(k, L);
#pragma unroll
      for (int cp = 0; cp < 2; ++cp) {
        const V2 *p = reinterpret_cast<const V2 *>(Jv + int64_t(4) * D * cumlev(k) + cp * 2 * nl * D + r * 2 * nl);
        j[cp][0] = V2{0, 0};
        j[cp][2] = V2{0, 0};
        if (k > 0) j[cp][0] = *p++;
        j[cp][1] = p[0];
        if (k < L) j[cp][2] = p[1];
      }
    };
    V2 jn[2][3];
    rows(0, jn);
    double4 wl[3] = {make_double4(0, 0, 0, 0), Ww[0], Ww[1]}, wvn = Wv[0];
    double a[4] = {0, 0, 0, 0};
    for (int k = 0; k <= L; ++k) {
      V2 j[2][3];
#pragma unroll
      for (int i = 0; i < 6; ++i) j[i / 3][i % 3] = jn[i / 3][i % 3];
      const double4 wv = wvn;
      double4 wn = wl[2];
      if (k < L) {
        rows(k + 1, jn);
        wvn = Wv[k + 1];
        if (k + 2 <= L) wn = Ww[k + 2];
      }
      double T[4] = {0, 0, 0, 0};
#pragma unroll
      for (int cp = 0; cp < 2; ++cp)
#pragma unroll
        for (int lev = 0; lev < 3; ++lev) {
          const double j0 = double(j[cp][lev].x), j1 = double(j[cp][lev].y);
          T[2 * cp] += j0 * wl[lev].x + j1 * wl[lev].z;
          T[2 * cp + 1] += j0 * wl[lev].y + j1 * wl[lev].w;
        }
      J0[k] = make_float2(float(T[0]), float(T[2]));
      J1[k] = make_float2(float(T[1]), float(T[3]));
      a[0] += wv.x * T[0] + wv.z * T[2];
      a[1] += wv.x * T[1] + wv.z * T[3];
      a[2] += wv.y * T[0] + wv.w * T[2];
      a[3] += wv.y * T[1] + wv.w * T[3];
      wl[0] = wl[1];
      wl[1] = wl[2];
      wl[2] = wn;
    }
    reinterpret_cast<double4 *>(A0)[e] = make_double4(a[0], a[1], a[2], a[3]);
  }
  __syncthreads();
  float *out = JP + int64_t(2) * nb * e0;
  for (int t = threadIdx.x; t < ne * 2 * nb; t += blockDim.x) out[t] = jsh[t];
}

// Diagonal-block inverse of every plane vertex and its Gershgorin row bound
// max over its two rows of sum_w |(D_v^-1 A_vw)| (entries of both columns); g, zero before, becomes
// the largest bound of the level (non-negative doubles order as their bits do, so each workgroup
// adds its own with one integer maximum).  A singular or non-finite block or bound marks the
// setup as failed.  A vertex's blocks are taken by GL lanes (with the maximum in a kernel of one
// workgroup after it: 14 us a level more).
constexpr int GL = 8;
__global__ __launch_bounds__(256) void diag_kernel(int n, const int32_t *__restrict__ ptr,
                                                   const int32_t *__restrict__ diag, const double *__restrict__ A,
                                                   double *__restrict__ Dinv, double *__restrict__ g,
                                                   int32_t *__restrict__ flag) {
  __shared__ double sh[4];
  const int64_t gid = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const int v = int(gid / GL), sub = int(gid % GL);
  double s0 = 0.0, s1 = 0.0, bound = 0.0;
  if (v < n) {
    const double4 a = reinterpret_cast<const double4 *>(A)[diag[v]];
    const double det = a.x * a.w - a.y * a.z;
    const double di[4] = {a.w / det, -a.y / det, -a.z / det, a.x / det};
    for (int e = ptr[v] + sub; e < ptr[v + 1]; e += GL) {
      const double4 b = reinterpret_cast<const double4 *>(A)[e];
      const double bb[4] = {b.x, b.y, b.z, b.w};
      double t[4];
      mul22(di, bb, t);
      s0 += fabs(t[0]) + fabs(t[1]);
      s1 += fabs(t[2]) + fabs(t[3]);
    }
#pragma unroll
    for (int off = GL / 2; off > 0; off >>= 1) {
      s0 += __shfl_xor(s0, off, GL);
      s1 += __shfl_xor(s1, off, GL);
    }
    bool ok = det != 0.0 && isfinite(det);
    for (int i = 0; i < 4; ++i) ok = ok && isfinite(di[i]);
    bound = fmax(s0, s1);
    if (!ok || !isfinite(bound) || !(bound > 0.0)) {
      if (sub == 0) flag[FLAG_DIAG] = 1;
      bound = 0.0;
    }
    if (sub == 0) reinterpret_cast<double4 *>(Dinv)[v] = make_double4(di[0], di[1], di[2], di[3]);
  }
#pragma unroll
  for (int off = 32; off >= GL; off >>= 1) bound = fmax(bound, __shfl_xor(bound, off, 64));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = bound;
  __syncthreads();
  if (threadIdx.x == 0) {
    bound = fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
    // most workgroups find a larger bound there already and leave the one address alone
    auto *gb = reinterpret_cast<unsigned long long *>(g);
    const auto mine = static_cast<unsigned long long>(__double_as_longlong(bound));
    if (mine > __hip_atomic_load(gb, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(gb, mine);
  }
}

// Degree-2 Chebyshev coefficients over [g / ratio, g]: d_0 = D^-1 r_0 / theta and
// d_1 = rho_1 rho_0 d_0 + 2 rho_1 / delta D^-1 r_1.
__device__ __forceinline__ void cheb_coeffs(PlaneCheb &c) {
  const double g = c.g;
  const double lo = g / CHEB_RATIO;
  const double theta = 0.5 * (g + lo), delta = 0.5 * (g - lo);
  const double sigma = theta / delta, rho0 = 1.0 / sigma, rho1 = 1.0 / (2.0 * sigma - rho0);
  c.inv_theta = 1.0 / theta;
  c.c1 = rho1 * rho0;
  c.c2 = 2.0 * rho1 / delta;
}

// Galerkin operator of unsmoothed aggregation: every coarse block is the sum of the fine
// blocks listed for it.  GL lanes share a block, lane i taking every GL-th entry of the list, then
// add their sums in a fixed order (and one forms the fine level's smoothing coefficients): the list's
// indices and the blocks they name are loads that wait for each other, and one lane per block walked
// all of them (all levels of a 125,000-vertex plane: 96 -> 31 us).
__global__ __launch_bounds__(256) void galerkin_kernel(int nnz_c, const int32_t *__restrict__ gptr,
                                                       const int32_t *__restrict__ gidx, const double *__restrict__ Af,
                                                       double *__restrict__ Ac, PlaneCheb *__restrict__ ch) {
  const int64_t gid = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const int c = int(gid / GL), sub = int(gid % GL);
  if (gid == 0) cheb_coeffs(*ch);
  double s[4] = {0, 0, 0, 0};
  if (c < nnz_c)
    for (int i = gptr[c] + sub; i < gptr[c + 1]; i += GL) {
      const double4 b = reinterpret_cast<const double4 *>(Af)[gidx[i]];
      s[0] += b.x;
      s[1] += b.y;
      s[2] += b.z;
      s[3] += b.w;
    }
#pragma unroll
  for (int off = GL / 2; off > 0; off >>= 1)
    for (int i = 0; i < 4; ++i) s[i] += __shfl_xor(s[i], off, GL);
  if (c < nnz_c && sub == 0) reinterpret_cast<double4 *>(Ac)[c] = make_double4(s[0], s[1], s[2], s[3]);
}

// largest of a key over the wave's 64 lanes, in every lane
__device__ __forceinline__ uint32_t wave_max(uint32_t x) {
  auto step = [&](uint32_t y) { x = y > x ? y : x; };
  step(uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0xB1, 0xf, 0xf, true)));    // quad_perm [1,0,3,2]
  step(uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x4E, 0xf, 0xf, true)));    // quad_perm [2,3,0,1]
  step(uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x141, 0xf, 0xf, true)));   // row_half_mirror
  step(uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x140, 0xf, 0xf, true)));   // row_mirror
  const uint32_t r0 = __builtin_amdgcn_readlane(x, 0), r1 = __builtin_amdgcn_readlane(x, 16);
  const uint32_t r2 = __builtin_amdgcn_readlane(x, 32), r3 = __builtin_amdgcn_readlane(x, 48);
  const uint32_t a = r0 > r1 ? r0 : r1, b = r2 > r3 ? r2 : r3;
  return a > b ? a : b;
}

// Inverse of the coarsest operator (nc = 2 n <= NC_MAX dofs) by Gauss-Jordan exchange steps in one
// workgroup: step k takes as pivot the largest entry of column k among the rows not taken yet (by
// its top 25 bits, so within 2^-13 of the largest; the lowest row on ties) and exchanges that row
// with column k.  No row moves: row perm[k] ends as row k of the inverse and column j as its column
// perm[j].  Written column-major.
//
// Bound by the chain of the steps.  Every thread keeps an 8 x 8 part of the matrix (rows and columns
// 16 apart) in registers, so a step passes only the pivot's column and its scaled row through LDS,
// with two barriers; each of the four waves finds the pivot by itself (~110 dofs: 101 us with the
// matrix in LDS and five barriers a step, 90 us as 4 x 4 parts of 1024 threads, which find the
// pivot sixteen times, 64 us now).
constexpr int INV_G = 16, INV_R = NC_MAX / INV_G;   // thread grid, rows and columns per thread
__global__ __launch_bounds__(INV_G *INV_G) void coarse_inverse_kernel(int n, const int32_t *__restrict__ ptr,
                                                                      const int32_t *__restrict__ idx,
                                                                      const double *__restrict__ A,
                                                                      double *__restrict__ Ainv,
                                                                      int32_t *__restrict__ flag) {
  __shared__ double a[NC_MAX * NC_MAX];
  __shared__ double col[2][NC_MAX], row[NC_MAX];
  __shared__ int perm[NC_MAX], rank[NC_MAX];
  const int nc = 2 * n, tid = threadIdx.x, lane = tid & 63, ti = tid / INV_G, tj = tid % INV_G;
  for (int t = tid; t < NC_MAX * NC_MAX; t += INV_G * INV_G) a[t] = 0.0;
  __syncthreads();
  for (int v = tid >> 2; v < n; v += INV_G * INV_G / 4)
    for (int e = ptr[v] + (tid & 3); e < ptr[v + 1]; e += 4) {
      const double4 b = reinterpret_cast<const double4 *>(A)[e];
      double *o = a + 2 * v * NC_MAX + 2 * idx[e];
      o[0] = b.x;
      o[1] = b.y;
      o[NC_MAX] = b.z;
      o[NC_MAX + 1] = b.w;
    }
  __syncthreads();
  double x[INV_R][INV_R];
#pragma unroll
  for (int r = 0; r < INV_R; ++r)
#pragma unroll
    for (int c = 0; c < INV_R; ++c) x[r][c] = a[(ti + INV_G * r) * NC_MAX + tj + INV_G * c];
  bool free0 = lane < nc, free1 = lane + 64 < nc;   // rows lane and lane + 64: not taken yet
#pragma unroll
  for (int kb = 0; kb < INV_R; ++kb)
    for (int kk = 0; kk < INV_G; ++kk) {
      const int k = INV_G * kb + kk;
      if (k >= nc) break;
      double *ck = col[kk & 1];   // in turn: the other waves may still read the last step's
      if (tj == kk)
#pragma unroll
        for (int r = 0; r < INV_R; ++r) {
          ck[ti + INV_G * r] = x[r][kb];
          x[r][kb] = 0.0;
        }
      __syncthreads();
      auto key = [&](int i, bool ok) {
        const uint32_t hi = uint32_t(__double2hiint(ck[i])) & 0x7fffff80u;
        return ok ? hi | 0x80000000u | uint32_t(127 - i) : 0u;
      };
      const uint32_t k0 = key(lane, free0), k1 = key(lane + 64, free1);
      const int p = 127 - int(wave_max(k0 > k1 ? k0 : k1) & 127u);
      free0 = free0 && p != lane;
      free1 = free1 && p != lane + 64;
      const double piv = ck[p];
      if (!(piv != 0.0) || !isfinite(piv)) {   // the same for every thread
        if (tid == 0) flag[FLAG_COARSE] = 1;
        return;
      }
      if (tid == 0) {
        perm[k] = p;
        rank[p] = k;
      }
      const int pr = p / INV_G;
      const bool mine = ti == p % INV_G;
      if (mine) {
        const double inv = 1.0 / piv;
#pragma unroll
        for (int r = 0; r < INV_R; ++r)
          if (r == pr) {   // the same for the wave: a branch, where selects would take 128 instructions
#pragma unroll
            for (int c = 0; c < INV_R; ++c) {
              const double t = c == kb && tj == kk ? 1.0 : x[r][c];
              const double q = t * inv;
              row[tj + INV_G * c] = fma(fma(-piv, q, t), inv, q);   // t / piv to rounding
            }
          }
      }
      __syncthreads();
      double rj[INV_R];
#pragma unroll
      for (int c = 0; c < INV_R; ++c) rj[c] = row[tj + INV_G * c];
#pragma unroll
      for (int r = 0; r < INV_R; ++r) {
        const double f = ck[ti + INV_G * r];
#pragma unroll
        for (int c = 0; c < INV_R; ++c) x[r][c] -= f * rj[c];
      }
      if (mine)
#pragma unroll
        for (int r = 0; r < INV_R; ++r)
          if (r == pr)
#pragma unroll
            for (int c = 0; c < INV_R; ++c) x[r][c] = rj[c];
    }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < INV_R; ++r)
#pragma unroll
    for (int c = 0; c < INV_R; ++c) {
      const int i = ti + INV_G * r, j = tj + INV_G * c;
      if (i < nc && j < nc) Ainv[perm[j] * nc + rank[i]] = x[r][c];
    }
}

// ---- application ------------------------------------------------------------------------

__device__ __forceinline__ double2 apply22(double4 d, double2 x) {
  return make_double2(d.x * x.x + d.y * x.y, d.z * x.x + d.w * x.y);
}

__device__ __forceinline__ double4 diag_inv(const LevelDev &P, int v) {
  return reinterpret_cast<const double4 *>(P.Dinv)[v];
}

// x1 = D^-1 b / theta of vertex v: a smoothed level's first iterate, from zero
__device__ __forceinline__ void store_x1(const LevelDev &P, int v, double2 b) {
  const double it = P.ch->inv_theta;
  const double2 t = apply22(diag_inv(P, v), b);
  reinterpret_cast<double2 *>(P.x1)[v] = make_double2(t.x * it, t.y * it);
}

// b_0[(v, c)] = sum over the column's levels and components of W[v][k][c'][c] r[(v, k, c')], and x1
// of the first level if it is smoothed.  RL lanes share a column, a lane taking every RL-th level:
// 16 bytes of r and of the FP32 weights, whose two columns c sit next to each other for every row
// (125,000 columns of 10 layers: 12.6 us, of which the 46 MB take 9; staged in LDS and summed by a
// thread per (column, c) 15).
constexpr int RL = 4;
__global__ __launch_bounds__(256) void restrict_fine_kernel(LevelDev P, int L, const float *__restrict__ W32,
                                                            const double *__restrict__ r) {
  const int64_t gid = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const int v = int(gid / RL), sub = int(gid % RL);
  double2 s = make_double2(0.0, 0.0);
  if (v < P.n) {
    const float4 *w = reinterpret_cast<const float4 *>(W32) + int64_t(v) * (L + 1);
    const double2 *rv = reinterpret_cast<const double2 *>(r) + int64_t(v) * (L + 1);
#pragma unroll 3
    for (int k = sub; k <= L; k += RL) {
      const float4 wk = w[k];
      const double2 rk = rv[k];
      s.x += double(wk.x) * rk.x + double(wk.z) * rk.y;
      s.y += double(wk.y) * rk.x + double(wk.w) * rk.y;
    }
  }
#pragma unroll
  for (int off = RL / 2; off > 0; off >>= 1) {
    s.x += __shfl_xor(s.x, off, RL);
    s.y += __shfl_xor(s.y, off, RL);
  }
  if (v < P.n && sub == 0) {
    reinterpret_cast<double2 *>(P.b)[v] = s;
    if (P.x1) store_x1(P, v, s);
  }
}

// The V-cycle's kernels.  The first plane level smooths with Chebyshev of degree 2 (x kept
// between the steps), the coarser ones with degree 1.  The pre-smoothed value from zero,
// x1 = D^-1 b / theta, is stored by the kernel that forms b: a neighbour's then costs 16 bytes
// instead of the 48 of its D^-1 and b.  A vertex's row
// blocks are taken by G lanes (consecutive blocks, coalesced 32-byte loads) and summed
// with shuffles; the restriction takes one wave per aggregate.
//
// Bound by the chain of loads (row bounds, neighbours, their values): the operator of a 125,000-vertex
// plane is 28 MB, 6 us at the rate of a large copy.  So the levels' addresses come as kernel
// arguments and the smoothing coefficients from the setup, the vertex's own values are loaded
// before the row, and G = 4 lanes take two blocks each at once, which holds a row of the usual 7 in
// one pass and all rows of that plane on the chip at a time.  With the addresses in memory, the
// coefficients worked out by every thread, 8 lanes and the vertex's values loaded last:
// pre-smoothing 14 -> 9 us, restriction 15 -> 13.6, post-smoothing 14 and 12.4 -> 10.6 and 9.
constexpr int G = 4;

// partial sums of A_vw u_w over this lane's blocks of row v, two blocks' loads in flight
template <class U>
__device__ __forceinline__ double2 row_partial(const LevelDev &P, int v, int sub, U u) {
  double2 s = make_double2(0.0, 0.0);
  const int end = P.ptr[v + 1];
  const double4 *A = reinterpret_cast<const double4 *>(P.A);
  for (int e = P.ptr[v] + sub; e < end; e += 2 * G) {
    const bool two = e + G < end;
    const int f = two ? e + G : e;
    const int w0 = P.idx[e], w1 = P.idx[f];
    const double4 a = A[e], b = A[f];
    const double2 x0 = u(w0), x1 = u(w1);
    s.x += a.x * x0.x + a.y * x0.y;
    s.y += a.z * x0.x + a.w * x0.y;
    s.x += two ? b.x * x1.x + b.y * x1.y : 0.0;
    s.y += two ? b.z * x1.x + b.w * x1.y : 0.0;
  }
  return s;
}

__device__ __forceinline__ double2 group_sum(double2 s) {
#pragma unroll
  for (int off = G / 2; off > 0; off >>= 1) {
    s.x += __shfl_xor(s.x, off, G);
    s.y += __shfl_xor(s.y, off, G);
  }
  return s;
}

// Degree-2 pre-smoothing from x = 0 on the first level: x1 = D^-1 b / theta,
// x = x1 + c1 x1 + c2 D^-1 (b - A x1).
__global__ __launch_bounds__(256) void pre2_kernel(LevelDev P) {
  const int64_t gid = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const int v = int(gid / G), sub = int(gid % G);
  if (v >= P.n) return;   // a whole group
  const PlaneCheb ch = *P.ch;
  const double2 *x1v = reinterpret_cast<const double2 *>(P.x1);
  const double2 b = reinterpret_cast<const double2 *>(P.b)[v], x1 = x1v[v];
  const double4 Dv = diag_inv(P, v);
  const double2 s = group_sum(row_partial(P, v, sub, [&](int w) { return x1v[w]; }));
  if (sub == 0) {
    const double2 ds = apply22(Dv, make_double2(b.x - s.x, b.y - s.y));
    reinterpret_cast<double2 *>(P.x)[v] =
        make_double2(x1.x + (ch.c1 * x1.x + ch.c2 * ds.x), x1.y + (ch.c1 * x1.y + ch.c2 * ds.y));
  }
}

// Residual and restriction in one pass, one wave per aggregate a of the next level:
// b_C[a] = sum over the members v of (b_v - A_v x), x the pre-smoothed vector (x1 for degree 1),
// and x1 of the next level if it is smoothed.  Lanes take (member, block) pairs, 16
// members (most aggregates have 7 to 10) and 8 blocks per pass.
template <int DEG>
__global__ __launch_bounds__(256) void resid_restrict_kernel(LevelDev P, LevelDev C) {
  const int a = int((int64_t(blockIdx.x) * blockDim.x + threadIdx.x) >> 6);
  const int lane = threadIdx.x & 63, mi = lane / G, sub = lane % G;
  double2 s = make_double2(0.0, 0.0);
  if (a < C.n) {
    const double2 *x = reinterpret_cast<const double2 *>(DEG == 2 ? P.x : P.x1);
    for (int i = P.mptr[a] + mi; i < P.mptr[a + 1]; i += 64 / G) {
      const int v = P.midx[i];
      const double2 b = reinterpret_cast<const double2 *>(P.b)[v];
      const double2 t = row_partial(P, v, sub, [&](int w) { return x[w]; });
      s.x += (sub == 0 ? b.x : 0.0) - t.x;
      s.y += (sub == 0 ? b.y : 0.0) - t.y;
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    s.x += __shfl_xor(s.x, off, 64);
    s.y += __shfl_xor(s.y, off, 64);
  }
  if (a < C.n && lane == 0) {
    reinterpret_cast<double2 *>(C.b)[a] = s;
    if (C.x1) store_x1(C, a, s);
  }
}

// Prolongation and the first post-smoothing step: x' = x + x_C[agg], d = D^-1 (b - A x') / theta,
// x_out = x' + d (x' of the neighbours formed on the fly; x is x1 for degree 1).  Degree 2
// writes x2 and d for the second step; degree 1 writes the level's final x.
template <int DEG>
__global__ __launch_bounds__(256) void post0_kernel(LevelDev P, LevelDev C) {
  const int64_t gid = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const int v = int(gid / G), sub = int(gid % G);
  if (v >= P.n) return;   // a whole group
  const PlaneCheb ch = *P.ch;
  const double2 *xv2 = reinterpret_cast<const double2 *>(DEG == 2 ? P.x : P.x1);
  const double2 *xc2 = reinterpret_cast<const double2 *>(C.x);
  auto xp = [&](int w) {
    const double2 xw = xv2[w], cw = xc2[P.agg[w]];
    return make_double2(xw.x + cw.x, xw.y + cw.y);
  };
  const double2 b = reinterpret_cast<const double2 *>(P.b)[v], xo = xp(v);
  const double4 Dv = diag_inv(P, v);
  const double2 s = group_sum(row_partial(P, v, sub, xp));
  if (sub == 0) {
    const double2 dv = apply22(Dv, make_double2(b.x - s.x, b.y - s.y));
    const double dx = dv.x * ch.inv_theta, dy = dv.y * ch.inv_theta;
    const double2 out = make_double2(xo.x + dx, xo.y + dy);
    if constexpr (DEG == 2) {
      reinterpret_cast<double2 *>(P.x2)[v] = out;
      reinterpret_cast<double2 *>(P.d)[v] = make_double2(dx, dy);
    } else {
      reinterpret_cast<double2 *>(P.x)[v] = out;
    }
  }
}

// Second degree-2 post-smoothing step: x = x2 + c1 d + c2 D^-1 (b - A x2).
__global__ __launch_bounds__(256) void post1_kernel(LevelDev P) {
  const int64_t gid = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const int v = int(gid / G), sub = int(gid % G);
  if (v >= P.n) return;   // a whole group
  const PlaneCheb ch = *P.ch;
  const double2 *xv2 = reinterpret_cast<const double2 *>(P.x2);
  const double2 b = reinterpret_cast<const double2 *>(P.b)[v], dv = reinterpret_cast<const double2 *>(P.d)[v];
  const double2 xo = xv2[v];
  const double4 Dv = diag_inv(P, v);
  const double2 s = group_sum(row_partial(P, v, sub, [&](int w) { return xv2[w]; }));
  if (sub == 0) {
    const double2 ds = apply22(Dv, make_double2(b.x - s.x, b.y - s.y));
    reinterpret_cast<double2 *>(P.x)[v] =
        make_double2(xo.x + (ch.c1 * dv.x + ch.c2 * ds.x), xo.y + (ch.c1 * dv.y + ch.c2 * ds.y));
  }
}

// The V-cycle from level P down as one matrix, two columns (of vertex blockIdx.x) per workgroup, from
// the next level's matrix C^T: with b a unit vector, x1 = D^-1 b / theta, x_C = C R (b - A x1),
// x' = x1 + P x_C and x' + D^-1 (b - A x') / theta.  x1 has one vertex and b - A x1 its neighbours
// (the plane graphs are symmetric).  Column-major, dofs n = 2 P.n.
__global__ __launch_bounds__(256) void dense_level_kernel(LevelDev P, int nC, const double *__restrict__ CT,
                                                          double *__restrict__ MT) {
  __shared__ double2 res[2][kMdscDenseMax];   // b - A x1 at the neighbours, per column
  __shared__ double2 xc[2][kMdscDenseMax];    // x_C per column
  const int j = blockIdx.x, tid = threadIdx.x, p0 = P.ptr[j], D = P.ptr[j + 1] - p0;
  const double it = P.ch->inv_theta;
  const double4 Dj = diag_inv(P, j);
  const double2 x1[2] = {make_double2(Dj.x * it, Dj.z * it), make_double2(Dj.y * it, Dj.w * it)};
  const double4 *A = reinterpret_cast<const double4 *>(P.A);
  for (int i = tid; i < D; i += 256) {
    const int w = P.idx[p0 + i];
    double4 a = make_double4(0, 0, 0, 0);
    for (int e = P.ptr[w]; e < P.ptr[w + 1]; ++e)
      if (P.idx[e] == j) a = A[e];
    for (int c = 0; c < 2; ++c)
      res[c][i] = make_double2((w == j && c == 0 ? 1.0 : 0.0) - (a.x * x1[c].x + a.y * x1[c].y),
                               (w == j && c == 1 ? 1.0 : 0.0) - (a.z * x1[c].x + a.w * x1[c].y));
  }
  __syncthreads();
  for (int q = tid; q < nC; q += 256) {
    double2 s[2] = {make_double2(0, 0), make_double2(0, 0)};
    for (int i = 0; i < D; ++i) {
      const int64_t a = 2 * P.agg[P.idx[p0 + i]];
      const double2 m0 = reinterpret_cast<const double2 *>(CT + a * 2 * nC)[q];
      const double2 m1 = reinterpret_cast<const double2 *>(CT + (a + 1) * 2 * nC)[q];
      for (int c = 0; c < 2; ++c) {
        s[c].x += m0.x * res[c][i].x + m1.x * res[c][i].y;
        s[c].y += m0.y * res[c][i].x + m1.y * res[c][i].y;
      }
    }
    xc[0][q] = s[0];
    xc[1][q] = s[1];
  }
  __syncthreads();
  for (int v = tid; v < P.n; v += 256) {
    double2 s[2] = {make_double2(0, 0), make_double2(0, 0)}, xv[2];
    for (int e = P.ptr[v]; e < P.ptr[v + 1]; ++e) {
      const int w = P.idx[e], aw = P.agg[w];
      const double4 a = A[e];
      for (int c = 0; c < 2; ++c) {
        double2 x = xc[c][aw];
        if (w == j) x = make_double2(x.x + x1[c].x, x.y + x1[c].y);
        s[c].x += a.x * x.x + a.y * x.y;
        s[c].y += a.z * x.x + a.w * x.y;
      }
    }
    for (int c = 0; c < 2; ++c) {
      xv[c] = xc[c][P.agg[v]];
      if (v == j) xv[c] = make_double2(xv[c].x + x1[c].x, xv[c].y + x1[c].y);
      const double2 d = apply22(diag_inv(P, v), make_double2((v == j && c == 0 ? 1.0 : 0.0) - s[c].x,
                                                            (v == j && c == 1 ? 1.0 : 0.0) - s[c].y));
      reinterpret_cast<double2 *>(MT)[int64_t(2 * j + c) * P.n + v] =
          make_double2(xv[c].x + d.x * it, xv[c].y + d.y * it);
    }
  }
}

// x = M b for the matrix of a level and all below it, column-major: 16 rows per workgroup, 64 groups of
// lanes over the columns, sums over a wave by shuffles and over the waves in LDS (430 dofs: 4.7 us, in
// place of 14 for that level's two kernels and the coarsest solve).
constexpr int DENSE_ROWS = 16, DENSE_THREADS = 1024;
__global__ __launch_bounds__(DENSE_THREADS) void dense_apply_kernel(LevelDev C, const double *__restrict__ MT) {
  __shared__ double sh[DENSE_THREADS / 64][DENSE_ROWS];
  const int nc = 2 * C.n, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = blockIdx.x * DENSE_ROWS + lane % DENSE_ROWS, ic = i < nc ? i : nc - 1;
  double sum = 0.0;
#pragma unroll 4
  for (int j = threadIdx.x / DENSE_ROWS; j < nc; j += DENSE_THREADS / DENSE_ROWS)
    sum += MT[int64_t(j) * nc + ic] * C.b[j];
#pragma unroll
  for (int off = 32; off >= DENSE_ROWS; off >>= 1) sum += __shfl_xor(sum, off, 64);
  if (lane < DENSE_ROWS) sh[wave][lane] = sum;
  __syncthreads();
  if (threadIdx.x < DENSE_ROWS && i < nc) {
    double t = 0.0;
    for (int w = 0; w < DENSE_THREADS / 64; ++w) t += sh[w][threadIdx.x];
    C.x[i] = t;
  }
}

unsigned blocks_for(int64_t n, int bs) { return unsigned((n + bs - 1) / bs); }

}  // namespace
}  // namespace fo

using namespace fo;

static void free_mdsc(fo_mdsc *p) {
  if (!p) return;
  auto F = [](void *q) { if (q) (void)hipFree(q); };
  for (PlaneLevel &l : p->lv) {
    F(l.own_ptr); F(l.own_idx); F(l.diag); F(l.A); F(l.Dinv); F(l.agg);
    F(l.mptr); F(l.midx); F(l.gptr); F(l.gidx); F(l.b); F(l.x); F(l.x2); F(l.d); F(l.MT);
  }
  F(p->blk_row); F(p->fac); F(p->W); F(p->W32); F(p->JP); F(p->flag);
  if (p->flag_host) (void)hipHostFree(p->flag_host);
  delete p;
}

namespace {
template <class T>
bool dev_alloc(T *&p, size_t count) {
  return hipMalloc(reinterpret_cast<void **>(&p), sizeof(T) * std::max<size_t>(count, 1)) == hipSuccess;
}
template <class T>
bool upload(T *&p, const std::vector<T> &h, hipStream_t s) {
  if (!dev_alloc(p, h.size())) return false;
  return h.empty() || hipMemcpyAsync(p, h.data(), sizeof(T) * h.size(), hipMemcpyHostToDevice, s) == hipSuccess;
}
}  // namespace

extern "C" fo_status fo_mdsc_create(const fo_mesh *m, void *stream, fo_mdsc **out) {
  if (!out) return fail(FO_EINVAL, "fo_mdsc_create: out is NULL");
  *out = nullptr;
  if (!m) return fail(FO_EINVAL, "fo_mdsc_create: mesh is NULL");
  int dev = -1;
  FO_HIP_TRY(hipGetDevice(&dev));
  if (dev != m->device) return fail(FO_EINVAL, "fo_mdsc_create: the mesh's device must be current");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int V = m->view.V, L = m->view.L;
  std::vector<int32_t> ptr(static_cast<size_t>(V) + 1), self(static_cast<size_t>(V));
  FO_HIP_TRY(hipStreamSynchronize(s));
  FO_HIP_TRY(hipMemcpy(ptr.data(), m->nbr_ptr, sizeof(int32_t) * (V + 1), hipMemcpyDeviceToHost));
  std::vector<int32_t> idx(static_cast<size_t>(ptr[V]));
  FO_HIP_TRY(hipMemcpy(idx.data(), m->nbr_idx, sizeof(int32_t) * ptr[V], hipMemcpyDeviceToHost));
  FO_HIP_TRY(hipMemcpy(self.data(), m->self_rank, sizeof(int32_t) * V, hipMemcpyDeviceToHost));

  fo_mdsc *p = new fo_mdsc();
  p->mesh = m;
  p->device = dev;
  auto bail = [&](fo_status st, const std::string &msg) { free_mdsc(p); return fail(st, msg); };
  // symbolic hierarchy on the host
  std::vector<PlaneTables> tabs;
  p->lv.emplace_back();
  p->lv[0].ptr_h = ptr;
  p->lv[0].idx_h = idx;
  while (p->lv.back().ptr_h.size() - 1 > size_t(kMdscCoarsestMax)) {
    if (int(p->lv.size()) >= kMdscMaxLevels) return bail(FO_EINVAL, "fo_mdsc_create: aggregation did not coarsen");
    PlaneLevel &f = p->lv.back();
    const int32_t n_agg = aggregate_graph(f.ptr_h, f.idx_h, f.agg_h);
    tabs.emplace_back();
    coarse_tables(f.ptr_h, f.idx_h, f.agg_h, n_agg, tabs.back());
    PlaneLevel c;
    c.ptr_h = tabs.back().cptr;
    c.idx_h = tabs.back().cidx;
    p->lv.push_back(std::move(c));
  }
  const size_t last = p->lv.size() - 1;
  // the first level that a matrix of its own stands for, with all below it
  p->dense = int(last);
  while (p->dense > 1 && p->lv[p->dense - 1].ptr_h.size() - 1 <= size_t(kMdscDenseMax)) --p->dense;
  // device arrays
  if (!dev_alloc(p->flag, STATUS_BYTES / sizeof(int32_t)))
    return bail(FO_ENOMEM, "fo_mdsc_create: device allocation failed");
  for (size_t l = 0; l <= last; ++l) {
    PlaneLevel &q = p->lv[l];
    q.n = int32_t(q.ptr_h.size()) - 1;
    q.nnzb = q.ptr_h[q.n];
    std::vector<int32_t> diag(static_cast<size_t>(q.n));
    for (int32_t v = 0; v < q.n; ++v)
      diag[v] = l == 0 ? ptr[v] + self[v]
                       : int32_t(std::lower_bound(q.idx_h.begin() + q.ptr_h[v], q.idx_h.begin() + q.ptr_h[v + 1], v) -
                                 q.idx_h.begin());
    bool ok = true;
    if (l == 0) {
      q.ptr = m->nbr_ptr;
      q.idx = m->nbr_idx;
    } else {
      ok = ok && upload(q.own_ptr, q.ptr_h, s) && upload(q.own_idx, q.idx_h, s);
      q.ptr = q.own_ptr;
      q.idx = q.own_idx;
    }
    ok = ok && upload(q.diag, diag, s) && dev_alloc(q.A, 4 * size_t(q.nnzb)) && dev_alloc(q.b, 2 * size_t(q.n)) &&
         dev_alloc(q.x, 2 * size_t(q.n));
    if (l < last) {
      const PlaneTables &t = tabs[l];
      q.ch = reinterpret_cast<PlaneCheb *>(p->flag + N_FLAGS) + l;
      ok = ok && dev_alloc(q.Dinv, 4 * size_t(q.n)) &&
           (int(l) >= p->dense || dev_alloc(q.x2, 2 * size_t(q.n))) && (l > 0 || dev_alloc(q.d, 2 * size_t(q.n))) &&
           (int(l) < p->dense || dev_alloc(q.MT, 4 * size_t(q.n) * size_t(q.n))) &&
           upload(q.agg, q.agg_h, s) && upload(q.mptr, t.mptr, s) && upload(q.midx, t.midx, s) &&
           upload(q.gptr, t.gptr, s) && upload(q.gidx, t.gidx, s);
    }
    if (!ok) return bail(FO_ENOMEM, "fo_mdsc_create: device allocation failed");
  }
  std::vector<int32_t> blk_row(static_cast<size_t>(ptr[V]));
  for (int32_t v = 0; v < V; ++v)
    for (int32_t e = ptr[v]; e < ptr[v + 1]; ++e) blk_row[e] = v;
  const size_t nodes = size_t(V) * size_t(L + 1);
  const int nc = 2 * p->lv[last].n;
  p->jp_count = size_t(2 * (L + 1)) * 2 * size_t(ptr[V]);
  if (!upload(p->blk_row, blk_row, s) || !dev_alloc(p->fac, 12 * nodes) || !dev_alloc(p->W, 4 * nodes) ||
      !dev_alloc(p->W32, 4 * nodes) || !dev_alloc(p->JP, p->jp_count) || !dev_alloc(p->lv[last].MT, size_t(nc) * nc))
    return bail(FO_ENOMEM, "fo_mdsc_create: device allocation failed");
  if (hipHostMalloc(reinterpret_cast<void **>(&p->flag_host), sizeof(int32_t) * N_FLAGS) != hipSuccess)
    return bail(FO_ENOMEM, "fo_mdsc_create: pinned allocation failed");
  if (hipStreamSynchronize(s) != hipSuccess) return bail(FO_EDEVICE, "fo_mdsc_create: upload failed");
  *out = p;
  return FO_OK;
}

extern "C" void fo_mdsc_destroy(fo_mdsc *p) { free_mdsc(p); }

extern "C" fo_status fo_mdsc_levels(const fo_mdsc *p, int32_t *n_levels, int32_t *n_verts) {
  if (!p) return fail(FO_EINVAL, "fo_mdsc_levels: NULL object");
  if (n_levels) *n_levels = int32_t(p->lv.size()) - 1;
  if (n_verts)
    for (size_t l = 0; l < p->lv.size(); ++l) n_verts[l] = p->lv[l].n;
  return FO_OK;
}

extern "C" fo_status fo_mdsc_graph(const fo_mdsc *p, int32_t level, int32_t *ptr, int32_t *idx, int32_t *agg) {
  if (!p || level < 0 || level >= int32_t(p->lv.size())) return fail(FO_EINVAL, "fo_mdsc_graph: bad object or level");
  const PlaneLevel &q = p->lv[level];
  if (agg && level == int32_t(p->lv.size()) - 1) return fail(FO_EINVAL, "fo_mdsc_graph: the coarsest level has no aggregates");
  if (ptr) std::copy(q.ptr_h.begin(), q.ptr_h.end(), ptr);
  if (idx) std::copy(q.idx_h.begin(), q.idx_h.end(), idx);
  if (agg) std::copy(q.agg_h.begin(), q.agg_h.end(), agg);
  return FO_OK;
}

namespace {
// What the kernels read of a level.  x1 shares x2, which the first level writes only after its last use.
LevelDev view(const PlaneLevel &q) {
  return LevelDev{q.n, q.ptr, q.idx, q.agg, q.mptr, q.midx, q.A, q.Dinv, q.ch, q.b, q.x, q.x2, q.x2, q.d};
}

template <class JT>
fo_status setup_t(fo_mdsc *p, const JT *J, hipStream_t s) {
  const fo_mesh *m = p->mesh;
  const MeshView &mv = m->view;
  const PlaneLevel &l0 = p->lv[0];
  // blocks per workgroup: their J P0 rows (4 (L+1) floats each) within 64 KB of LDS
  const size_t blk_bytes = size_t(4) * (mv.L + 1) * sizeof(float);
  int tpb = 256;
  while (tpb > 1 && tpb * blk_bytes > 65536) tpb /= 2;
  hipLaunchKernelGGL(plane_kernel<JT>, dim3(blocks_for(l0.nnzb, tpb)), dim3(tpb), tpb * blk_bytes, s, mv, m->nbr_ptr,
                     m->nbr_idx, p->blk_row, l0.nnzb, J, p->W, p->JP, l0.A);
  FO_LAUNCH_CHECK("mdsc plane");
  return FO_OK;
}
}  // namespace

extern "C" fo_status fo_mdsc_setup(fo_mdsc *p, const void *J, int32_t dtype, void *stream) {
  if (!p || !J) return fail(FO_EINVAL, "fo_mdsc_setup: NULL argument");
  if (dtype != FO_F64 && dtype != FO_F32) return fail(FO_EINVAL, "fo_mdsc_setup: bad dtype");
  hipStream_t s = static_cast<hipStream_t>(stream);
  p->ready = false;
  fo_status st;
  if ((st = launch_fill_zero(p->flag, STATUS_BYTES, s)) != FO_OK) return st;
  if ((st = colblock_factor_weights(p->mesh, J, dtype, p->fac, p->W, p->W32, s)) != FO_OK) return st;
  st = dtype == FO_F64 ? setup_t(p, static_cast<const double *>(J), s) : setup_t(p, static_cast<const float *>(J), s);
  if (st != FO_OK) return st;
  const size_t last = p->lv.size() - 1;
  for (size_t l = 0; l < last; ++l) {
    PlaneLevel &q = p->lv[l];
    hipLaunchKernelGGL(diag_kernel, dim3(blocks_for(int64_t(q.n) * GL, 256)), dim3(256), 0, s, q.n, q.ptr, q.diag, q.A,
                       q.Dinv, &q.ch->g, p->flag);
    FO_LAUNCH_CHECK("mdsc diag");
    const PlaneLevel &c = p->lv[l + 1];
    hipLaunchKernelGGL(galerkin_kernel, dim3(blocks_for(int64_t(c.nnzb) * GL, 256)), dim3(256), 0, s, c.nnzb,
                       q.gptr, q.gidx, q.A, c.A, q.ch);
    FO_LAUNCH_CHECK("mdsc galerkin");
  }
  const PlaneLevel &c = p->lv[last];
  hipLaunchKernelGGL(coarse_inverse_kernel, dim3(1), dim3(INV_G * INV_G), 0, s, c.n, c.ptr, c.idx, c.A, c.MT,
                     p->flag);
  FO_LAUNCH_CHECK("mdsc coarse inverse");
  for (int l = int(last) - 1; l >= p->dense; --l) {
    hipLaunchKernelGGL(dense_level_kernel, dim3(p->lv[l].n), dim3(256), 0, s, view(p->lv[l]), p->lv[l + 1].n,
                       p->lv[l + 1].MT, p->lv[l].MT);
    FO_LAUNCH_CHECK("mdsc dense level");
  }
  FO_HIP_TRY(hipMemcpyAsync(p->flag_host, p->flag, sizeof(int32_t) * N_FLAGS, hipMemcpyDeviceToHost, s));
  FO_HIP_TRY(hipStreamSynchronize(s));
  if (p->flag_host[FLAG_DIAG])
    return fail(FO_ENONFINITE, "fo_mdsc_setup: a plane diagonal block is singular or not finite");
  if (p->flag_host[FLAG_COARSE])
    return fail(FO_ENONFINITE, "fo_mdsc_setup: the coarsest plane operator is singular or not finite");
  p->ready = true;
  return FO_OK;
}

extern "C" fo_status fo_mdsc_apply(const fo_mdsc *p, const double *r, double *z, void *stream) {
  if (!p || !r || !z || r == z) return fail(FO_EINVAL, "fo_mdsc_apply: NULL or aliased vectors");
  if ((reinterpret_cast<uintptr_t>(r) & 15) || (reinterpret_cast<uintptr_t>(z) & 15))
    return fail(FO_EINVAL, "fo_mdsc_apply: vectors must be 16-byte aligned");
  if (!p->ready) return fail(FO_EINVAL, "fo_mdsc_apply: no successful fo_mdsc_setup");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const MeshView &mv = p->mesh->view;
  const PlaneLevel &l0 = p->lv[0];
  const int nd = p->dense;
  hipLaunchKernelGGL(restrict_fine_kernel, dim3(blocks_for(int64_t(mv.V) * RL, 256)), dim3(256), 0, s, view(l0), mv.L,
                     p->W32, r);
  FO_LAUNCH_CHECK("mdsc restrict");
  // level 0 smooths with degree 2, the coarser levels with degree 1
  for (int l = 0; l < nd; ++l) {
    const LevelDev P = view(p->lv[l]), C = view(p->lv[l + 1]);
    const unsigned gv = blocks_for(int64_t(P.n) * G, 256), ga = blocks_for(int64_t(C.n) * 64, 256);
    if (l == 0) {
      hipLaunchKernelGGL(pre2_kernel, dim3(gv), dim3(256), 0, s, P);
      hipLaunchKernelGGL(resid_restrict_kernel<2>, dim3(ga), dim3(256), 0, s, P, C);
    } else {
      hipLaunchKernelGGL(resid_restrict_kernel<1>, dim3(ga), dim3(256), 0, s, P, C);
    }
    FO_LAUNCH_CHECK("mdsc pre-smoothing");
  }
  hipLaunchKernelGGL(dense_apply_kernel, dim3(blocks_for(2 * p->lv[nd].n, DENSE_ROWS)), dim3(DENSE_THREADS), 0, s,
                     view(p->lv[nd]), p->lv[nd].MT);
  FO_LAUNCH_CHECK("mdsc dense solve");
  for (int l = nd - 1; l >= 0; --l) {
    const LevelDev P = view(p->lv[l]), C = view(p->lv[l + 1]);
    const unsigned gv = blocks_for(int64_t(P.n) * G, 256);
    if (l == 0) {
      hipLaunchKernelGGL(post0_kernel<2>, dim3(gv), dim3(256), 0, s, P, C);
      hipLaunchKernelGGL(post1_kernel, dim3(gv), dim3(256), 0, s, P);
    } else {
      hipLaunchKernelGGL(post0_kernel<1>, dim3(gv), dim3(256), 0, s, P, C);
    }
    FO_LAUNCH_CHECK("mdsc post-smoothing");
  }
  return colblock_apply_correction(p->mesh, p->fac, p->W32, p->JP, l0.x, r, z, s);
}

extern "C" fo_status fo_mdsc_export(const fo_mdsc *p, int32_t what, int32_t level, double *host, size_t count,
                                    void *stream) {
  if (!p || !host) return fail(FO_EINVAL, "fo_mdsc_export: NULL argument");
  if (!p->ready) return fail(FO_EINVAL, "fo_mdsc_export: no successful fo_mdsc_setup");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const double *src = nullptr;
  size_t n = 0;
  const int32_t nl = int32_t(p->lv.size());
  if (what == FO_MDSC_WEIGHTS) {
    src = p->W;
    n = 4 * size_t(p->mesh->view.V) * size_t(p->mesh->view.L + 1);
  } else if (what == FO_MDSC_PLANE && level >= 0 && level < nl) {
    src = p->lv[level].A;
    n = 4 * size_t(p->lv[level].nnzb);
  } else if (what == FO_MDSC_BOUND && level >= 0 && level < nl - 1) {
    src = &p->lv[level].ch->g;
    n = 1;
  } else {
    return fail(FO_EINVAL, "fo_mdsc_export: bad field or level");
  }
  if (count != n) return fail(FO_EINVAL, "fo_mdsc_export: count must be " + std::to_string(n));
  FO_HIP_TRY(hipMemcpyAsync(host, src, sizeof(double) * n, hipMemcpyDeviceToHost, s));
  FO_HIP_TRY(hipStreamSynchronize(s));
  return FO_OK;
}
