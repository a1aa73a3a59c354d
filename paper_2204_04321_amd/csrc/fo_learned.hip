// Learned Newton initial guess: per-column features, a 10-128-128-128-22 tanh MLP whose
// products run on gfx950 BF16 matrix cores (v_mfma_f32_16x16x32_bf16, FP32 accumulation),
// its backward pass, MSE gradient and Adam, and the guess itself with its shallow-ice
// fallback.  Not part of the paper: the network only supplies the starting point of the
// damped Newton solve of Sec. 3.1 (eq. linearsystem).
//
// Rounding points: products take BF16 (round to nearest even) copies of inputs, weights,
// hidden activations and backpropagated errors; sums are FP32; biases, tanh and its
// derivative use the unrounded FP32 values.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>

#include "fo_device.h"
#include "fo_internal.h"
#include "fo_solver.h"

namespace fo {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int NIN = 10, NH = 128, NOUT = 22;
constexpr int LAY[5] = {NIN, NH, NH, NH, NOUT};

// offsets of W_l ([out][in]) and b_l ([out]) in the flat FP32 parameter vector
constexpr int woff(int l) { int o = 0; for (int i = 0; i < l; ++i) o += LAY[i] * LAY[i + 1] + LAY[i + 1]; return o; }
constexpr int boff(int l) { return woff(l) + LAY[l] * LAY[l + 1]; }
constexpr int NPARAM = woff(4);

// ---- column features --------------------------------------------------------------------
// VERT_LANES lanes share a vertex: a cell of the surface gradient each, then a neighbour each (every
// eighth where there are more), of which the group picks the nearest in turn; lane r keeps the r-th
// and works out its angle.  Bound by that chain (2,000 vertices: 31 us with a thread per vertex, 10.6
// now).  `clear`, where given, is set to 0 for a later kernel.
__global__ __launch_bounds__(64) void features_kernel(MeshView m, const int32_t *__restrict__ nbr_ptr,
                                                      const int32_t *__restrict__ nbr_idx,
                                                      const int32_t *__restrict__ vc_ptr,
                                                      const int32_t *__restrict__ vc_idx,
                                                      const float *__restrict__ norm, float *__restrict__ F,
                                                      int *__restrict__ clear) {
  constexpr int G = VERT_LANES;
  const int64_t gid = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const int v = int(gid / G), sub = int(gid % G);
  if (clear && gid == 0) *clear = 0;
  if (v >= m.V) return;   // all lanes of a vertex
  const double4 gv = m.geo[v];
  const double Hv = gv.w;
  const double beta = m.sb[v].y;
  const int p0 = nbr_ptr[v], p1 = nbr_ptr[v + 1];
  auto dist2 = [&](int w) {
    const double4 g = m.geo[w];
    const double dx = g.x - gv.x, dy = g.y - gv.y;
    return dx * dx + dy * dy;
  };
  const int w0 = p0 + sub < p1 ? nbr_idx[p0 + sub] : v;   // the lane's first neighbour
  const double d0 = dist2(w0);
  double gx, gy;
  vertex_surface_gradient(m, vc_ptr, vc_idx, v, sub, gx, gy);
  // the 6 nearest neighbours (distance, then index), ordered by angle from -grad s
  int sel = -1, nsel = 0;
  double last_d2 = -1.0;
  int last_w = -1;
  for (int r = 0; r < 6; ++r) {
    double best_d2 = 0.0;
    int best_w = -1;
    auto consider = [&](int w, double d2) {
      const bool after = d2 > last_d2 || (d2 == last_d2 && w > last_w);
      const bool better = best_w < 0 || d2 < best_d2 || (d2 == best_d2 && w < best_w);
      if (w != v && after && better) { best_d2 = d2; best_w = w; }
    };
    consider(w0, d0);
    for (int p = p0 + G + sub; p < p1; p += G) consider(nbr_idx[p], dist2(nbr_idx[p]));
#pragma unroll
    for (int off = 1; off < G; off <<= 1) {
      const double od = __shfl_xor(best_d2, off, G);
      const int ow = __shfl_xor(best_w, off, G);
      if (ow >= 0 && (best_w < 0 || od < best_d2 || (od == best_d2 && ow < best_w))) { best_d2 = od; best_w = ow; }
    }
    if (best_w < 0) break;
    if (sub == r) sel = best_w;
    ++nsel;
    last_d2 = best_d2;
    last_w = best_w;
  }
  const double ref = (gx != 0.0 || gy != 0.0) ? atan2(-gy, -gx) : 0.0;
  const double twopi = 6.283185307179586476925286766559;
  double ang = 0.0, Hs = 0.0;
  if (sub < nsel) {
    const double4 g = m.geo[sel];
    ang = fmod(atan2(g.y - gv.y, g.x - gv.x) - ref, twopi);
    if (ang < 0) ang += twopi;
    Hs = g.w;
  }
  int rank = 0;   // by (angle, index)
  for (int i = 0; i < nsel; ++i) {
    const double ai = __shfl(ang, i, G);
    const int wi = __shfl(sel, i, G);
    rank += ai < ang || (!(ang < ai) && (ai == ang ? wi < sel : i < sub)) ? 1 : 0;
  }
  double mine = Hv;   // lane j: the j-th of that order
  for (int i = 0; i < nsel; ++i) {
    const double h = __shfl(Hs, i, G);
    if (__shfl(rank, i, G) == sub) mine = h;
  }
  float *Fv = F + int64_t(v) * 10;
  auto put = [&](int i, double f) {
    Fv[i] = float(norm ? (f - double(norm[i])) / double(norm[10 + i]) : f);
  };
  if (sub < 4) put(sub, sub == 0 ? Hv : sub == 1 ? gx : sub == 2 ? gy : log(beta > 1e-3 ? beta : 1e-3));
  if (sub < 6) put(4 + sub, mine);
}

// ---- the network on BF16 matrix cores -------------------------------------------------------
// Both passes run whole row tiles of the batch through all layers in one kernel of eight waves:
// wave w owns output columns 16 w .. 16 w + 15 of every 128-wide layer and keeps that layer's
// weight fragments in registers for all of its block's tiles, so the weights are read once per
// block and the activations of a tile pass from layer to layer through LDS.  Fragments of
// v_mfma_f32_16x16x32_bf16: lane (r = l % 16, q = l / 16) supplies A row r and B column r at
// k = 8 q .. 8 q + 7 of each 32-block and receives C rows 4 q .. 4 q + 3 of column r.  K is
// consumed 32 at a time in ascending order.
constexpr int MLP_WAVES = 8, MLP_THREADS = 64 * MLP_WAVES;
constexpr int FWD_ROWS = 16, BWD_ROWS = 32;
constexpr int LDA = NH + 8;          // BF16 row stride of a tile in LDS: 16-byte aligned rows, banks shifted
constexpr int LDT = BWD_ROWS + 8;    // row stride of a transposed tile

__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Eight consecutive entries k0 .. k0 + 7 of a row of length K, zero from K on
__device__ __forceinline__ bf16x8 row_frag(const float *__restrict__ row, int k0, int K) {
  bf16x8 f;
#pragma unroll
  for (int j = 0; j < 8; ++j) f[j] = k0 + j < K ? __bf16(row[k0 + j]) : __bf16(0.f);
  return f;
}

// Eight consecutive entries (at an address that is only 4-byte aligned), two 16-byte loads
__device__ __forceinline__ bf16x8 full_frag(const float *__restrict__ p) {
  float v[8];
  __builtin_memcpy(v, p, sizeof v);
  bf16x8 f;
#pragma unroll
  for (int j = 0; j < 8; ++j) f[j] = __bf16(v[j]);
  return f;
}

// Y = W_3 tanh(W_2 tanh(W_1 tanh(W_0 x + b_0) + b_1) + b_2) + b_3 over tiles of 16 rows.  Bound
// by the latency of a tile's four dependent layers and, for large batches, by the stores of the
// activations (1.6 KB a row); 16 rows a tile so that a batch of 4096 fills the 256 compute
// units.  acts may be NULL (inference).  Measured against one GEMM launch per layer: 33 -> 10 us
// (512 rows), 49 -> 11 us (4096), 539 -> 47 us (65536).
__global__ __launch_bounds__(MLP_THREADS, 4) void mlp_forward_kernel(const float *__restrict__ P,
                                                                     const float *__restrict__ X, int B,
                                                                     float *__restrict__ acts,
                                                                     float *__restrict__ Y) {
  __shared__ __align__(16) __bf16 tile[2][FWD_ROWS * LDA];
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63, r = l & 15, q = l >> 4;
  const int n = 16 * wave + r;
  const bool head = 16 * wave < NOUT;            // the waves of the output layer
  const bool out_col = head && n < NOUT;
  bf16x8 w0 = row_frag(P + woff(0) + n * NIN, 8 * q, NIN), w1[4], w2[4], w3[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    w1[j] = full_frag(P + woff(1) + n * NH + 32 * j + 8 * q);
    w2[j] = full_frag(P + woff(2) + n * NH + 32 * j + 8 * q);
    w3[j] = full_frag(P + woff(3) + (out_col ? n : 0) * NH + 32 * j + 8 * q);   // other columns are not stored
  }
  const float b0 = P[boff(0) + n], b1 = P[boff(1) + n], b2 = P[boff(2) + n], b3 = out_col ? P[boff(3) + n] : 0.f;
  const int tiles = (B + FWD_ROWS - 1) / FWD_ROWS;
  int buf = 0;
  for (int t = blockIdx.x; t < tiles; t += gridDim.x) {
    const int64_t m0 = int64_t(t) * FWD_ROWS;
    const int rows = B - m0 < FWD_ROWS ? int(B - m0) : FWD_ROWS;
    bf16x8 x = row_frag(X + (m0 + (r < rows ? r : 0)) * NIN, 8 * q, r < rows ? NIN : 0);
    f32x4 acc = mfma(x, w0, f32x4{0.f, 0.f, 0.f, 0.f});
    // a layer's tanh, stored for the backward pass and passed on in BF16
    auto hidden = [&](int layer, float bias) {
      __bf16 *dst = tile[buf];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int m = 4 * q + i;
        const float a = tanhf(acc[i] + bias);
        if (acts && m < rows) acts[(int64_t(layer) * B + m0 + m) * NH + n] = a;
        dst[m * LDA + n] = m < rows ? __bf16(a) : __bf16(0.f);
      }
      __syncthreads();
    };
    auto layer = [&](const bf16x8 *w) {
      const __bf16 *src = tile[buf] + r * LDA + 8 * q;
      acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < 4; ++j) acc = mfma(*reinterpret_cast<const bf16x8 *>(src + 32 * j), w[j], acc);
      buf ^= 1;
    };
    hidden(0, b0);
    layer(w1);
    hidden(1, b1);
    layer(w2);
    hidden(2, b2);
    if (head) {
      layer(w3);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (out_col && 4 * q + i < rows) Y[(m0 + 4 * q + i) * NOUT + n] = acc[i] + b3;
    } else {
      buf ^= 1;
    }
  }
}

// The 32 batch rows of a tile as the k of a weight gradient: element j of lane q is row
// 4 q + j (j < 4) or 16 + 4 q + j - 4, the rows that the same lane holds of two stacked
// 16-row accumulators, so a wave's own backpropagated errors and activations are fragments
// without any exchange.
__device__ __forceinline__ int tile_row(int q, int j) { return j < 4 ? 4 * q + j : 12 + 4 * q + j; }

// Gradients of all layers over tiles of 32 rows: the errors dZ_2, dZ_1, dZ_0 pass from layer to
// layer through LDS in BF16, and each tile adds its 32-row products to the block's weight
// gradients, held in accumulators (up to 76 registers a lane) until the block's last tile.  HI: the
// sums of layers 2 and 3, LO: of layers 0 and 1; a block forms one half or both (backward_plan) and
// writes its sums to its part of the scratch, or to the gradients when it is the only one; the
// blocks' sums are added by mlp_reduce_kernel in block order.  Bound by the latency of a tile
// (three dependent layers, two barriers), so a tile's loads are issued ahead of the chain.
// Measured, with the sum over the blocks, against one wave per 16x16 tile of each weight gradient
// walking the whole batch: 230 -> 30 us (512 rows), 2333 -> 27 us (4096), 36.7 ms -> 73 us (65536).
constexpr int64_t SPLIT_BELOW = 192;   // blocks of all layers that the scratch holds (backward_plan)

struct BackwardLds {
  __align__(16) __bf16 err[2][BWD_ROWS * LDA];       // dZ_2, dZ_1 by row
  __align__(16) __bf16 actT[2][2][NH * LDT];         // [tile parity][layer 0, 1]: activations by column
};

template <bool HI, bool LO>
__device__ __forceinline__ void backward_tiles(const float *__restrict__ P, const float *__restrict__ X, int B,
                                               const float *__restrict__ acts, const float *__restrict__ dY,
                                               float *__restrict__ G, BackwardLds &S, int block, int blocks) {
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63, r = l & 15, q = l >> 4;
  const int n = 16 * wave + r;
  // W_l as the right operand of dZ_l W_l: k over the layer's outputs, column n of its inputs
  bf16x8 w3, w2[4], w1[4];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int k = 8 * q + e;
    w3[e] = k < NOUT ? __bf16(P[woff(3) + k * NH + n]) : __bf16(0.f);
#pragma unroll
    for (int j = 0; LO && j < 4; ++j) {
      w2[j][e] = __bf16(P[woff(2) + (32 * j + k) * NH + n]);
      w1[j][e] = __bf16(P[woff(1) + (32 * j + k) * NH + n]);
    }
  }
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 g3[2] = {zero, zero}, g2[8], g1[8], g0 = zero;
#pragma unroll
  for (int t = 0; t < 8; ++t) g2[t] = g1[t] = zero;
  float s3[2] = {0.f, 0.f}, s2 = 0.f, s1 = 0.f, s0 = 0.f;       // bias gradients: this lane's rows
  const int tiles = (B + BWD_ROWS - 1) / BWD_ROWS;
  int par = 0;
  for (int t = block; t < tiles; t += blocks, par ^= 1) {
    const int64_t m0 = int64_t(t) * BWD_ROWS;
    const int rows = B - m0 < BWD_ROWS ? int(B - m0) : BWD_ROWS;
    float a2[8], a1[8], a0[8];
    bf16x8 x, y[2];                       // right operand X, left operand dY^T (outputs 0-15, 16-21)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int m = tile_row(q, j);
      const bool in = m < rows;
      const int64_t mm = m0 + (in ? m : 0);
      const float *am = acts + mm * NH + n;
      a2[j] = in ? am[2 * int64_t(B) * NH] : 0.f;
      a1[j] = in ? am[int64_t(B) * NH] : 0.f;
      if constexpr (LO) {
        a0[j] = in ? am[0] : 0.f;
        x[j] = in && r < NIN ? __bf16(X[mm * NIN + (r < NIN ? r : 0)]) : __bf16(0.f);
      }
      if constexpr (!HI) continue;
      const float y0 = in ? dY[mm * NOUT + r] : 0.f;
      const float y1 = in && 16 + r < NOUT ? dY[mm * NOUT + (16 + r < NOUT ? 16 + r : 0)] : 0.f;
      s3[0] += y0;
      s3[1] += y1;
      y[0][j] = __bf16(y0);
      y[1][j] = __bf16(y1);
    }
    auto bf16_of = [](const float *v) {
      bf16x8 h;
#pragma unroll
      for (int j = 0; j < 8; ++j) h[j] = __bf16(v[j]);
      return h;
    };
    if constexpr (LO) *reinterpret_cast<bf16x8 *>(&S.actT[par][0][n * LDT + 8 * q]) = bf16_of(a0);
    if constexpr (HI) {
      *reinterpret_cast<bf16x8 *>(&S.actT[par][1][n * LDT + 8 * q]) = bf16_of(a1);
      const bf16x8 h2 = bf16_of(a2);
      g3[0] = mfma(y[0], h2, g3[0]);
      g3[1] = mfma(y[1], h2, g3[1]);
    }
    // dZ = (product) (1 - a^2) of the lane's eight entries, zero past the batch
    auto through_tanh = [&](const f32x4 *c, const float *a, float &sum, float *d) {
      bf16x8 f;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        float v = c[j >> 2][j & 3];
        v *= 1.0f - a[j] * a[j];
        d[j] = tile_row(q, j) < rows ? v : 0.f;
        sum += d[j];
        f[j] = __bf16(d[j]);
      }
      return f;
    };
    auto put = [&](__bf16 *dst, bf16x8 f) {
#pragma unroll
      for (int j = 0; j < 8; ++j) dst[tile_row(q, j) * LDA + n] = f[j];
    };
    f32x4 c[2];
    float d[8];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int m = 16 * h + r;
      c[h] = mfma(row_frag(dY + (m0 + (m < rows ? m : 0)) * NOUT, 8 * q, m < rows ? NOUT : 0), w3, zero);
    }
    const bf16x8 d2 = through_tanh(c, a2, s2, d);
    if constexpr (LO) put(S.err[0], d2);
    __syncthreads();
    if constexpr (LO) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const __bf16 *src = S.err[0] + (16 * h + r) * LDA + 8 * q;
        c[h] = zero;
#pragma unroll
        for (int j = 0; j < 4; ++j) c[h] = mfma(*reinterpret_cast<const bf16x8 *>(src + 32 * j), w2[j], c[h]);
      }
    }
    if constexpr (HI) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        g2[i] = mfma(d2, *reinterpret_cast<const bf16x8 *>(&S.actT[par][1][(16 * i + r) * LDT + 8 * q]), g2[i]);
    }
    if constexpr (LO) {
      const bf16x8 d1 = through_tanh(c, a1, s1, d);
      put(S.err[1], d1);
      __syncthreads();
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const __bf16 *src = S.err[1] + (16 * h + r) * LDA + 8 * q;
        c[h] = zero;
#pragma unroll
        for (int j = 0; j < 4; ++j) c[h] = mfma(*reinterpret_cast<const bf16x8 *>(src + 32 * j), w1[j], c[h]);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i)
        g1[i] = mfma(d1, *reinterpret_cast<const bf16x8 *>(&S.actT[par][0][(16 * i + r) * LDT + 8 * q]), g1[i]);
      const bf16x8 d0 = through_tanh(c, a0, s0, d);
      g0 = mfma(d0, x, g0);
    }
  }
  auto over_q = [](float v) {
    v += __shfl_xor(v, 16);
    return v + __shfl_xor(v, 32);
  };
  if constexpr (HI) {
    s3[0] = over_q(s3[0]);
    s3[1] = over_q(s3[1]);
    s2 = over_q(s2);
    if (q == 0) {
      if (wave == 0) {
        G[boff(3) + r] = s3[0];
        if (16 + r < NOUT) G[boff(3) + 16 + r] = s3[1];
      }
      G[boff(2) + n] = s2;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = 4 * q + i;              // row of a 16-row tile of outputs
      G[woff(3) + m * NH + n] = g3[0][i];
      if (16 + m < NOUT) G[woff(3) + (16 + m) * NH + n] = g3[1][i];
#pragma unroll
      for (int j = 0; j < 8; ++j) G[woff(2) + (16 * wave + m) * NH + 16 * j + r] = g2[j][i];
    }
  }
  if constexpr (LO) {
    s1 = over_q(s1);
    s0 = over_q(s0);
    if (q == 0) {
      G[boff(1) + n] = s1;
      G[boff(0) + n] = s0;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = 4 * q + i;
#pragma unroll
      for (int j = 0; j < 8; ++j) G[woff(1) + (16 * wave + m) * NH + 16 * j + r] = g1[j][i];
      if (r < NIN) G[woff(0) + (16 * wave + m) * NIN + r] = g0[i];
    }
  }
}

// Which block forms what (backward_plan), and where block b of a kind leaves its sums: parameter p at
// base + b stride + p.
struct BackwardPlan {
  int split;                        // blocks of layers 2 and 3, then blocks of layers 0 and 1; or all layers
  int hi_blocks, lo_blocks;         // blocks with sums of layers 2 and 3, of layers 0 and 1
  int64_t hi_base, hi_stride, lo_base, lo_stride;
};

__global__ __launch_bounds__(MLP_THREADS, 2) void mlp_backward_kernel(const float *__restrict__ P,
                                                                      const float *__restrict__ X, int B,
                                                                      const float *__restrict__ acts,
                                                                      const float *__restrict__ dY,
                                                                      float *__restrict__ part, BackwardPlan L) {
  __shared__ BackwardLds S;
  const int b = blockIdx.x;
  if (!L.split) {
    backward_tiles<true, true>(P, X, B, acts, dY, part + b * L.hi_stride, S, b, L.hi_blocks);
  } else if (b < L.hi_blocks) {
    backward_tiles<true, false>(P, X, B, acts, dY, part + L.hi_base + b * L.hi_stride, S, b, L.hi_blocks);
  } else {
    const int c = b - L.hi_blocks;
    backward_tiles<false, true>(P, X, B, acts, dY, part + L.lo_base + c * L.lo_stride, S, c, L.lo_blocks);
  }
}

// G = sum of the blocks' gradients in a fixed order: 64 parameters a block, four waves over
// the blocks
__global__ __launch_bounds__(256) void mlp_reduce_kernel(BackwardPlan L, const float *__restrict__ part,
                                                         float *__restrict__ G) {
  __shared__ float sh[4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, p = int(blockIdx.x) * 64 + lane;
  const bool hi = p >= woff(2);
  const int nb = hi ? L.hi_blocks : L.lo_blocks;
  const int64_t base = hi ? L.hi_base : L.lo_base, stride = hi ? L.hi_stride : L.lo_stride;
  float s = 0.f;
  if (p < NPARAM) {
#pragma unroll 8
    for (int b = w; b < nb; b += 4) s += part[base + b * stride + p];
  }
  sh[w][lane] = s;
  __syncthreads();
  if (w == 0 && p < NPARAM) G[p] = (sh[0][lane] + sh[1][lane]) + (sh[2][lane] + sh[3][lane]);
}

__global__ void mse_grad_kernel(int64_t n, const float *__restrict__ Y, const float *__restrict__ T,
                                float *__restrict__ dY, double *__restrict__ loss) {
  __shared__ double red[4];
  double s = 0.0;
  const float scale = 2.0f / float(n);
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x) {
    const float d = Y[i] - T[i];
    dY[i] = scale * d;
    s += double(d) * double(d);
  }
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0 && loss) atomicAdd(loss, (red[0] + red[1] + red[2] + red[3]) / double(n));
}

__global__ void adam_kernel(int n, float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m,
                            float *__restrict__ v, float lr, float b1, float b2, float eps, float c1, float c2) {
  const int i = int(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
}

// D = 10 sinh(Y): the network's correction of the shallow-ice profile (a column's outputs are
// its dofs in order)
__device__ __forceinline__ double correction(float y) { return 10.0 * sinh(double(y)); }

__global__ void correction_kernel(int64_t n, const float *__restrict__ Y, double *__restrict__ D) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  D[i] = correction(Y[i]);
}

// One Jacobi sweep over the base mesh: Dn_v = (D_v + mean of D_w over v's neighbours w != v) / 2,
// for each of the nd dofs of a column.
__global__ void smooth_kernel(int V, int nd, const int32_t *__restrict__ nbr_ptr, const int32_t *__restrict__ nbr_idx,
                              const double *__restrict__ D, double *__restrict__ Dn) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= int64_t(V) * nd) return;
  const int v = int(i / nd), r = int(i % nd);
  double s = 0.0;
  int cnt = 0;
  for (int p = nbr_ptr[v]; p < nbr_ptr[v + 1]; ++p) {
    const int w = nbr_idx[p];
    if (w == v) continue;
    s += D[int64_t(w) * nd + r];
    ++cnt;
  }
  const double d = D[i];
  Dn[i] = cnt > 0 ? 0.5 * (d + s / double(cnt)) : d;
}

// U = U_sia + D; flag non-finite values.  Without smoothing between, D comes straight from the network's
// output Y.
__global__ void compose_kernel(int64_t n, const double *__restrict__ D, const float *__restrict__ Y,
                               const double *__restrict__ Us, double *__restrict__ U, int *__restrict__ bad) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double u = Us[i] + (D ? D[i] : correction(Y[i]));
  U[i] = u;
  if (!isfinite(u)) atomicOr(bad, 1);
}

// T = asinh((U - U_sia) / 10), rounded to FP32
__global__ void targets_kernel(int64_t n, const double *__restrict__ U, const double *__restrict__ Us,
                               float *__restrict__ T) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  T[i] = float(asinh((U[i] - Us[i]) / 10.0));
}

// Xn = (X - mean) / std per feature, in FP64 and rounded once, as features_kernel normalises
__global__ void normalise_kernel(int64_t n, const float *__restrict__ X, const float *__restrict__ norm,
                                 float *__restrict__ Xn) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int j = int(i % NIN);
  Xn[i] = float((double(X[i]) - double(norm[j])) / double(norm[NIN + j]));
}

// Per feature column j (one block each): mean, then sqrt(sum (x - mean)^2 / (n - 1)) + 1e-6.
__global__ __launch_bounds__(256) void feature_stats_kernel(const float *__restrict__ X, int64_t n,
                                                            float *__restrict__ norm) {
  const int j = blockIdx.x;
  __shared__ double red[4];
  __shared__ double mean_s;
  double s = 0.0;
  for (int64_t r = threadIdx.x; r < n; r += blockDim.x) s += double(X[r * NIN + j]);
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) mean_s = (red[0] + red[1] + red[2] + red[3]) / double(n);
  __syncthreads();
  const double mean = mean_s;
  double q = 0.0;
  for (int64_t r = threadIdx.x; r < n; r += blockDim.x) {
    const double d = double(X[r * NIN + j]) - mean;
    q += d * d;
  }
  for (int off = 32; off > 0; off >>= 1) q += __shfl_xor(q, off);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = q;
  __syncthreads();
  if (threadIdx.x == 0) {
    norm[j] = float(mean);
    norm[NIN + j] = float(sqrt((red[0] + red[1] + red[2] + red[3]) / double(n - 1)) + 1e-6);
  }
}

}  // namespace

// forward through all layers: acts [3][B][NH] (FP32 tanh outputs, or NULL), Y [B][NOUT].  Two
// blocks share a compute unit, so 512 blocks hold the whole chip.
fo_status mlp_forward_impl(const float *P, const float *X, int B, float *acts, float *Y, hipStream_t s) {
  if (B <= 0) return FO_OK;
  const int tiles = (B + FWD_ROWS - 1) / FWD_ROWS;
  hipLaunchKernelGGL(mlp_forward_kernel, dim3(unsigned(tiles < 512 ? tiles : 512)), dim3(MLP_THREADS), 0, s, P, X, B,
                     acts, Y);
  FO_LAUNCH_CHECK("mlp_forward_kernel");
  return FO_OK;
}

}  // namespace fo

using namespace fo;

extern "C" int32_t fo_mlp_param_count(void) { return NPARAM; }

static fo_status launch_features(const fo_mesh *m, const float *norm, float *F, int *clear, hipStream_t s) {
  const unsigned blocks = unsigned((int64_t(m->view.V) * VERT_LANES + 63) / 64);
  hipLaunchKernelGGL(features_kernel, dim3(blocks), dim3(64), 0, s, m->view, m->nbr_ptr, m->nbr_idx, m->vc_ptr,
                     m->vc_idx, norm, F, clear);
  FO_LAUNCH_CHECK("features_kernel");
  return FO_OK;
}

extern "C" fo_status fo_column_features(const fo_mesh *m, const float *norm, float *F, void *stream) {
  if (!m || !F) return fail(FO_EINVAL, "fo_column_features: NULL argument");
  return launch_features(m, norm, F, nullptr, static_cast<hipStream_t>(stream));
}

extern "C" fo_status fo_mlp_forward(const float *P, const float *X, int32_t B, float *acts, float *Y, void *stream) {
  if (!P || !X || !acts || !Y || B < 0) return fail(FO_EINVAL, "fo_mlp_forward: bad argument");
  return mlp_forward_impl(P, X, B, acts, Y, static_cast<hipStream_t>(stream));
}

// The scratch (2 B NH floats) bounds the blocks, each of which leaves its sums there.  A block of layers 0
// and 1 only, or of 2 and 3 only, leaves half as much, so twice as many work on the tiles; the former
// take longer for a tile (they pass the errors through all layers), so there are half as many more of
// them.  Where the scratch holds most of a block per compute unit anyway, blocks of all layers do not
// load the tiles and form the first errors twice.  Both, with the sum over the blocks, by rows: 512
// 29.6 us in halves, 37.4 not; 4096 27.2, 36.2; 16384 36.9, 46.3; 24000 43.7, 48.7; 27952 49.4, 50.7.
// Less scratch than three such blocks: one of each kind, straight into the gradients (200 rows: 32 us,
// 39 in one block).
static BackwardPlan backward_plan(int32_t B) {
  constexpr int64_t LO = woff(2), HI = NPARAM - LO, MOST = 256;
  const int64_t scratch = 2 * int64_t(B) * NH, tiles = (int64_t(B) + BWD_ROWS - 1) / BWD_ROWS;
  if (scratch < HI + 2 * LO) return {1, 1, 1, 0, 0, 0, 0};
  if (scratch / NPARAM >= SPLIT_BELOW) {
    const int nb = int(std::min({scratch / NPARAM, tiles, MOST}));
    return {0, nb, nb, 0, NPARAM, 0, NPARAM};
  }
  const int64_t nhi = std::min({2 * scratch / (2 * HI + 3 * LO), tiles, 2 * MOST / 5});
  const int64_t nlo = std::min({(scratch - nhi * HI) / LO, tiles, MOST - nhi});
  return {1, int(nhi), int(nlo), -LO, HI, nhi * HI, LO};
}

extern "C" fo_status fo_mlp_backward(const float *P, const float *X, int32_t B, const float *acts, const float *dY,
                                     float *dacts, float *G, void *stream) {
  if (!P || !X || !acts || !dY || !dacts || !G || B < 0) return fail(FO_EINVAL, "fo_mlp_backward: bad argument");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const BackwardPlan L = backward_plan(B);
  const bool direct = L.hi_blocks == 1 && L.lo_blocks == 1;   // no sums to add: the gradients themselves
  hipLaunchKernelGGL(mlp_backward_kernel, dim3(unsigned(L.split ? L.hi_blocks + L.lo_blocks : L.hi_blocks)),
                     dim3(MLP_THREADS), 0, s, P, X, B, acts, dY, direct ? G : dacts, L);
  FO_LAUNCH_CHECK("mlp_backward_kernel");
  if (!direct) {
    hipLaunchKernelGGL(mlp_reduce_kernel, dim3((NPARAM + 63) / 64), dim3(256), 0, s, L, dacts, G);
    FO_LAUNCH_CHECK("mlp_reduce_kernel");
  }
  return FO_OK;
}

extern "C" fo_status fo_mse_grad(const float *Y, const float *T, int64_t n, float *dY, double *loss, void *stream) {
  if (!Y || !T || !dY || n <= 0) return fail(FO_EINVAL, "fo_mse_grad: bad argument");
  int64_t blocks = (n + 255) / 256;
  if (blocks > 1024) blocks = 1024;
  hipLaunchKernelGGL(mse_grad_kernel, dim3(unsigned(blocks)), dim3(256), 0, static_cast<hipStream_t>(stream), n, Y, T,
                     dY, loss);
  FO_LAUNCH_CHECK("mse_grad_kernel");
  return FO_OK;
}

extern "C" fo_status fo_adam_step(float *P, const float *G, float *Mom, float *Var, int32_t n, float lr, float b1,
                                  float b2, float eps, int32_t step, void *stream) {
  if (!P || !G || !Mom || !Var || n <= 0 || step < 1) return fail(FO_EINVAL, "fo_adam_step: bad argument");
  const float c1 = float(1.0 / (1.0 - std::pow(double(b1), step)));
  const float c2 = float(1.0 / (1.0 - std::pow(double(b2), step)));
  hipLaunchKernelGGL(adam_kernel, dim3(unsigned((n + 255) / 256)), dim3(256), 0, static_cast<hipStream_t>(stream), n,
                     P, G, Mom, Var, lr, b1, b2, eps, c1, c2);
  FO_LAUNCH_CHECK("adam_kernel");
  return FO_OK;
}

namespace {
constexpr size_t ALIGN = 256;
size_t up(size_t x) { return (x + ALIGN - 1) / ALIGN * ALIGN; }
struct LLayout { size_t F, partial, Y, Us, R, D, dots, flag, total; };
LLayout llayout(const fo_mesh *m) {
  const size_t V = size_t(m->view.V), n = size_t(m->view.n_dofs);
  LLayout L{};
  size_t off = 0;
  auto take = [&](size_t b) { size_t a = off; off += up(b); return a; };
  L.F = take(4 * V * NIN);
  // The dot products' partial sums: 8 multidot_blocks(n) bytes, at most 4 KB, where 4.5 KB lie here from
  // three vertices on.  The rest of the region is not used (inference stores no activations); its size is
  // part of the total that callers were told, and of the limit of the variant without a workspace.
  L.partial = take(up(4 * 3 * V * NH) + 8 * std::min<size_t>(std::max<size_t>((n + 4095) / 4096, 1), 512));
  L.Y = take(4 * V * NOUT);
  L.Us = take(8 * n);
  L.R = take(8 * n);
  L.D = take(8 * 2 * n);
  L.dots = take(16);
  L.flag = take(16);
  L.total = off;
  return L;
}
}  // namespace

namespace fo {
size_t learned_workspace_bytes(const fo_mesh *m) { return llayout(m).total; }

fo_status learned_guess(const fo_mesh *m, const float *P, const float *norm, double *U, int32_t fallback,
                        int32_t sweeps, void *ws, size_t ws_bytes, int32_t *used_network, int32_t *n_residuals,
                        hipStream_t s) {
  if (n_residuals) *n_residuals = 0;
  if (!m || !P || !norm || !U || !ws) return fail(FO_EINVAL, "fo_initial_guess_learned: NULL argument");
  if (fallback != 0 && fallback != 1) return fail(FO_EINVAL, "fo_initial_guess_learned: fallback must be 0 or 1");
  if (sweeps < 0 || sweeps > 10000) return fail(FO_EINVAL, "fo_initial_guess_learned: smooth_sweeps must be in 0..10000");
  if (m->view.L + 1 != NOUT / 2) return fail(FO_EINVAL, "fo_initial_guess_learned: the network predicts 11 levels (L = 10)");
  if (reinterpret_cast<uintptr_t>(ws) & 255) return fail(FO_EINVAL, "fo_initial_guess_learned: workspace must be 256-byte aligned");
  const LLayout L = llayout(m);
  if (ws_bytes < L.total) return fail(FO_EINVAL, "fo_initial_guess_learned: workspace too small");
  char *w = static_cast<char *>(ws);
  float *F = reinterpret_cast<float *>(w + L.F);
  float *Y = reinterpret_cast<float *>(w + L.Y);
  double *Us = reinterpret_cast<double *>(w + L.Us), *R = reinterpret_cast<double *>(w + L.R);
  double *D0 = reinterpret_cast<double *>(w + L.D);
  double *part = reinterpret_cast<double *>(w + L.partial), *dots = reinterpret_cast<double *>(w + L.dots);
  int *flag = reinterpret_cast<int *>(w + L.flag);
  const int V = m->view.V;
  const int64_t n = m->view.n_dofs;
  double *D1 = D0 + n;
  fo_status st;
  if ((st = launch_sia(m, Us, s)) != FO_OK) return st;
  if ((st = launch_features(m, norm, F, flag, s)) != FO_OK) return st;
  if ((st = mlp_forward_impl(P, F, V, nullptr, Y, s)) != FO_OK) return st;
  const unsigned nb = unsigned((n + 255) / 256);
  if (sweeps > 0) {
    hipLaunchKernelGGL(correction_kernel, dim3(nb), dim3(256), 0, s, n, Y, D0);
    FO_LAUNCH_CHECK("correction_kernel");
  }
  for (int k = 0; k < sweeps; ++k) {
    hipLaunchKernelGGL(smooth_kernel, dim3(nb), dim3(256), 0, s, V, NOUT, m->nbr_ptr, m->nbr_idx, D0, D1);
    FO_LAUNCH_CHECK("smooth_kernel");
    std::swap(D0, D1);
  }
  hipLaunchKernelGGL(compose_kernel, dim3(nb), dim3(256), 0, s, n, sweeps > 0 ? D0 : nullptr, Y, Us, U, flag);
  FO_LAUNCH_CHECK("compose_kernel");
  // fall back to the shallow-ice guess if the network output is non-finite, or (fallback = 1)
  // if its residual norm exceeds the shallow-ice guess's
  double hv[2] = {0.0, 0.0};
  int bad = 0;
  FO_HIP_TRY(hipMemcpyAsync(&bad, flag, sizeof(int), hipMemcpyDeviceToHost, s));
  if (fallback == 1) {
    if ((st = launch_assemble(m, Us, R, nullptr, FO_F64, FO_JAC_NEWTON, false, s)) != FO_OK) return st;
    if (n_residuals) ++*n_residuals;
    if ((st = multidot(n, nullptr, 0, 0, R, part, dots, 0.0, nullptr, 0, s)) != FO_OK) return st;
    FO_HIP_TRY(hipMemcpyAsync(&hv[1], dots, sizeof(double), hipMemcpyDeviceToHost, s));
  }
  FO_HIP_TRY(hipStreamSynchronize(s));
  bool use_nn = bad == 0;
  if (use_nn && fallback == 1) {
    if ((st = launch_assemble(m, U, R, nullptr, FO_F64, FO_JAC_NEWTON, false, s)) != FO_OK) return st;
    if (n_residuals) ++*n_residuals;
    if ((st = multidot(n, nullptr, 0, 0, R, part, dots, 0.0, nullptr, 0, s)) != FO_OK) return st;
    FO_HIP_TRY(hipMemcpyAsync(&hv[0], dots, sizeof(double), hipMemcpyDeviceToHost, s));
    FO_HIP_TRY(hipStreamSynchronize(s));
    use_nn = std::isfinite(hv[0]) && hv[0] <= hv[1];
  }
  if (!use_nn) FO_HIP_TRY(hipMemcpyAsync(U, Us, sizeof(double) * n, hipMemcpyDeviceToDevice, s));
  FO_HIP_TRY(hipStreamSynchronize(s));
  if (used_network) *used_network = use_nn ? 1 : 0;
  return FO_OK;
}
}  // namespace fo

extern "C" size_t fo_learned_workspace_bytes(const fo_mesh *m) { return m ? llayout(m).total : 0; }

extern "C" fo_status fo_initial_guess_learned(const fo_mesh *m, const float *P, const float *norm, double *U,
                                              int32_t fallback, int32_t smooth_sweeps, void *ws, size_t ws_bytes,
                                              int32_t *used_network, void *stream) {
  return learned_guess(m, P, norm, U, fallback, smooth_sweeps, ws, ws_bytes, used_network, nullptr,
                       static_cast<hipStream_t>(stream));
}

// Workspace of fo_initial_guess_learned_noalloc: a library-owned array on each device,
// resolved to its device address once per device (the array's name in host code is a
// host-side stand-in, never a device address) and held until the process ends.
namespace {
__device__ __align__(256) unsigned char scratch[FO_LEARNED_SCRATCH_BYTES];
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_dev[kMaxDevices] = {};

fo_status scratch_address(int device, void **out) {
  if (device < 0 || device >= kMaxDevices) return fo::fail(FO_EDEVICE, "device index out of range");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_dev[device]) {
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      return fo::fail(FO_EDEVICE, std::string("hipGetSymbolAddress(scratch) failed: ") + hipGetErrorString(e));
    g_scratch_dev[device] = p;
  }
  *out = g_scratch_dev[device];
  return FO_OK;
}
}  // namespace

extern "C" fo_status fo_initial_guess_learned_noalloc(const fo_mesh *m, const float *P, const float *norm, double *U,
                                                      int32_t fallback, int32_t smooth_sweeps, int32_t *used_network,
                                                      void *stream) {
  if (!m) return fail(FO_EINVAL, "fo_initial_guess_learned_noalloc: NULL mesh");
  const size_t need = llayout(m).total;
  if (need > FO_LEARNED_SCRATCH_BYTES)
    return fail(FO_EINVAL, "fo_initial_guess_learned_noalloc: mesh needs " + std::to_string(need) +
                               " bytes of workspace, more than the library's " +
                               std::to_string(size_t(FO_LEARNED_SCRATCH_BYTES)) + "-byte array");
  int dev = -1;
  FO_HIP_TRY(hipGetDevice(&dev));
  if (dev != m->device)
    return fail(FO_EINVAL, "fo_initial_guess_learned_noalloc: the mesh's device must be the current device");
  void *ws = nullptr;
  fo_status st = scratch_address(dev, &ws);
  if (st != FO_OK) return st;
  return learned_guess(m, P, norm, U, fallback, smooth_sweeps, ws, FO_LEARNED_SCRATCH_BYTES, used_network, nullptr,
                       static_cast<hipStream_t>(stream));
}

extern "C" fo_status fo_learned_targets(const fo_mesh *m, const double *U, const double *Us, float *T, void *stream) {
  if (!m || !U || !Us || !T) return fail(FO_EINVAL, "fo_learned_targets: NULL argument");
  if (m->view.L + 1 != NOUT / 2) return fail(FO_EINVAL, "fo_learned_targets: the network predicts 11 levels (L = 10)");
  const int64_t n = m->view.n_dofs;
  hipLaunchKernelGGL(targets_kernel, dim3(unsigned((n + 255) / 256)), dim3(256), 0, static_cast<hipStream_t>(stream),
                     n, U, Us, T);
  FO_LAUNCH_CHECK("targets_kernel");
  return FO_OK;
}

extern "C" fo_status fo_feature_stats(const float *X, int64_t n_rows, float *norm, float *Xn, void *stream) {
  if (!X || !norm || n_rows < 2) return fail(FO_EINVAL, "fo_feature_stats: NULL argument or fewer than 2 rows");
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(feature_stats_kernel, dim3(NIN), dim3(256), 0, s, X, n_rows, norm);
  FO_LAUNCH_CHECK("feature_stats_kernel");
  if (Xn) {
    const int64_t n = n_rows * NIN;
    hipLaunchKernelGGL(normalise_kernel, dim3(unsigned((n + 255) / 256)), dim3(256), 0, s, n, X, norm, Xn);
    FO_LAUNCH_CHECK("normalise_kernel");
  }
  return FO_OK;
}
