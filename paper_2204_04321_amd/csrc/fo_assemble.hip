// Cell-parallel assembly of the first-order Stokes residual and Jacobian on gfx950.
//
// Physics (arXiv:2204.04321 Sec. 2): momentum balance eq. (FOStokes) with the
// strain-rate vectors eps1 = (2 e_xx + e_yy, e_xy, e_xz), eps2 = (e_xy,
// e_xx + 2 e_yy, e_yz); Glen viscosity eq. (effvisc) with the effective strain
// rate eq. (effeps), regularised by eps0; stress-free surface; linear bed
// friction beta u.  Discrete residual eq. (residual); Jacobian eq. (linearsystem)
// by forward-mode AD (Sec. 3.2): the tangent of the element residual along each
// element dof is pushed through strain rate -> eps_e^2 -> mu -> residual.
//
// Owner-computes decomposition.  Every CSR row block belongs to one vertex column
// v (all dofs of v, every level).  Work item = (v, base cell t around v): one lane
// walks the column of t from the bed up, layer by layer, and evaluates each cell
// at its quadrature points (geometry, strain rate, viscosity: the primal), then
// the residual rows of v's two nodes in the cell and their derivatives along all
// element dofs (the AD tangents, one register accumulator per derivative
// direction and row).  A wave owns a run of consecutive vertex columns (<= 64
// items); its lanes add their rows into a two-level window of those columns in
// LDS, and once level k has received both cells that touch it (layers k-1 and k)
// the wave copies it into its contiguous CSR range.  No global atomics, no
// zero fill of J or R, every value written once; results do not depend on
// scheduling.  Each cell is evaluated by each of its vertex columns (3 or 4
// times) in exchange.  Prisms spread an item over two lanes (prism_task below), hexahedra over
// four (hex_task); base triangles split into tetrahedra take one lane (tet_task).  The level
// windows are FP64 for either Jacobian value type.
//
// CSR slot of row (v, level kr, comp c) and column (vertex of rank r in v's sorted
// neighbour list, level kc, comp d): colptr[v] + 4 D_v cumlev(kr) + c 2 nlev(kr) D_v
// + r 2 nlev(kr) + 2 (kc - max(kr-1, 0)) + d.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "fo_internal.h"

// Multiply-adds are fused only where one source expression holds both operations, so
// the residual-only, R+J and ensemble kernels, which share the element arithmetic, round
// it identically (fusion chosen by the backend depends on each kernel's other uses).
#pragma clang fp contract(on)

namespace fo {
namespace {

constexpr int WAVE = 64;

constexpr double G1 = 0.21132486540518711775;   // 1/2 - 1/(2 sqrt 3)
constexpr double G2 = 0.78867513459481288225;   // 1/2 + 1/(2 sqrt 3)

__device__ __forceinline__ int nlev(int k, int L) { return (k == 0 || k == L) ? 2 : 3; }
__device__ __forceinline__ int cumlev(int k) { return k == 0 ? 0 : 3 * k - 1; }

// 1/x: hardware estimate refined by two Newton steps (full double precision).
__device__ __forceinline__ double rcp64(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  r = fma(r, fma(-x, r, 1.0), r);
  return r;
}

// x^(-1/3) for x > 0: single-precision exp2/log2 estimate (~1e-7) refined by two Newton
// steps on y^-3 = x, y <- y (4 - x y^3) / 3 (quadratic convergence to double precision).
__device__ __forceinline__ double rcbrt64(double x) {
  const double y = double(__builtin_amdgcn_exp2f(-__builtin_amdgcn_logf(float(x)) * (1.0f / 3.0f)));
  // one third-order step: with r = 1 - x y^3, x^(-1/3) = y (1 - r)^(-1/3)
  // = y (1 + r/3 + 2 r^2/9 + O(r^3)), and |r| ~ 1e-7 leaves O(1e-21)
  const double r = fma(-x, y * y * y, 1.0);
  return fma(y * r, fma(2.0 / 9.0, r, 1.0 / 3.0), y);
}

// q^p for the viscosity power, q = eps_e^2 + eps0^2 >= 0: exp2(p log2 q), which needs none
// of the general pow's cases for negative or special arguments; p = 0 (n = 1) gives 1.
__device__ __forceinline__ double powq(double q, double p) {
  return p == 0.0 ? 1.0 : exp2(p * log2(q));
}

template <class T>
__device__ __forceinline__ void lds_add(T *p, T v) {
  atomicAdd(p, v);   // LDS atomics: lanes of one wave may hit the same entry
}

// A table that no kernel writes, in scalar registers: read with scalar loads, which do not wait for
// the vector loads in flight (sigma read through a generic pointer made every layer wait for the
// next layer's velocities).
typedef const double __attribute__((address_space(4))) *ScalarTable;
__device__ __forceinline__ ScalarTable scalar_table(const double *p) {
  uint64_t v = reinterpret_cast<uint64_t>(p);
  asm volatile("" : "+s"(v));     // a register pair of its own, apart from the kernel arguments' block
  return reinterpret_cast<ScalarTable>(v);
}

// The block is one wave: a workgroup barrier orders its LDS traffic.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Picks a, b, c or d by a lane-varying index i (d for any i outside 0..2) without a branch:
// all four operands are evaluated and combined through bit masks.  Written as a compare
// chain, the selection becomes a switch, i.e. a divergent branch tree, and the register
// allocator has placed copies of values that stay live across it inside the masked part,
// so lanes outside the mask later read copies they never wrote.
__device__ __forceinline__ double sel4(int i, double a, double b, double c, double d) {
  using u64 = unsigned long long;
  const u64 m0 = 0ull - u64(i == 0), m1 = 0ull - u64(i == 1), m2 = 0ull - u64(i == 2);
  const u64 m3 = ~(m0 | m1 | m2);
  const u64 r = (__builtin_bit_cast(u64, a) & m0) | (__builtin_bit_cast(u64, b) & m1) |
                (__builtin_bit_cast(u64, c) & m2) | (__builtin_bit_cast(u64, d) & m3);
  return __builtin_bit_cast(double, r);
}

// v with its sign flipped where sign = 0x80000000 (0: as it is)
__device__ __forceinline__ double flip(double v, uint32_t sign) {
  return __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, v) ^ (uint64_t(sign) << 32));
}

// i ? b : a without a branch (both operands in registers)
__device__ __forceinline__ double sel2(int i, double a, double b) { return sel4(i, a, b, b, b); }

// Two consecutive Jacobian entries as one streaming (nontemporal) store; p is 8-entry aligned.
template <class JT>
__device__ __forceinline__ void store2_nt(JT *p, double x, double y) {
  typedef JT v2 __attribute__((ext_vector_type(2)));
  v2 t;
  t.x = JT(x);
  t.y = JT(y);
  __builtin_nontemporal_store(t, reinterpret_cast<v2 *>(p));
}

// Metadata of a task's vertex columns, one column per lane (a task has at most 64)
struct TaskColumns {
  int deg, soff, col_lo, col_hi;
};

__device__ __forceinline__ TaskColumns load_columns(const MeshView &m, int vb, int nvt, int lane) {
  TaskColumns t = {0, 0, 0, 0};
  if (lane < nvt) {
    t.deg = m.deg[vb + lane];
    t.soff = m.slot_off[vb + lane];
    const int64_t c = m.colptr[vb + lane];
    t.col_lo = int(uint32_t(uint64_t(c)));
    t.col_hi = int(uint32_t(uint64_t(c) >> 32));
  }
  return t;
}

template <bool JAC>
__device__ __forceinline__ void clear_windows(const MeshView &m, double *Jw, double *Rw, int vb, int ve, int max_slot,
                                              int max_tv, int lane) {
  if constexpr (JAC) {
    const int slot_size = m.slot_off[ve - 1] + 12 * m.deg[ve - 1];
    for (int e = lane; e < slot_size; e += WAVE) { Jw[e] = 0.0; Jw[max_slot + e] = 0.0; }
  }
  for (int e = lane; e < 2 * (ve - vb); e += WAVE) { Rw[e] = 0.0; Rw[2 * max_tv + e] = 0.0; }
}

// Where a lane's share of an interior level goes.  On three levels a column's rows fill its whole
// slot (12 D entries), so a task's window is one contiguous run; lane l moves the entry pairs
// 2 l + 128 i.  off[i]: the pair's place on level 1, in entries from the task's first; deg: its
// column's degree, 8 bits per i.  Each further level lies 12 D entries on.
// N parts: 4 hold the windows of 32 items around vertices of up to six or seven cells, 8 those of 64.
template <int N>
struct FlatCopy {
  uint32_t off[N], deg[N / 4];
  int slot_size;      // 0: the window or the offsets are too large, columns are copied one by one
  int64_t base;       // colptr of the task's first column
};

template <bool JAC, int N>
__device__ __forceinline__ FlatCopy<N> flat_copy(const MeshView &m, const TaskColumns &cols, int vb, int nvt, int lane) {
  FlatCopy<N> f = {};
  if constexpr (!JAC) return f;
  const int n = __builtin_amdgcn_readlane(cols.soff, nvt - 1) + 12 * __builtin_amdgcn_readlane(cols.deg, nvt - 1);
  f.base = int64_t(unsigned(__builtin_amdgcn_readlane(cols.col_lo, 0))) |
           (int64_t(__builtin_amdgcn_readlane(cols.col_hi, 0)) << 32);
  if (n > 128 * N || m.L > 4096) return f;
  f.slot_size = n;
  for (int c = 0; c < nvt; ++c) {
    const int so = __builtin_amdgcn_readlane(cols.soff, c), D = __builtin_amdgcn_readlane(cols.deg, c);
    const uint32_t start = uint32_t(__builtin_amdgcn_readlane(cols.col_lo, c)) - uint32_t(f.base) + 8u * uint32_t(D);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int e = 2 * lane + 128 * i;
      if (e >= so) {
        f.off[i] = start + uint32_t(e - so);
        f.deg[i / 4] = (f.deg[i / 4] & ~(255u << (8 * (i & 3)))) | (uint32_t(D) << (8 * (i & 3)));
      }
    }
  }
  return f;
}

// Copies a finished level's window to its rows and clears it for level + 2 (store = false: clears it
// only); all LDS reads are issued before the first store.  With a Jacobian, interior levels only.
template <bool JAC, int N, class JT>
__device__ __forceinline__ void copy_out_flat(const FlatCopy<N> &f, int lev, int slot, bool store, int vb, int nvt, int L,
                                              double *Jw, double *Rw, int max_slot, int max_tv, int lane,
                                              double *__restrict__ R, JT *__restrict__ J) {
  if constexpr (JAC) {
    double *wb = Jw + slot * max_slot + 2 * lane;
    JT *dst = J + f.base;
    const uint32_t up = 12u * uint32_t(lev - 1);
    double2 val[N];
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (128 * i < f.slot_size)     // past the window's end: other LDS of the task, not stored
        val[i] = *reinterpret_cast<const double2 *>(wb + (2 * lane + 128 * i < f.slot_size ? 128 * i : 0));
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (128 * i < f.slot_size && 2 * lane + 128 * i < f.slot_size) {
        if (store) store2_nt(dst + (f.off[i] + up * ((f.deg[i / 4] >> (8 * (i & 3))) & 255u)), val[i].x, val[i].y);
        *reinterpret_cast<double2 *>(wb + 128 * i) = make_double2(0.0, 0.0);
      }
  }
  for (int e = lane; e < 2 * nvt; e += WAVE) {
    double *rs = Rw + slot * 2 * max_tv + e;
    if (R && store) R[2 * (int64_t(vb + (e >> 1)) * (L + 1) + lev) + (e & 1)] = *rs;
    *rs = 0.0;
  }
}

// Copies a finished level's window to its CSR rows and clears it for level + 2 (store = false:
// clears it only).  Four vertex columns at a time: all LDS reads of a batch are issued before
// the first global store, so one LDS latency is exposed per batch, not per chunk.  Each lane moves
// two consecutive entries: one 16-byte LDS read and one 16-byte clearing write per column cover
// up to 128 entries (degree <= 10 on three levels).
template <class JT>
__device__ __forceinline__ void copy_out(const TaskColumns &cols, int lev, int slot, bool store, int vb, int nvt,
                                         int L, double *Jw, double *Rw, int max_slot, int max_tv, int lane,
                                         double *__restrict__ R, JT *__restrict__ J) {
  const int nl = nlev(lev, L);
  const int lk = cumlev(lev);
  double *wb = Jw + slot * max_slot;   // 16-byte aligned, as is every column's slot
  for (int i0 = 0; i0 < nvt; i0 += 4) {
    double2 val[4];
    int nn[4], so[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int ii = i0 + i < nvt ? i0 + i : nvt - 1;
      so[i] = __builtin_amdgcn_readlane(cols.soff, ii);
      nn[i] = i0 + i < nvt ? 4 * nl * __builtin_amdgcn_readlane(cols.deg, ii) : 0;
      const int e = 2 * lane;
      val[i] = *reinterpret_cast<const double2 *>(wb + so[i] + (e < nn[i] ? e : 0));
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (i0 + i >= nvt) break;
      const int ii = i0 + i;
      const int D = __builtin_amdgcn_readlane(cols.deg, ii);
      const int64_t col = int64_t(unsigned(__builtin_amdgcn_readlane(cols.col_lo, ii))) |
                          (int64_t(__builtin_amdgcn_readlane(cols.col_hi, ii)) << 32);
      JT *dst = J + col + int64_t(4) * D * lk;
      double *src = wb + so[i];
      const int e = 2 * lane;   // nn is a multiple of 4, so e < nn implies e + 1 < nn
      if (e < nn[i]) {
        if (store) store2_nt(dst + e, val[i].x, val[i].y);
        *reinterpret_cast<double2 *>(src + e) = make_double2(0.0, 0.0);
      }
      for (int f = e + 2 * WAVE; f < nn[i]; f += 2 * WAVE) {
        const double2 w = *reinterpret_cast<const double2 *>(src + f);
        if (store) store2_nt(dst + f, w.x, w.y);
        *reinterpret_cast<double2 *>(src + f) = make_double2(0.0, 0.0);
      }
    }
    if (lane < 8 && i0 + (lane >> 1) < nvt) {
      const int u = vb + i0 + (lane >> 1);
      double *rs = Rw + slot * 2 * max_tv + 2 * (u - vb) + (lane & 1);
      if (R && store) R[2 * (int64_t(u) * (L + 1) + lev) + (lane & 1)] = *rs;
      *rs = 0.0;
    }
  }
}

// A finished level by its kind: with a Jacobian the rows of the first and the last level (two levels each)
// leave gaps in the columns' slots.  The residual alone has no slots, so any level goes in one piece
// (one-layer sheet of 125,000 columns: 40 -> 38 us).
template <bool JAC, int N, class JT>
__device__ __forceinline__ void copy_level(const FlatCopy<N> &f, const TaskColumns &cols, int lev, int slot, bool store,
                                           int vb, int nvt, int L, double *Jw, double *Rw, int max_slot, int max_tv,
                                           int lane, double *__restrict__ R, JT *__restrict__ J) {
  if constexpr (!JAC) {
    copy_out_flat<false>(f, lev, slot, store, vb, nvt, L, Jw, Rw, max_slot, max_tv, lane, R, J);
  } else if (lev > 0 && lev < L && f.slot_size > 0) {
    copy_out_flat<true>(f, lev, slot, store, vb, nvt, L, Jw, Rw, max_slot, max_tv, lane, R, J);
  } else {
    copy_out(cols, lev, slot, store, vb, nvt, L, Jw, Rw, max_slot, max_tv, lane, R, J);
  }
}

// Value of lane (lane ^ X), X = 1 or 2
__device__ __forceinline__ int quad_xor_i(int v, bool two) {
  return two ? __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true) : __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true);
}
template <int X>
__device__ __forceinline__ double quad_xor(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = uint32_t(quad_xor_i(int(uint32_t(u)), X == 2));
  const uint32_t hi = uint32_t(quad_xor_i(int(uint32_t(u >> 32)), X == 2));
  return __builtin_bit_cast(double, uint64_t(lo) | (uint64_t(hi) << 32));
}
template <int X>
__device__ __forceinline__ float quad_xor(float v) {
  return __builtin_bit_cast(float, quad_xor_i(__builtin_bit_cast(int, v), X == 2));
}

// ---- prisms ----------------------------------------------------------------------------------
// Two lanes per item, one per zeta Gauss point (three triangle points each): a lane evaluates the
// physics of its three points, accumulates its share of the item's tangents, and one exchange
// leaves each lane half of the entries.  One lane per item needs 56 accumulators for its six
// points and loops over zeta; here zeta is fixed, so 40 do: with b the gradient of a column node,
// every entry is sum_q L_q . b_q, where L_q (three numbers per row node a and component pair
// cd) depends on the row only.  For a prism, b = l h_j -+ lam_j p with h_j = (dN_j/dx, dN_j/dy, 0)
// constant over the cell, l = 1 - zeta, zeta the level's weight and p = grad zeta the same for
// all corners: so the lane sums L (x, y parts) over its points, and L . p per triangle point.
// The slopes of bed and thickness, 1/H at the points and the horizontal gradients are constants
// of the whole column.
//
// z = lane & 1.  Of row node a (0 lower, 1 upper) a lane ends with the entries at level a ^ z: the
// weight of the kept level is then G2 (a = 0) or G1 (a = 1) in either lane, and only the sign of
// p differs.  Lane z = 0 holds the upper row's entries at the upper level, which the next layer's
// lower row adds to the same places: they are carried in registers (a quarter fewer LDS adds).
// The cell's corners are taken in cyclic order from the item's own vertex, which is thus always
// corner 0.
//
// With a Jacobian it is bound by FP64 issue and the LDS adds alike (ice sheet of 125,000 columns of
// 10 layers: vector units 76% busy while two waves share a SIMD, the LDS 66% of the kernel's
// time); the residual alone, four waves per SIMD, by vector issue.  R+J 705 -> 551-575 us in FP64 and
// 670 -> 519 us with FP32 values, residual 175-180 -> 151 us, against one lane per item (of one layer
// R+J 140 -> 126 us, but the residual 34.5 -> 38: both lanes of an item load and work out its
// constants; from two layers on it is even, from three faster).  The parts:
// the split itself, with the constants in LDS, -7%; items of one vertex spread over the wave
// (below) -5%; sigma through scalar loads and the wait before the copy-out -2%; the copy-out of a
// level in one piece -6%.  Carrying the shared entries in FP64 too spills (+5%).
constexpr int PRISM_WAVES = 2;
constexpr int PRISM_CONST = 18;         // FP64 constants of an item (144 bytes: its 16-byte reads spread over all banks)
constexpr int PRISM_ITEMS = WAVE / 2;   // items per pass of a wave

// The levels kb <= k < ke of a task's columns (and level L if ke = L).  kb > 0 starts with layer
// kb - 1, whose lower rows belong to the range below and are dropped.  PASSES: the task holds
// more items than one pass of a wave takes (a vertex in more cells than that is a task of its
// own), so the item constants are reloaded for every layer and pass.
template <bool JAC, class JT, bool N3, bool PASSES>
__device__ __forceinline__ void prism_task(const MeshView &m, const int4 task, const double *__restrict__ U,
                                           double *__restrict__ R, JT *__restrict__ J, int picard, int max_slot,
                                           int max_tv, int kb, int ke, unsigned char *smem) {
  using AT = JT;   // derivative arithmetic type
  // The level windows accumulate in FP64 for either value type: FP32 LDS atomics on this
  // scatter pattern saturate the LDS data path (measured), FP64 ones do not.
  double *Jw = reinterpret_cast<double *>(smem);                                               // [2][max_slot]
  double *Rw = reinterpret_cast<double *>(smem + (JAC ? 2 * size_t(max_slot) * sizeof(double) : 0));  // [2][2 max_tv]
  const double tfac = picard ? 0.0 : m.visc_exp;
  double *const item_c = Rw + 4 * size_t(max_tv);   // [PRISM_ITEMS][PRISM_CONST]
  const ScalarTable sigma = scalar_table(m.sigma);
  const int lane = threadIdx.x, z = lane & 1;
  // items of one vertex add to the same places: neighbours in the list go to different quarters of
  // the wave, which the LDS takes one after another
  const int slot = 4 * ((lane >> 1) & 7) + (lane >> 4);
  const uint32_t minus = z ? 0u : 0x80000000u;
  const int vb = task.y, ve = task.z, ib = task.w, ie = m.vc_ptr[ve];
  const int L = m.L, nvt = ve - vb;
  const TaskColumns cols = load_columns(m, vb, nvt, lane);
  const FlatCopy<4> flat = flat_copy<JAC, 4>(m, cols, vb, nvt, lane);
  clear_windows<JAC>(m, Jw, Rw, vb, ve, max_slot, max_tv, lane);
  const double zeta = z ? G2 : G1;

  // item constants in LDS (in registers they spill): horizontal gradients, slopes of bed and H,
  // gravity's row sums, 2 visc_pref x weight x determinant x thickness and 1/H at the triangle points
  enum { LX = 0, LY = 3, BED = 6, THK = 8, GRAV = 10, WH = 12, INVH = 15 };
  double *const c_ = item_c + PRISM_CONST * slot;
  int vid[3] = {0, 0, 0}, Dv = 0, soff = 0, rloc = 0;
  uint32_t rk = 0u;
  bool act = false;
  auto gather = [&](int lev, double2 (&a)[3]) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
      a[i] = *reinterpret_cast<const double2 *>(U + 2 * (int64_t(vid[i]) * (L + 1) + lev));
  };
  const int k0 = kb > 0 ? kb - 1 : 0;
  double2 lo[3], up[3];                       // u, v of the corners on levels k and k + 1
  // a layer's upper velocities are kept for the next one's lower level, and those above loaded a
  // layer ahead; with a Jacobian the general power's constants leave no registers for either
  constexpr bool AHEAD = N3 && !PASSES;
  auto load_item = [&](int first) {
    act = first + slot < ie;
    const int item = act ? first + slot : ib;
    const int v = m.item_vtx[item], t = m.vc_idx[item], rot = m.vc_pos[item];
    Dv = m.deg[v];
    soff = m.slot_off[v];
    rloc = 2 * (v - vb);
    rk = m.item_rank[item];
    rk = (rk >> (8 * rot)) | (rk << (8 * (3 - rot)));   // the low three bytes
#pragma unroll
    for (int i = 0; i < 3; ++i) vid[i] = m.cells[3 * int64_t(t) + (i + rot >= 3 ? i + rot - 3 : i + rot)];
    if constexpr (AHEAD) {      // with the geometry's loads (one layer of 125,000 columns, R alone: 42 -> 40 us)
      gather(k0, lo);
      gather(k0 + 1, up);
    }
    double4 g[3];
    double s[3], lx[3], ly[3], c[PRISM_CONST];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      g[i] = m.geo[vid[i]];
      s[i] = m.sb[vid[i]].x;
    }
    const double x_xi = g[1].x - g[0].x, x_eta = g[2].x - g[0].x;
    const double y_xi = g[1].y - g[0].y, y_eta = g[2].y - g[0].y;
    const double det = x_xi * y_eta - x_eta * y_xi;
    const double iG = rcp64(det);
    lx[1] = y_eta * iG; lx[2] = -y_xi * iG; lx[0] = -(lx[1] + lx[2]);
    ly[1] = -x_eta * iG; ly[2] = x_xi * iG; ly[0] = -(ly[1] + ly[2]);
    const double wd = det * (1.0 / 12.0), Hm = (g[0].w + g[1].w + g[2].w) * (1.0 / 6.0);
    double sx = 0.0, sy = 0.0, Hl = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) c[BED + i] = 0.0;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      c[LX + i] = lx[i];
      c[LY + i] = ly[i];
      sx = fma(s[i], lx[i], sx); sy = fma(s[i], ly[i], sy);
      c[BED] = fma(g[i].z, lx[i], c[BED]); c[BED + 1] = fma(g[i].z, ly[i], c[BED + 1]);
      c[THK] = fma(g[i].w, lx[i], c[THK]); c[THK + 1] = fma(g[i].w, ly[i], c[THK + 1]);
      const double Hp = fma(0.5, g[i].w, Hm);     // point i: 2/3 of corner i and 1/6 of the others
      Hl = fma(i == 0 ? 2.0 / 3.0 : 1.0 / 6.0, Hp, Hl);
      c[WH + i] = 2.0 * m.visc_pref * wd * Hp;
      c[INVH + i] = rcp64(Hp);
    }
    c[GRAV] = m.rho_g * sx * (wd * Hl);
    c[GRAV + 1] = m.rho_g * sy * (wd * Hl);
    if (z == 0) {
#pragma unroll
      for (int i = 0; i < PRISM_CONST; i += 2)
        *reinterpret_cast<double2 *>(c_ + i) = make_double2(c[i], c[i + 1]);
    }
    wave_sync();
  };
  // slopes of u and v along x and y on one level
  struct Slopes { double ux, uy, vx, vy; };
  auto slopes = [&](const double2 (&a)[3]) {
    Slopes f = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const double lx = c_[LX + i], ly = c_[LY + i];
      f.ux = fma(lx, a[i].x, f.ux); f.uy = fma(ly, a[i].x, f.uy);
      f.vx = fma(lx, a[i].y, f.vx); f.vy = fma(ly, a[i].y, f.vy);
    }
    return f;
  };
  wave_sync();

  Slopes f0 = {0, 0, 0, 0};
  constexpr bool CARRY = sizeof(JT) == 4;
  AT carry[4][3];                             // lane z = 0: the upper row at the upper level of the layer below
#pragma unroll
  for (int cd = 0; cd < 4; ++cd)
#pragma unroll
    for (int j = 0; j < 3; ++j) carry[cd][j] = AT(0);

  // ---- bed friction on the lower face of the bottom layer: rows of the level-0 nodes, lane z
  // component z -------------------------------------------------------------------------------
  if (kb == 0) {
    for (int g = ib; PASSES ? g < ie : g == ib; g += PRISM_ITEMS) {
      load_item(g);
      if constexpr (!AHEAD) gather(0, lo);
      // face normal from the slopes of its z; basis products at the three points (2/3, 1/6, 1/6)
      const double bx = fma(m.sigma[0], c_[THK], c_[BED]), by = fma(m.sigma[0], c_[THK + 1], c_[BED + 1]);
      // the cell's doubled base area from its gradients: 1 / (lx_1 ly_2 - lx_2 ly_1)
      const double det = rcp64(c_[LX + 1] * c_[LY + 2] - c_[LX + 2] * c_[LY + 1]);
      const double area = det * sqrt(fma(bx, bx, fma(by, by, 1.0)));
      double be[3], q[3];
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        be[i] = m.sb[vid[i]].y;
        q[i] = sel2(z, lo[i].x, lo[i].y);
      }
      const double bm = (be[0] + be[1] + be[2]) * (1.0 / 6.0), qm = (q[0] + q[1] + q[2]) * (1.0 / 6.0);
      double Rf = 0.0, Jf[3] = {0, 0, 0};
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        const double w = area * (1.0 / 6.0) * fma(0.5, be[r], bm) * (r == 0 ? 2.0 / 3.0 : 1.0 / 6.0);
        Rf = fma(w, fma(0.5, q[r], qm), Rf);
#pragma unroll
        for (int j = 0; j < 3; ++j) Jf[j] = fma(w, r == j ? 2.0 / 3.0 : 1.0 / 6.0, Jf[j]);
      }
      if (act) {
        lds_add(Rw + rloc + z, Rf);
        if constexpr (JAC) {
          const int nl0 = nlev(0, L);
#pragma unroll
          for (int j = 0; j < 3; ++j)
            lds_add(Jw + soff + z * 2 * nl0 * Dv + int((rk >> (8 * j)) & 255u) * 2 * nl0 + z, double(AT(Jf[j])));
        }
      }
    }
  }
  if constexpr (!PASSES) {
    if (kb > 0) load_item(ib);
    if constexpr (AHEAD) {
      f0 = slopes(lo);
      asm volatile("" : "+v"(up[0].x), "+v"(up[0].y), "+v"(up[1].x), "+v"(up[1].y), "+v"(up[2].x), "+v"(up[2].y));   // waited for here, as below
    }
  }

  for (int k = k0; k < ke; ++k) {
    const int cur = k & 1, nxt = cur ^ 1;
    const double s0 = sigma[k], ds = sigma[k + 1] - s0;
    const double ids = rcp64(ds);
    for (int g = ib; PASSES ? g < ie : g == ib; g += PRISM_ITEMS) {
      if constexpr (PASSES) load_item(g);
      if constexpr (!AHEAD) {
        gather(k, lo);
        f0 = slopes(lo);
        gather(k + 1, up);
      }
      // nothing derived from the ids is kept across layers (hoisted addresses spill)
      asm volatile("" : "+v"(vid[0]), "+v"(vid[1]), "+v"(vid[2]), "+v"(Dv), "+v"(soff), "+v"(rloc), "+v"(rk));
      const Slopes f1 = slopes(up);
      // differences first: exact where the levels are close
      double du[3], dv[3];
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        du[i] = up[i].x - lo[i].x;
        dv[i] = up[i].y - lo[i].y;
        lo[i] = up[i];
      }
      if (AHEAD && k + 1 < ke) gather(k + 2, up);
      const double dum_ = (du[0] + du[1] + du[2]) * (1.0 / 6.0), dvm_ = (dv[0] + dv[1] + dv[2]) * (1.0 / 6.0);
      const double l0 = 1.0 - zeta, l1 = zeta, sz = fma(zeta, ds, s0);
      const double zxs = fma(sz, c_[THK], c_[BED]), zys = fma(sz, c_[THK + 1], c_[BED + 1]);
      const double ucx = fma(l0, f0.ux, l1 * f1.ux), ucy = fma(l0, f0.uy, l1 * f1.uy);
      const double vcx = fma(l0, f0.vx, l1 * f1.vx), vcy = fma(l0, f0.vy, l1 * f1.vy);
      f0 = f1;
      const double gx = ds * c_[GRAV], gy = ds * c_[GRAV + 1], lx0 = c_[LX], ly0 = c_[LY];
      AT S[2][4][2], B[2][4][3];     // sums of L (x, y) and, per triangle point, of L . p (signed by the lane)
      // The gradient of level a's basis function is l_a (lx, ly, 0) -+ lam (px, py, iz): the residual's
      // sums are those of the two parts (h, p), not of the two levels.  Both kernels sum alike, so
      // their residuals are the same bits (residual alone 166 -> 152 us; with the Jacobian, whose rows
      // need both levels, as long as before: 552 and 551, in an ensemble 455 and 458).
      double RH[2] = {gx, gy}, RP[2] = {0.0, 0.0};
#pragma unroll
      for (int tp = 0; tp < 3; ++tp) {
        const double iz = c_[INVH + tp] * ids, W = c_[WH + tp] * ds, lam_a = tp == 0 ? 2.0 / 3.0 : 1.0 / 6.0;
        const double dum = fma(0.5, du[tp], dum_), dvm = fma(0.5, dv[tp], dvm_);
        const double px = -zxs * iz, py = -zys * iz;        // d zeta / dx, d zeta / dy
        const double ux = fma(px, dum, ucx), uy = fma(py, dum, ucy);
        const double vx = fma(px, dvm, vcx), vy = fma(py, dvm, vcy);
        const double hz = 0.5 * iz, exx = ux, eyy = vy, exy = 0.5 * (uy + vx), exz = hz * dum, eyz = hz * dvm;
        const double qe = fma(exx, exx, fma(eyy, exx + eyy, fma(exy, exy, fma(exz, exz, fma(eyz, eyz, m.eps0_sq)))));
        // s2 = 2 mu W and t2 = mu' / mu = visc_exp / q; for n = 3, mu is q^(-1/3) and 1/q its cube
        double s2, t2;
        if constexpr (N3) {
          const double y = rcbrt64(qe);
          s2 = y * W;
          t2 = tfac * (y * y * y);
        } else {
          s2 = powq(qe, m.visc_exp) * W;
          t2 = tfac == 0.0 ? 0.0 : tfac * rcp64(qe);     // n = 1 is defined at q = 0
        }
        const double E1x = 2.0 * exx + eyy, E2y = exx + 2.0 * eyy;
        const double mx = flip(px, minus), my = flip(py, minus), mz = flip(iz, minus);
        const AT spx = AT(mx), spy = AT(my), spz = AT(mz);
        const AT e1x = AT(E1x), e1y = AT(exy), e2y = AT(E2y), e1z = AT(exz), e2z = AT(eyz), half = AT(0.5);
        const double hX = s2 * lx0, hY = s2 * ly0, s2l = s2 * lam_a;
        const double h0 = fma(E1x, hX, exy * hY), h1 = fma(exy, hX, E2y * hY);
        const double p0 = s2l * fma(E1x, px, fma(exy, py, exz * iz)), p1 = s2l * fma(exy, px, fma(E2y, py, eyz * iz));
        RH[0] += h0;
        RH[1] += h1;
        RP[0] += p0;
        RP[1] += p1;
        if constexpr (JAC) {
          // the part of A along p for either level: formed once where registers allow (the sums of
          // FP32 values take half of theirs), else from the lane-signed p that B reads
          constexpr bool KEPT = sizeof(AT) == 4;
          const double qX = s2l * px, qY = s2l * py, qZ = s2l * iz, s2m = flip(s2l, minus);
#pragma unroll
          for (int a = 0; a < 2; ++a) {
            const double l = a ? l1 : l0, sm = a ? s2m : -s2m;
            const AT Ax = AT(KEPT ? fma(l, hX, a ? qX : -qX) : fma(sm, mx, l * hX));
            const AT Ay = AT(KEPT ? fma(l, hY, a ? qY : -qY) : fma(sm, my, l * hY));
            const AT Az = AT(KEPT ? (a ? qZ : -qZ) : sm * mz);
            const AT T0 = AT(t2 * fma(l, h0, a ? p0 : -p0)), T1 = AT(t2 * fma(l, h1, a ? p1 : -p1));
            const AT hAx = half * Ax, hAy = half * Ay, hAz = half * Az;
            // L for uu, uv, vu, vv: coefficients of (bx, by, bz) in d R_(a,c) / d U_(b,d)
            const AT Lx[4] = {fma(T0, e1x, Ax + Ax), fma(T0, e1y, hAy), fma(T1, e1x, Ay), fma(T1, e1y, hAx)};
            const AT Ly[4] = {fma(T0, e1y, hAy), fma(T0, e2y, Ax), fma(T1, e1y, hAx), fma(T1, e2y, Ay + Ay)};
            const AT Lz[4] = {fma(T0, e1z, hAz), T0 * e2z, T1 * e1z, fma(T1, e2z, hAz)};
#pragma unroll
            for (int cd = 0; cd < 4; ++cd) {
              S[a][cd][0] = tp == 0 ? Lx[cd] : S[a][cd][0] + Lx[cd];
              S[a][cd][1] = tp == 0 ? Ly[cd] : S[a][cd][1] + Ly[cd];
              B[a][cd][tp] = fma(Lx[cd], spx, fma(Ly[cd], spy, Lz[cd] * spz));
            }
          }
        }
      }
      __builtin_amdgcn_s_setprio(1);
      // residual: lane z ends with row node z
      {
        const double p0 = flip(RP[0], minus), p1 = flip(RP[1], minus);
        const double k0_ = fma(G2, RH[0], p0), k1_ = fma(G2, RH[1], p1);
        const double s0_ = fma(G1, RH[0], -p0), s1_ = fma(G1, RH[1], -p1);
        const double r0 = k0_ + quad_xor<1>(s0_), r1 = k1_ + quad_xor<1>(s1_);
        if (act) {
          double *r = Rw + (z ? nxt : cur) * 2 * max_tv + rloc;
          lds_add(r, r0);
          lds_add(r + 1, r1);
        }
      }
      if constexpr (JAC) {
        AT hx[3], hy[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          hx[j] = AT(c_[LX + j]);
          hy[j] = AT(c_[LY + j]);
        }
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          // level k sits at window position 1 unless k = 0
          const int nl = a ? nlev(k + 1, L) : nlev(k, L);
          double *w = Jw + (a ? nxt : cur) * max_slot + soff + 2 * ((a ^ z) + (!a && k > 0 ? 1 : 0));
          double *wj[3];
#pragma unroll
          for (int j = 0; j < 3; ++j) wj[j] = w + int((rk >> (8 * j)) & 255u) * 2 * nl;
          const bool add = act && (a == 0 || !CARRY || z == 1 || k + 1 == L || PASSES);
          const AT lkept = AT(a ? G1 : G2), lsent = AT(a ? G2 : G1), sixth = AT(1.0 / 6.0), half = AT(0.5);
#pragma unroll
          for (int cd = 0; cd < 4; ++cd) {
            const AT bm = sixth * (B[a][cd][0] + B[a][cd][1] + B[a][cd][2]);
            AT e[3];
#pragma unroll
            for (int j = 0; j < 3; ++j) {
              const AT h = fma(hx[j], S[a][cd][0], hy[j] * S[a][cd][1]);
              const AT lb = fma(half, B[a][cd][j], bm);
              e[j] = fma(lkept, h, a ? -lb : lb) + quad_xor<1>(fma(lsent, h, a ? lb : -lb));
            }
            const int off = (cd >> 1) * 2 * nl * Dv + (cd & 1);
            if (add) {
#pragma unroll
              for (int j = 0; j < 3; ++j)     // cells are summed in FP64
                lds_add(wj[j] + off, CARRY && a == 0 ? double(e[j]) + double(carry[cd][j]) : double(e[j]));
            }
            if (CARRY && a == 1) {
#pragma unroll
              for (int j = 0; j < 3; ++j) carry[cd][j] = z || PASSES ? AT(0) : e[j];
            }
          }
        }
      }
    }
    // the next level's velocities are waited for here: after the copy-out the wait would be for its
    // stores too, which retire through the same counter
    if constexpr (AHEAD) asm volatile("" : "+v"(up[0].x), "+v"(up[0].y), "+v"(up[1].x), "+v"(up[1].y), "+v"(up[2].x), "+v"(up[2].y));
    wave_sync();
    // The copy-out runs at raised wave priority (2), the window adds at 1: the copy-out's LDS reads
    // and streaming stores then issue ahead of the other waves' work instead of queuing behind it.
    __builtin_amdgcn_s_setprio(2);
    copy_level<JAC>(flat, cols, k, cur, k >= kb, vb, nvt, L, Jw, Rw, max_slot, max_tv, lane, R, J);
    if (k == L - 1) copy_level<JAC>(flat, cols, L, nxt, true, vb, nvt, L, Jw, Rw, max_slot, max_tv, lane, R, J);
    wave_sync();
    __builtin_amdgcn_s_setprio(0);
  }
}

// ---- hexahedra ----------------------------------------------------------------------------
// Four lanes per item, one per Gauss point of the base quadrilateral (two zeta points each): a
// lane evaluates the physics of its two points once, and the entries of the item's rows are
// formed from its own point and summed over the four lanes by two exchanges, after which every
// lane holds a quarter of them.
// Nothing of the Jacobian stays in registers across points (one lane per item needed 64
// accumulators and ran one wave per SIMD with 40 of its 64 lanes busy, the window budget being
// ten columns), and the horizontal map, gradients and the slopes of bed and thickness at a lane's
// point are constants of the whole column.  Bound by FP64 issue: about 1000 vector instructions
// a layer.  30,000 columns of 7 layers (210,000 hexahedra), FP64 R+J: 294 -> 121 us; 2000
// hexahedra (with the levels split over blocks): 68 -> 10.6 us.  Compiled for three or four waves
// per SIMD the column constants spill: 333 and 572 us.  For n != 3 the general power's constants
// beside the velocities loaded ahead spill 47 registers (27 with FP32 values); with n = 2.5 the
// 30,000 columns take 182 us (152), 340 (331) with one lane per item.
//
// Exchanges without selections: lane bits b0 = lane & 1, b1 = lane >> 1 & 1.  A lane forms the
// entries at level b0 as "kept" and at the other level as "sent" (lane-constant weights l_b0 and
// l_(1-b0)), and walks the corners in the order jj -> (jj + 2 b1) & 3, so that its first two
// are kept in the second exchange.  It ends with corners 2 b1 and 2 b1 + 1 at level b0.
constexpr int HEX_ITEMS = WAVE / 4;   // items per pass of a wave

// The levels kb <= k < ke of a task's columns (and level L if ke = L).  kb > 0 starts with layer
// kb - 1, whose lower rows belong to the range below and are dropped.  PASSES: the task holds
// more items than one pass of a wave takes (a vertex in more cells than that is a task of its
// own), so the item constants are reloaded for every layer and pass.
template <bool JAC, class JT, bool N3, bool PASSES>
__device__ __forceinline__ void hex_task(const MeshView &m, const int4 task, const double *__restrict__ U,
                                         double *__restrict__ R, JT *__restrict__ J, int picard, int max_slot,
                                         int max_tv, int kb, int ke, unsigned char *smem) {
  using AT = JT;   // derivative arithmetic type
  double *Jw = reinterpret_cast<double *>(smem);                                               // [2][max_slot]
  double *Rw = reinterpret_cast<double *>(smem + (JAC ? 2 * size_t(max_slot) * sizeof(double) : 0));  // [2][2 max_tv]
  const double tfac = picard ? 0.0 : 2.0 * m.visc_exp;   // 2 mu' = 2 visc_exp mu / q
  const ScalarTable sigma = scalar_table(m.sigma);
  const int lane = threadIdx.x, b0 = lane & 1, b1 = (lane >> 1) & 1;
  const int slot = 4 * ((lane >> 2) & 3) + (lane >> 4);   // as for prisms
  const int vb = task.y, ve = task.z, ib = task.w, ie = m.vc_ptr[ve];
  const int L = m.L, nvt = ve - vb;
  const TaskColumns cols = load_columns(m, vb, nvt, lane);
  // this lane's base point and its basis, corners in the lane's order
  const double xi = b0 ? G2 : G1, eta = b1 ? G2 : G1, mx = 1.0 - xi, my = 1.0 - eta;
  double lam[4], lx[4], ly[4];
  {
    const double la[4] = {mx * my, xi * my, xi * eta, mx * eta};
#pragma unroll
    for (int j = 0; j < 4; ++j) lam[j] = b1 ? la[(j + 2) & 3] : la[j];
  }
  const FlatCopy<4> flat = flat_copy<JAC, 4>(m, cols, vb, nvt, lane);
  clear_windows<JAC>(m, Jw, Rw, vb, ve, max_slot, max_tv, lane);

  // item constants: corner ids, gradients at the lane's point, weight x determinant x thickness,
  // the slopes of s, bed and H there, and the item's own corner's basis
  int vid[4], Dv = 0, soff = 0, rloc = 0;
  uint32_t rk = 0u;
  bool act = false;
  double wH = 0, sx = 0, sy = 0, iH = 0, Bx = 0, By = 0, Hx = 0, Hy = 0, lam_a = 0, lxa = 0, lya = 0;
  auto load_item = [&](int first) {
    act = first + slot < ie;
    const int item = act ? first + slot : ib;
    const int v = m.item_vtx[item], t = m.vc_idx[item], al = (int(m.vc_pos[item]) - 2 * b1) & 3;
    Dv = m.deg[v];
    soff = m.slot_off[v];
    rloc = 2 * (v - vb);
    rk = m.item_rank[item];
    if (b1) rk = (rk >> 16) | (rk << 16);
    const int4 c4 = *reinterpret_cast<const int4 *>(m.cells + 4 * int64_t(t));
    vid[0] = b1 ? c4.z : c4.x;
    vid[1] = b1 ? c4.w : c4.y;
    vid[2] = b1 ? c4.x : c4.z;
    vid[3] = b1 ? c4.y : c4.w;
    double4 g[4];
    double s[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      g[j] = m.geo[vid[j]];
      s[j] = m.sb[vid[j]].x;
    }
    // derivatives of the basis along xi and eta: (-my, my, eta, -eta), (-mx, -xi, xi, mx), the
    // second pair's signs flipped where the corner order starts at the opposite corner
    const double p = b1 ? eta : my, q = b1 ? my : eta, sg = b1 ? -1.0 : 1.0;
    const double u = b1 ? xi : mx, w = b1 ? mx : xi;
    const double dx[4] = {-sg * p, sg * p, sg * q, -sg * q}, dy[4] = {-sg * u, -sg * w, sg * w, sg * u};
    double x_xi = 0, x_eta = 0, y_xi = 0, y_eta = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const double x = g[j].x - g[0].x, y = g[j].y - g[0].y;
      x_xi = fma(x, dx[j], x_xi); x_eta = fma(x, dy[j], x_eta);
      y_xi = fma(y, dx[j], y_xi); y_eta = fma(y, dy[j], y_eta);
    }
    const double det = x_xi * y_eta - x_eta * y_xi;
    const double iG = rcp64(det);
    const double i00 = y_eta * iG, i01 = -x_eta * iG, i10 = -y_xi * iG, i11 = x_xi * iG;
    double Hq = 0.0;
    sx = sy = Bx = By = Hx = Hy = 0.0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      lx[j] = dx[j] * i00 + dy[j] * i10;
      ly[j] = dx[j] * i01 + dy[j] * i11;
      sx = fma(s[j], lx[j], sx); sy = fma(s[j], ly[j], sy);
      Bx = fma(g[j].z, lx[j], Bx); By = fma(g[j].z, ly[j], By);
      Hx = fma(g[j].w, lx[j], Hx); Hy = fma(g[j].w, ly[j], Hy);
      Hq = fma(g[j].w, lam[j], Hq);
    }
    wH = 0.125 * det * Hq;
    iH = rcp64(Hq);
    lam_a = sel4(al, lam[0], lam[1], lam[2], lam[3]);
    lxa = sel4(al, lx[0], lx[1], lx[2], lx[3]);
    lya = sel4(al, ly[0], ly[1], ly[2], ly[3]);
    return make_double4(x_xi, x_eta, y_xi, y_eta);
  };
  auto gather = [&](int lev, double2 (&a)[4]) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      a[j] = *reinterpret_cast<const double2 *>(U + 2 * (int64_t(vid[j]) * (L + 1) + lev));
  };
  // slopes of u and v along x and y at the lane's point on one level
  struct Slopes { double ux, uy, vx, vy; };
  auto slopes = [&](const double2 (&a)[4]) {
    Slopes f = {0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      f.ux = fma(lx[j], a[j].x, f.ux); f.uy = fma(ly[j], a[j].x, f.uy);
      f.vx = fma(lx[j], a[j].y, f.vx); f.vy = fma(ly[j], a[j].y, f.vy);
    }
    return f;
  };
  auto sum4 = [](double v) {   // over the item's four lanes, the same in each
    v += quad_xor<1>(v);
    return v + quad_xor<2>(v);
  };
  wave_sync();

  const int k0 = kb > 0 ? kb - 1 : 0;
  double2 lo[4], up[4];                     // u, v of the corners on levels k and k + 1
  Slopes f0 = {0, 0, 0, 0};

  // ---- bed friction on the lower face of the bottom layer: rows of the level-0 nodes -----------
  if (kb == 0) {
    for (int g = ib; PASSES ? g < ie : g == ib; g += HEX_ITEMS) {
      const double4 map = load_item(g);
      gather(0, lo);
      double br = 0.0, ur = 0.0, vr = 0.0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        br = fma(m.sb[vid[j]].y, lam[j], br);
        ur = fma(lo[j].x, lam[j], ur);
        vr = fma(lo[j].y, lam[j], vr);
      }
      // tangents of the face: z along x and y at fixed zeta, through the map
      const double bx = fma(m.sigma[0], Hx, Bx), by = fma(m.sigma[0], Hy, By);
      const double txx = map.x, tyx = map.y, txy = map.z, tyy = map.w;
      const double txz = txx * bx + txy * by, tyz = tyx * bx + tyy * by;
      const double nx_ = txy * tyz - txz * tyy, ny_ = txz * tyx - txx * tyz, nz_ = txx * tyy - txy * tyx;
      const double wa = 0.25 * sqrt(nx_ * nx_ + ny_ * ny_ + nz_ * nz_) * br * lam_a;
      const double Rf0 = sum4(wa * ur), Rf1 = sum4(wa * vr);
      const double h0 = wa * lam[0] + quad_xor<2>(wa * lam[2]), h1 = wa * lam[1] + quad_xor<2>(wa * lam[3]);
      const double own = (b0 ? h1 : h0) + quad_xor<1>(b0 ? h0 : h1);   // corner 2 b1 + b0
      if (act) {
        if (b1 == 0) lds_add(Rw + rloc + b0, b0 ? Rf1 : Rf0);
        if constexpr (JAC) {
          const int nl0 = nlev(0, L), r0 = int((rk >> (8 * b0)) & 255u);
          lds_add(Jw + soff + r0 * 2 * nl0, double(AT(own)));
          lds_add(Jw + soff + 2 * nl0 * Dv + r0 * 2 * nl0 + 1, double(AT(own)));
        }
      }
    }
  }
  if constexpr (!PASSES) {
    if (kb > 0) load_item(ib);
    gather(k0, lo);
    f0 = slopes(lo);
    gather(k0 + 1, up);
    asm volatile("" : "+v"(up[0].x), "+v"(up[0].y), "+v"(up[1].x), "+v"(up[1].y), "+v"(up[2].x), "+v"(up[2].y), "+v"(up[3].x), "+v"(up[3].y));   // waited for here, as below
  }

  // lane-constant weights of the kept and sent levels at the two zeta points, and signed basis
  const AT lk[2] = {AT(b0 ? G1 : 1.0 - G1), AT(b0 ? G2 : 1.0 - G2)}, ls[2] = {AT(1) - lk[0], AT(1) - lk[1]};
  for (int k = k0; k < ke; ++k) {
    const int cur = k & 1, nxt = cur ^ 1;
    const double s0 = sigma[k], ds = sigma[k + 1] - s0;
    const double ids = rcp64(ds);
    for (int g = ib; PASSES ? g < ie : g == ib; g += HEX_ITEMS) {
      if constexpr (PASSES) {
        load_item(g);
        gather(k, lo);
        f0 = slopes(lo);
        gather(k + 1, up);
      }
      const Slopes f1 = slopes(up);
      double dum = 0.0, dvm = 0.0;          // differences first: exact where the levels are close
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        dum = fma(lam[j], up[j].x - lo[j].x, dum);
        dvm = fma(lam[j], up[j].y - lo[j].y, dvm);
        lo[j] = up[j];
      }
      if (!PASSES && k + 1 < ke) gather(k + 2, up);
      const double iz = iH * ids, Wz = wH * ds;
      const double exz = 0.5 * (iz * dum), eyz = 0.5 * (iz * dvm);
      // the physics of the lane's two points
      double s2[2], t2[2], E1x[2], Exy[2], E2y[2], px[2], py[2];
#pragma unroll
      for (int zi = 0; zi < 2; ++zi) {
        const double zeta = zi ? G2 : G1, l0 = 1.0 - zeta, l1 = zeta;
        const double sz = fma(zeta, ds, s0);
        px[zi] = -fma(sz, Hx, Bx) * iz;         // d zeta / dx, d zeta / dy
        py[zi] = -fma(sz, Hy, By) * iz;
        const double ux = fma(l0, f0.ux, fma(l1, f1.ux, px[zi] * dum));
        const double uy = fma(l0, f0.uy, fma(l1, f1.uy, py[zi] * dum));
        const double vx = fma(l0, f0.vx, fma(l1, f1.vx, px[zi] * dvm));
        const double vy = fma(l0, f0.vy, fma(l1, f1.vy, py[zi] * dvm));
        const double exx = ux, eyy = vy, exy = 0.5 * (uy + vx);
        const double qq = exx * exx + eyy * eyy + exx * eyy + exy * exy + exz * exz + eyz * eyz;
        const double qe = qq + m.eps0_sq;
        double mu;
        if constexpr (N3) mu = m.visc_pref * rcbrt64(qe);
        else mu = m.visc_pref * powq(qe, m.visc_exp);
        s2[zi] = 2.0 * mu * Wz;
        t2[zi] = !N3 && tfac == 0.0 ? 0.0 : (mu * rcp64(qe)) * (tfac * Wz);     // n = 1 is defined at q = 0
        E1x[zi] = 2.0 * exx + eyy;
        Exy[zi] = exy;
        E2y[zi] = exx + 2.0 * eyy;
      }
      f0 = f1;
      const double gvx = Wz * m.rho_g * sx, gvy = Wz * m.rho_g * sy;
      const AT iza = AT(iz), e1z = AT(exz), e2z = AT(eyz), half = AT(0.5);
      const int r0 = int(rk & 255u), r1 = int((rk >> 8) & 255u);
      double Rl[2][2] = {{0, 0}, {0, 0}};
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        // row node a: its gradient, residual, and 2 mu W grad N_a and 2 mu' W E_c . grad N_a
        AT A[2][3], T[2][2];
#pragma unroll
        for (int zi = 0; zi < 2; ++zi) {
          const double zeta = zi ? G2 : G1, l = a ? zeta : 1.0 - zeta, la = a ? lam_a : -lam_a;
          const double ax = fma(l, lxa, la * px[zi]), ay = fma(l, lya, la * py[zi]), az = la * iz;
          const double g0 = E1x[zi] * ax + Exy[zi] * ay + exz * az, g1 = Exy[zi] * ax + E2y[zi] * ay + eyz * az;
          const double nb = lam_a * l;
          Rl[a][0] = fma(s2[zi], g0, fma(gvx, nb, Rl[a][0]));
          Rl[a][1] = fma(s2[zi], g1, fma(gvy, nb, Rl[a][1]));
          if constexpr (JAC) {
            A[zi][0] = AT(s2[zi] * ax); A[zi][1] = AT(s2[zi] * ay); A[zi][2] = AT(s2[zi] * az);
            T[zi][0] = AT(t2[zi] * g0); T[zi][1] = AT(t2[zi] * g1);
          }
        }
        if constexpr (JAC) {
          // where the lane's two entries of a row go: level k sits at window position 1 unless k = 0
          const int nl = a ? nlev(k + 1, L) : nlev(k, L);
          double *w = Jw + (a ? nxt : cur) * max_slot + soff + 2 * (b0 + (!a && k > 0 ? 1 : 0));
          double *w0 = w + r0 * 2 * nl, *w1 = w + r1 * 2 * nl;
#pragma unroll
          for (int cd = 0; cd < 4; ++cd) {
            const int c = cd >> 1, d = cd & 1;
            AT Kx = AT(0), Ky = AT(0), Sx = AT(0), Sy = AT(0), Bs = AT(0);
#pragma unroll
            for (int zi = 0; zi < 2; ++zi) {
              const AT Ax = A[zi][0], Ay = A[zi][1], Az = A[zi][2], Tc = T[zi][c];
              // coefficients of (bx, by, bz) in d R_(a,c) / d U_(b,d)
              const AT ex = AT(d ? Exy[zi] : E1x[zi]), ey = AT(d ? E2y[zi] : Exy[zi]), ez = d ? e2z : e1z;
              AT Lx, Ly, Lz;
              if (cd == 0) { Lx = fma(Tc, ex, Ax + Ax); Ly = fma(Tc, ey, half * Ay); Lz = fma(Tc, ez, half * Az); }
              else if (cd == 1) { Lx = fma(Tc, ex, half * Ay); Ly = fma(Tc, ey, Ax); Lz = Tc * ez; }
              else if (cd == 2) { Lx = fma(Tc, ex, Ay); Ly = fma(Tc, ey, half * Ax); Lz = Tc * ez; }
              else { Lx = fma(Tc, ex, half * Ax); Ly = fma(Tc, ey, Ay + Ay); Lz = fma(Tc, ez, half * Az); }
              Kx = fma(lk[zi], Lx, Kx); Ky = fma(lk[zi], Ly, Ky);
              Sx = fma(ls[zi], Lx, Sx); Sy = fma(ls[zi], Ly, Sy);
              Bs = fma(Lx, AT(px[zi]), fma(Ly, AT(py[zi]), fma(Lz, iza, Bs)));
            }
            const AT Bk = b0 ? Bs : -Bs;      // the upper level's gradient carries +lam grad zeta
            AT r[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const AT hx = AT(lx[j]), hy = AT(ly[j]), lb = AT(lam[j]) * Bk;
              r[j] = fma(hx, Kx, fma(hy, Ky, lb)) + quad_xor<1>(fma(hx, Sx, fma(hy, Sy, -lb)));
            }
            const AT o0 = r[0] + quad_xor<2>(r[2]), o1 = r[1] + quad_xor<2>(r[3]);
            if (act) {
              lds_add(w0 + c * 2 * nl * Dv + d, double(o0));
              lds_add(w1 + c * 2 * nl * Dv + d, double(o1));
            }
          }
        }
      }
      // residual: the lane ends with row node b0, component b1
      {
        const double k0_ = b0 ? Rl[1][0] : Rl[0][0], k1_ = b0 ? Rl[1][1] : Rl[0][1];
        const double s0_ = b0 ? Rl[0][0] : Rl[1][0], s1_ = b0 ? Rl[0][1] : Rl[1][1];
        const double q0 = k0_ + quad_xor<1>(s0_), q1 = k1_ + quad_xor<1>(s1_);
        const double own = (b1 ? q1 : q0) + quad_xor<2>(b1 ? q0 : q1);
        if (act) lds_add(Rw + (b0 ? nxt : cur) * 2 * max_tv + rloc + b1, own);
      }
    }
    // the next level's velocities are waited for here: after the copy-out the wait would be for its
    // stores too, which retire through the same counter
    if constexpr (!PASSES) asm volatile("" : "+v"(up[0].x), "+v"(up[0].y), "+v"(up[1].x), "+v"(up[1].y), "+v"(up[2].x), "+v"(up[2].y), "+v"(up[3].x), "+v"(up[3].y));
    wave_sync();
    __builtin_amdgcn_s_setprio(2);
    copy_level<JAC>(flat, cols, k, cur, k >= kb, vb, nvt, L, Jw, Rw, max_slot, max_tv, lane, R, J);
    if (k == L - 1) copy_level<JAC>(flat, cols, L, nxt, true, vb, nvt, L, Jw, Rw, max_slot, max_tv, lane, R, J);
    wave_sync();
    __builtin_amdgcn_s_setprio(0);
  }
}

// ---- tetrahedra --------------------------------------------------------------------------
// Each layer of a base triangle's prism is split into three tetrahedra by the global order of its
// corners (taken sorted, so corner r has the r-th smallest vertex id): (0,1,2,0'), (1,2,0',1'),
// (2,0',1',2'), primes one level up.  Linear basis: gradients, strain rate and viscosity are
// constant on a tetrahedron, so every integral is exact (V times the integrand, int phi_a = V/4).
//
// Tetrahedron q holds the vertical edge of column q and one node of each other column j: its lower
// one for j > q, its upper one for j < q.  With lam_j the barycentric coordinates of the base
// triangle, h_j their gradients, and z = Pi_q(x, y) the plane through the nodes but q's upper
// one, the upper node of q has the basis (z - Pi_q) / dz_q, of gradient P_q = (-grad Pi_q, 1) / dz_q,
// the lower one lam_q minus that, and the others lam_j.  So a column's entries are those of a
// prism with one point per tetrahedron: h_j . L, and -+ P_q . L for j = q, and the slopes of u, v
// and z on the planes follow from one tetrahedron to the next by adding h_q times column q's rise.
//
// One lane per item.  Row node (r, lower) lies in tetrahedra q <= r, (r, upper) in q >= r; r
// varies by lane, so both rows are formed on all three tetrahedra with weights 0 and 1.  The
// physics of the three stays in registers while one row node and component pair after the other
// is formed and added, without accumulators.  With a Jacobian it is bound by the LDS adds (82% of
// the kernel's time before the structural zeros were left out).  Ice sheet of 7.5M tetrahedra,
// FP64 R+J: 715 us with each tetrahedron's gradients from cross products into 48 accumulators,
// 469 us with the planes, 439 us without adding structural zeros, 413 us with tasks that let
// eight waves share a compute unit's LDS.
constexpr int TET_WAVES = 2;
constexpr int TET_CONST = 10;      // FP64 constants of an item in LDS

template <bool JAC, class JT, bool N3>
__device__ __forceinline__ void tet_task(const MeshView &m, const int4 task, const double *__restrict__ U,
                                         double *__restrict__ R, JT *__restrict__ J, int picard, int max_slot,
                                         int max_tv, int kb, int ke, unsigned char *smem) {
  using AT = JT;   // derivative arithmetic type
  double *Jw = reinterpret_cast<double *>(smem);                                               // [2][max_slot]
  double *Rw = reinterpret_cast<double *>(smem + (JAC ? 2 * size_t(max_slot) * sizeof(double) : 0));  // [2][2 max_tv]
  // item constants in LDS (in registers they spill), [constant][lane]: slopes of bed and H, H at the
  // corners, 2/3 visc_pref x base area, gravity's x and y scale
  enum { BED = 0, THK = 2, HC = 4, VISC = 7, GRAV = 8 };
  double *const c_ = Rw + 4 * size_t(max_tv) + threadIdx.x;
  const double tfac = picard ? 0.0 : m.visc_exp;
  const ScalarTable sigma = scalar_table(m.sigma);
  const int lane = threadIdx.x, slot = 4 * (lane & 15) + (lane >> 4);   // as for prisms
  const int vb = task.y, ve = task.z, ib = task.w, ie = m.vc_ptr[ve];
  const int L = m.L, nvt = ve - vb;
  const TaskColumns cols = load_columns(m, vb, nvt, lane);
  const FlatCopy<8> flat = flat_copy<JAC, 8>(m, cols, vb, nvt, lane);
  clear_windows<JAC>(m, Jw, Rw, vb, ve, max_slot, max_tv, lane);

  // item constants, corners sorted by vertex id
  const bool act = ib + slot < ie;
  const int item = act ? ib + slot : ib;
  const int v = m.item_vtx[item], t = m.vc_idx[item];
  int Dv = m.deg[v], soff = m.slot_off[v], rloc = 2 * (v - vb);
  int vid[3];
  uint32_t rk = 0u;
  int own;
  {
    int c[3];
    const uint32_t ranks = m.item_rank[item];
#pragma unroll
    for (int i = 0; i < 3; ++i) c[i] = m.cells[3 * int64_t(t) + i];
    int at[3];    // sorted position of each corner
#pragma unroll
    for (int i = 0; i < 3; ++i) at[i] = int(c[i] > c[(i + 1) % 3]) + int(c[i] > c[(i + 2) % 3]);
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      vid[r] = at[0] == r ? c[0] : at[1] == r ? c[1] : c[2];
      const uint32_t b = at[0] == r ? ranks : at[1] == r ? ranks >> 8 : ranks >> 16;
      rk |= (b & 255u) << (8 * r);
    }
    const int al = m.vc_pos[item];
    own = al == 0 ? at[0] : al == 1 ? at[1] : at[2];
  }
  double lx[3], ly[3], hx, hy;
  // 0/1 weights: the own corner lies at or above q (a_q: lower row), below q (1 - a_q for q > 0: upper row)
  const double a1 = own >= 1 ? 1.0 : 0.0, a2 = own >= 2 ? 1.0 : 0.0;
  {
    double4 g[3];
    double sx = 0, sy = 0, Bx = 0, By = 0, Hx = 0, Hy = 0;
#pragma unroll
    for (int i = 0; i < 3; ++i) g[i] = m.geo[vid[i]];
    const double x_xi = g[1].x - g[0].x, x_eta = g[2].x - g[0].x;
    const double y_xi = g[1].y - g[0].y, y_eta = g[2].y - g[0].y;
    const double det = x_xi * y_eta - x_eta * y_xi;      // either sign: the sorted corners may run clockwise
    const double iG = rcp64(det);
    lx[1] = y_eta * iG; lx[2] = -y_xi * iG; lx[0] = -(lx[1] + lx[2]);
    ly[1] = -x_eta * iG; ly[2] = x_xi * iG; ly[0] = -(ly[1] + ly[2]);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const double s = m.sb[vid[i]].x;
      sx = fma(s, lx[i], sx); sy = fma(s, ly[i], sy);
      Bx = fma(g[i].z, lx[i], Bx); By = fma(g[i].z, ly[i], By);
      Hx = fma(g[i].w, lx[i], Hx); Hy = fma(g[i].w, ly[i], Hy);
      c_[(HC + i) * WAVE] = g[i].w;
    }
    const double area2 = fabs(det), grav = m.rho_g * area2 * (1.0 / 24.0);
    c_[BED * WAVE] = Bx; c_[(BED + 1) * WAVE] = By;
    c_[THK * WAVE] = Hx; c_[(THK + 1) * WAVE] = Hy;
    c_[VISC * WAVE] = area2 * (1.0 / 3.0) * m.visc_pref;
    c_[GRAV * WAVE] = grav * sx; c_[(GRAV + 1) * WAVE] = grav * sy;
    hx = own == 0 ? lx[0] : own == 1 ? lx[1] : lx[2];
    hy = own == 0 ? ly[0] : own == 1 ? ly[1] : ly[2];
  }
  auto gather = [&](int lev, double2 (&a)[3]) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
      a[i] = *reinterpret_cast<const double2 *>(U + 2 * (int64_t(vid[i]) * (L + 1) + lev));
  };
  wave_sync();

  const int k0 = kb > 0 ? kb - 1 : 0;
  double2 lo[3], up[3];                       // u, v of the corners on levels k and k + 1
  // ---- bed friction on the lower face of the bottom layer: rows of the level-0 nodes -----------
  if (kb == 0) {
    gather(0, lo);
    const double bx = fma(sigma[0], c_[THK * WAVE], c_[BED * WAVE]);
    const double by = fma(sigma[0], c_[(THK + 1) * WAVE], c_[(BED + 1) * WAVE]);
    const double area = fabs(rcp64(lx[1] * ly[2] - lx[2] * ly[1])) * sqrt(fma(bx, bx, fma(by, by, 1.0)));
    double be[3], Rf0 = 0.0, Rf1 = 0.0, Jf[3] = {0, 0, 0};
#pragma unroll
    for (int i = 0; i < 3; ++i) be[i] = m.sb[vid[i]].y;
    const double bm = (be[0] + be[1] + be[2]) * (1.0 / 6.0);
    const double um = (lo[0].x + lo[1].x + lo[2].x) * (1.0 / 6.0), vm = (lo[0].y + lo[1].y + lo[2].y) * (1.0 / 6.0);
#pragma unroll
    for (int r = 0; r < 3; ++r) {     // point r: 2/3 of corner r and 1/6 of the others
      const double w = area * (1.0 / 6.0) * fma(0.5, be[r], bm) * (r == own ? 2.0 / 3.0 : 1.0 / 6.0);
      Rf0 = fma(w, fma(0.5, lo[r].x, um), Rf0);
      Rf1 = fma(w, fma(0.5, lo[r].y, vm), Rf1);
#pragma unroll
      for (int j = 0; j < 3; ++j) Jf[j] = fma(w, r == j ? 2.0 / 3.0 : 1.0 / 6.0, Jf[j]);
    }
    if (act) {
      lds_add(Rw + rloc, Rf0);
      lds_add(Rw + rloc + 1, Rf1);
      if constexpr (JAC) {
        const int nl0 = nlev(0, L);
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int j = 0; j < 3; ++j)
            lds_add(Jw + soff + c * 2 * nl0 * Dv + int((rk >> (8 * j)) & 255u) * 2 * nl0 + c, double(AT(Jf[j])));
      }
    }
  }
  constexpr bool AHEAD = N3;      // as for prisms
  if constexpr (AHEAD) {
    gather(k0, lo);
    gather(k0 + 1, up);
    asm volatile("" : "+v"(up[0].x), "+v"(up[0].y), "+v"(up[1].x), "+v"(up[1].y), "+v"(up[2].x), "+v"(up[2].y));
  }

  for (int k = k0; k < ke; ++k) {
    const int cur = k & 1, nxt = cur ^ 1;
    const double s0 = sigma[k], ds = sigma[k + 1] - s0;
    asm volatile("" : "+v"(vid[0]), "+v"(vid[1]), "+v"(vid[2]), "+v"(Dv), "+v"(soff), "+v"(rloc), "+v"(rk));
    if constexpr (!AHEAD) {
      gather(k, lo);
      gather(k + 1, up);
    }
    double ux = 0, uy = 0, vx = 0, vy = 0;      // slopes of u and v on the plane of tetrahedron q
    double zx = fma(s0, c_[THK * WAVE], c_[BED * WAVE]), zy = fma(s0, c_[(THK + 1) * WAVE], c_[(BED + 1) * WAVE]);
    const double visc = c_[VISC * WAVE] * ds;
    double dz[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      ux = fma(lx[i], lo[i].x, ux); uy = fma(ly[i], lo[i].x, uy);
      vx = fma(lx[i], lo[i].y, vx); vy = fma(ly[i], lo[i].y, vy);
    }
    // the physics of the three tetrahedra
    double s2[3], t2[3], E1x[3], Exy[3], E2y[3], Exz[3], Eyz[3], Px[3], Py[3], Pz[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const double du = up[q].x - lo[q].x, dv = up[q].y - lo[q].y, Hq = c_[(HC + q) * WAVE];
      dz[q] = ds * Hq;
      Pz[q] = rcp64(dz[q]);
      Px[q] = -zx * Pz[q];
      Py[q] = -zy * Pz[q];
      const double exx = fma(Px[q], du, ux), eyy = fma(Py[q], dv, vy);
      const double exy = 0.5 * (fma(Py[q], du, uy) + fma(Px[q], dv, vx));
      const double exz = 0.5 * (Pz[q] * du), eyz = 0.5 * (Pz[q] * dv);
      const double qe = fma(exx, exx, fma(eyy, exx + eyy, fma(exy, exy, fma(exz, exz, fma(eyz, eyz, m.eps0_sq)))));
      const double W = visc * Hq;     // 2 visc_pref V
      if constexpr (N3) {      // mu is q^(-1/3) and 1/q its cube
        const double y = rcbrt64(qe);
        s2[q] = y * W;
        t2[q] = (s2[q] * tfac) * (y * y * y);
      } else {
        s2[q] = powq(qe, m.visc_exp) * W;
        t2[q] = tfac == 0.0 ? 0.0 : (s2[q] * tfac) * rcp64(qe);     // n = 1 is defined at q = 0
      }
      E1x[q] = 2.0 * exx + eyy; Exy[q] = exy; E2y[q] = exx + 2.0 * eyy; Exz[q] = exz; Eyz[q] = eyz;
      if (q < 2) {      // on to the next plane: column q's node moves up
        ux = fma(lx[q], du, ux); uy = fma(ly[q], du, uy);
        vx = fma(lx[q], dv, vx); vy = fma(ly[q], dv, vy);
        zx = fma(lx[q], dz[q], zx); zy = fma(ly[q], dz[q], zy);
      }
      lo[q] = up[q];
    }
    if (AHEAD && k + 1 < ke) gather(k + 2, up);
    __builtin_amdgcn_s_setprio(1);
    const int r0 = int(rk & 255u), r1 = int((rk >> 8) & 255u), r2 = int((rk >> 16) & 255u);
    const double in[2][3] = {{1.0, a1, a2}, {0.0, 1.0 - a1, 1.0 - a2}};       // row node's own gradient h
    const double rows[2] = {dz[0] + a1 * dz[1] + a2 * dz[2], (1.0 - a1) * dz[0] + (1.0 - a2) * dz[1] + dz[2]};
    const double apex[3] = {1.0 - a1, a1 - a2, a2};                          // and -+ P on its vertical edge
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      double Ra0 = rows[a] * c_[GRAV * WAVE], Ra1 = rows[a] * c_[(GRAV + 1) * WAVE];
      AT A[3][3], T[3][2];
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const double w = a ? apex[q] : -apex[q];
        const double ax = fma(w, Px[q], in[a][q] * hx), ay = fma(w, Py[q], in[a][q] * hy), az = w * Pz[q];
        const double g0 = E1x[q] * ax + Exy[q] * ay + Exz[q] * az, g1 = Exy[q] * ax + E2y[q] * ay + Eyz[q] * az;
        Ra0 = fma(s2[q], g0, Ra0);
        Ra1 = fma(s2[q], g1, Ra1);
        if constexpr (JAC) {
          A[q][0] = AT(s2[q] * ax); A[q][1] = AT(s2[q] * ay); A[q][2] = AT(s2[q] * az);
          T[q][0] = AT(t2[q] * g0); T[q][1] = AT(t2[q] * g1);
        }
      }
      if (act) {
        double *r = Rw + (a ? nxt : cur) * 2 * max_tv + rloc;
        lds_add(r, Ra0);
        lds_add(r + 1, Ra1);
      }
      if constexpr (JAC) {
        const AT half = AT(0.5);
        const int nl = a ? nlev(k + 1, L) : nlev(k, L);
        // level k sits at window position 1 unless k = 0
        double *w = Jw + (a ? nxt : cur) * max_slot + soff + (!a && k > 0 ? 2 : 0);
        double *w0 = w + r0 * 2 * nl, *w1 = w + r1 * 2 * nl, *w2 = w + r2 * 2 * nl;
#pragma unroll
        for (int cd = 0; cd < 4; ++cd) {
          const int c = cd >> 1, d = cd & 1;
          AT Lx[3], Ly[3], B[3];
#pragma unroll
          for (int q = 0; q < 3; ++q) {
            const AT Ax = A[q][0], Ay = A[q][1], Az = A[q][2], Tc = T[q][c];
            // coefficients of (bx, by, bz) in d R_(a,c) / d U_(b,d)
            const AT ex = AT(d ? Exy[q] : E1x[q]), ey = AT(d ? E2y[q] : Exy[q]), ez = AT(d ? Eyz[q] : Exz[q]);
            AT Lz;
            if (cd == 0) { Lx[q] = fma(Tc, ex, Ax + Ax); Ly[q] = fma(Tc, ey, half * Ay); Lz = fma(Tc, ez, half * Az); }
            else if (cd == 1) { Lx[q] = fma(Tc, ex, half * Ay); Ly[q] = fma(Tc, ey, Ax); Lz = Tc * ez; }
            else if (cd == 2) { Lx[q] = fma(Tc, ex, Ay); Ly[q] = fma(Tc, ey, half * Ax); Lz = Tc * ez; }
            else { Lx[q] = fma(Tc, ex, half * Ax); Ly[q] = fma(Tc, ey, Ay + Ay); Lz = fma(Tc, ez, half * Az); }
            B[q] = fma(Lx[q], AT(Px[q]), fma(Ly[q], AT(Py[q]), Lz * AT(Pz[q])));
          }
          // column j's lower node lies in tetrahedra q <= j, its upper one in q >= j
          const AT x01 = Lx[0] + Lx[1], y01 = Ly[0] + Ly[1], x12 = Lx[1] + Lx[2], y12 = Ly[1] + Ly[2];
          const AT l0 = fma(AT(lx[0]), Lx[0], fma(AT(ly[0]), Ly[0], -B[0]));
          const AT l1 = fma(AT(lx[1]), x01, fma(AT(ly[1]), y01, -B[1]));
          const AT l2 = fma(AT(lx[2]), x01 + Lx[2], fma(AT(ly[2]), y01 + Ly[2], -B[2]));
          const AT u0 = fma(AT(lx[0]), x12, fma(AT(ly[0]), y12, B[0]));
          const AT u1 = fma(AT(lx[1]), Lx[2], fma(AT(ly[1]), Ly[2], B[1]));
          const AT u2 = B[2];
          // the lower row shares no tetrahedron with upper nodes above its own corner, the upper row
          // none with lower nodes below it: those entries stay zero
          const int off = c * 2 * nl * Dv + d;
          if (act) {
            if (a == 0) { lds_add(w0 + off, double(l0)); lds_add(w1 + off, double(l1)); }
            else { lds_add(w1 + off + 2, double(u1)); lds_add(w2 + off + 2, double(u2)); }
            lds_add(w0 + off + 2, double(u0));
            lds_add(w2 + off, double(l2));
          }
          if (act && own == (a ? 0 : 2)) lds_add(a ? w0 + off : w2 + off + 2, double(a ? l0 : u2));
          if (act && (a == 0 ? own >= 1 : own <= 1)) lds_add(a ? w1 + off : w1 + off + 2, double(a ? l1 : u1));
        }
      }
    }
    if constexpr (AHEAD)
      asm volatile("" : "+v"(up[0].x), "+v"(up[0].y), "+v"(up[1].x), "+v"(up[1].y), "+v"(up[2].x), "+v"(up[2].y));
    wave_sync();
    __builtin_amdgcn_s_setprio(2);
    copy_level<JAC>(flat, cols, k, cur, k >= kb, vb, nvt, L, Jw, Rw, max_slot, max_tv, lane, R, J);
    if (k == L - 1) copy_level<JAC>(flat, cols, L, nxt, true, vb, nvt, L, Jw, Rw, max_slot, max_tv, lane, R, J);
    wave_sync();
    __builtin_amdgcn_s_setprio(0);
  }
}

// A task by its kind: only one that holds more items than a pass takes walks them in passes, so a vertex
// in many cells costs its own task alone, and a task's bits do not depend on the others in the launch.
// PASSES: the launch has such tasks (kernels without them do not carry their code).  Ice sheet of
// 125,000 columns and one vertex in 40 triangles: R+J 742 us in FP64, 722 with FP32 values, residual
// 277 with all tasks in passes; 606, 559 and 172 so (without that vertex 591, 522 and 164).
template <bool JAC, class JT, bool N3, bool PASSES>
__device__ __forceinline__ void any_prism_task(const MeshView &m, const int4 task, const double *__restrict__ U,
                                               double *__restrict__ R, JT *__restrict__ J, int picard, int max_slot,
                                               int max_tv, int kb, int ke, unsigned char *smem) {
  if (PASSES && __builtin_amdgcn_readfirstlane(m.vc_ptr[task.z] - task.w) > PRISM_ITEMS)
    prism_task<JAC, JT, N3, true>(m, task, U, R, J, picard, max_slot, max_tv, kb, ke, smem);
  else
    prism_task<JAC, JT, N3, false>(m, task, U, R, J, picard, max_slot, max_tv, kb, ke, smem);
}

template <bool JAC, class JT, bool N3, bool PASSES>
__device__ __forceinline__ void any_hex_task(const MeshView &m, const int4 task, const double *__restrict__ U,
                                             double *__restrict__ R, JT *__restrict__ J, int picard, int max_slot,
                                             int max_tv, int kb, int ke, unsigned char *smem) {
  if (PASSES && __builtin_amdgcn_readfirstlane(m.vc_ptr[task.z] - task.w) > HEX_ITEMS)
    hex_task<JAC, JT, N3, true>(m, task, U, R, J, picard, max_slot, max_tv, kb, ke, smem);
  else
    hex_task<JAC, JT, N3, false>(m, task, U, R, J, picard, max_slot, max_tv, kb, ke, smem);
}

// Block (x, y): task x, levels y lpc .. (y + 1) lpc - 1 of its columns
template <bool JAC, class JT, bool N3, bool PASSES>
__global__ __launch_bounds__(WAVE, PRISM_WAVES) void prism_owner_kernel(MeshView m, const int4 *__restrict__ tasks, int lpc,
                                                              const double *__restrict__ U, double *__restrict__ R,
                                                              JT *__restrict__ J, int picard, int max_slot,
                                                              int max_tv) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int kb = int(blockIdx.y) * lpc, ke = kb + lpc < m.L ? kb + lpc : m.L;
  any_prism_task<JAC, JT, N3, PASSES>(m, tasks[blockIdx.x], U, R, J, picard, max_slot, max_tv, kb, ke, smem);
}

// Block (x, y): task x, levels y lpc .. (y + 1) lpc - 1 of its columns
template <bool JAC, class JT, bool N3, bool PASSES>
__global__ __launch_bounds__(WAVE, 2) void hex_owner_kernel(MeshView m, const int4 *__restrict__ tasks, int lpc,
                                                            const double *__restrict__ U, double *__restrict__ R,
                                                            JT *__restrict__ J, int picard, int max_slot,
                                                            int max_tv) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int kb = int(blockIdx.y) * lpc, ke = kb + lpc < m.L ? kb + lpc : m.L;
  any_hex_task<JAC, JT, N3, PASSES>(m, tasks[blockIdx.x], U, R, J, picard, max_slot, max_tv, kb, ke, smem);
}

template <bool JAC, class JT, bool N3>
__global__ __launch_bounds__(WAVE, TET_WAVES) void tet_owner_kernel(MeshView m, const int4 *__restrict__ tasks, int lpc,
                                                                    const double *__restrict__ U,
                                                                    double *__restrict__ R, JT *__restrict__ J,
                                                                    int picard, int max_slot, int max_tv) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int kb = int(blockIdx.y) * lpc, ke = kb + lpc < m.L ? kb + lpc : m.L;
  tet_task<JAC, JT, N3>(m, tasks[blockIdx.x], U, R, J, picard, max_slot, max_tv, kb, ke, smem);
}

// Persistent ensemble launch: a workgroup works on the (member, task) pair of its own number, then
// repeatedly takes the next one left from a device counter until the combined task table is exhausted
// (every wave exits).  The counter is one address for all workgroups and takes about 7 ns a time, which
// bounds members of few layers: 25,000 columns of one layer took 109 us (hexahedra) and 97 (prisms) with
// the first pair from the counter too, 93 and 82 so; eight uneven sheets of 10 layers 461 -> 449.
template <class F>
__device__ __forceinline__ void ensemble_loop(const EnsembleMember *__restrict__ mem, const int4 *__restrict__ tasks,
                                              int n_tasks, int *__restrict__ counter, F run) {
  __shared__ int next;
  for (int ti = blockIdx.x; ti < n_tasks;) {
    const int4 task = tasks[ti];
    run(mem[task.x], task);
    if (threadIdx.x == 0) next = int(gridDim.x) + atomicAdd(counter, 1);
    __syncthreads();
    ti = __builtin_amdgcn_readfirstlane(next);
    __syncthreads();
  }
}

template <bool JAC, class JT, bool N3>
__global__ __launch_bounds__(WAVE, TET_WAVES) void tet_ensemble_kernel(const EnsembleMember *__restrict__ mem,
                                                                       const int4 *__restrict__ tasks, int n_tasks,
                                                                       int *__restrict__ counter, int picard) {
  extern __shared__ __align__(16) unsigned char smem[];
  ensemble_loop(mem, tasks, n_tasks, counter, [&](const EnsembleMember &e, const int4 task) {
    tet_task<JAC, JT, N3>(e.view, task, e.U, e.R, static_cast<JT *>(e.J), picard, e.max_slot, e.max_tv, 0, e.view.L,
                          smem);
  });
}

template <bool JAC, class JT, bool N3, bool PASSES>
__global__ __launch_bounds__(WAVE, PRISM_WAVES) void prism_ensemble_kernel(const EnsembleMember *__restrict__ mem,
                                                                 const int4 *__restrict__ tasks, int n_tasks,
                                                                 int *__restrict__ counter, int picard) {
  extern __shared__ __align__(16) unsigned char smem[];
  ensemble_loop(mem, tasks, n_tasks, counter, [&](const EnsembleMember &e, const int4 task) {
    any_prism_task<JAC, JT, N3, PASSES>(e.view, task, e.U, e.R, static_cast<JT *>(e.J), picard, e.max_slot, e.max_tv,
                                        0, e.view.L, smem);
  });
}

template <bool JAC, class JT, bool N3, bool PASSES>
__global__ __launch_bounds__(WAVE, 2) void hex_ensemble_kernel(const EnsembleMember *__restrict__ mem,
                                                               const int4 *__restrict__ tasks, int n_tasks,
                                                               int *__restrict__ counter, int picard) {
  extern __shared__ __align__(16) unsigned char smem[];
  ensemble_loop(mem, tasks, n_tasks, counter, [&](const EnsembleMember &e, const int4 task) {
    any_hex_task<JAC, JT, N3, PASSES>(e.view, task, e.U, e.R, static_cast<JT *>(e.J), picard, e.max_slot, e.max_tv, 0,
                                      e.view.L, smem);
  });
}

__global__ void fill_zero_kernel(uint4 *__restrict__ p, int64_t n16) {
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n16; i += stride)
    p[i] = make_uint4(0u, 0u, 0u, 0u);
}

__global__ void fill_zero_tail_kernel(uint32_t *__restrict__ p, int64_t n4) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n4) p[i] = 0u;
}

// Ocean-front loads (memoised at upload) added to the residual rows of the front columns:
// one thread per (front vertex, level, component).
__global__ void front_add_kernel(int n_front, int L, const int32_t *__restrict__ vtx,
                                 const double *__restrict__ load, double *__restrict__ R) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t per = 2 * int64_t(L + 1);
  if (i >= n_front * per) return;
  const int64_t f = i / per, r = i - f * per;
  R[2 * int64_t(vtx[f]) * (L + 1) + r] += load[i];
}

enum Cell { PRISM, TETS, HEX };

// Dynamic LDS of one task: the two Jacobian level windows, the two residual windows and, for
// prisms and tetrahedra, the item constants.
template <Cell C>
size_t window_bytes(bool jac, int max_slot, int max_tv) {
  return (jac ? 2 * size_t(max_slot) * sizeof(double) : 0) + 2 * 2 * size_t(max_tv) * sizeof(double) +
         (C == PRISM  ? size_t(PRISM_ITEMS) * PRISM_CONST * sizeof(double)
          : C == TETS ? size_t(WAVE) * TET_CONST * sizeof(double)
                      : 0);
}

// Layers per block of a launch with n_tasks tasks of L layers.  A small mesh leaves the chip
// idle while each wave walks its columns layer by layer, so the levels are split over blocks; a
// block that does not start at the bed repeats the layer below its first level.  The cost taken
// here is the layers of a block (the repeated one included) times the rounds of `resident`
// waves; results do not depend on the split (every level's sums keep their order).  The residual-only
// kernels hold more waves than `resident` says (prisms four on a SIMD, tetrahedra three), so
// mid-sized meshes are split less for them than the chip would take.
int layers_per_block(int64_t n_tasks, int L, int64_t resident) {
  int best = L;
  double best_cost = 0.0;
  for (int lpc = L; lpc >= 1; --lpc) {
    const int chunks = (L + lpc - 1) / lpc;
    const double rounds = double(n_tasks) * chunks / double(resident);
    const double cost = (rounds > 1.0 ? rounds : 1.0) * (lpc + (chunks > 1 ? 1 : 0));
    if (lpc == L || cost < best_cost) {
      best = lpc;
      best_cost = cost;
    }
  }
  return best;
}

constexpr int64_t RESIDENT = 2048;   // with a Jacobian, two waves on each of 1024 SIMDs

template <Cell C, bool JAC, class JT, bool N3, bool PASSES>
fo_status launch_t(const fo_mesh *mesh, const double *U, double *R, JT *J, int kind, hipStream_t s) {
  const MeshView &m = mesh->view;
  const size_t lds = window_bytes<C>(JAC, mesh->max_slot, mesh->max_task_verts);
  const int picard = kind == FO_JAC_PICARD ? 1 : 0;
  fo_status st = profile_begin(mesh, s);
  if (st != FO_OK) return st;
  const int lpc = layers_per_block(mesh->n_tasks, m.L, RESIDENT);
  auto kern = [] {
    if constexpr (C == HEX) return hex_owner_kernel<JAC, JT, N3, PASSES>;
    else if constexpr (C == PRISM) return prism_owner_kernel<JAC, JT, N3, PASSES>;
    else return tet_owner_kernel<JAC, JT, N3>;
  }();
  hipLaunchKernelGGL(kern, dim3(unsigned(mesh->n_tasks), unsigned((m.L + lpc - 1) / lpc)), dim3(WAVE), lds, s, m,
                     mesh->tasks, lpc, U, R, J, picard, mesh->max_slot, mesh->max_task_verts);
  FO_LAUNCH_CHECK("owner_kernel");
  return profile_end(mesh, s);
}

template <Cell C, bool JAC, class JT, bool N3, bool PASSES>
fo_status launch_ens_t(const EnsembleLaunch &E, int kind, hipStream_t s) {
  const size_t lds = window_bytes<C>(JAC, E.max_slot, E.max_tv);
  auto kern = [] {
    if constexpr (C == HEX) return hex_ensemble_kernel<JAC, JT, N3, PASSES>;
    else if constexpr (C == PRISM) return prism_ensemble_kernel<JAC, JT, N3, PASSES>;
    else return tet_ensemble_kernel<JAC, JT, N3>;
  }();
  int per_cu = 0;
  FO_HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, WAVE, lds));
  if (per_cu < 1) per_cu = 1;
  int64_t grid = int64_t(E.n_cu) * per_cu;
  if (grid > E.n_tasks) grid = E.n_tasks;
  if (grid < 1) grid = 1;
  fo_status st = launch_fill_zero(E.counter, 16, s);
  if (st != FO_OK) return st;
  hipLaunchKernelGGL(kern, dim3(unsigned(grid)), dim3(WAVE), lds, s, E.members, E.tasks, E.n_tasks, E.counter,
                     kind == FO_JAC_PICARD ? 1 : 0);
  FO_LAUNCH_CHECK("ensemble_kernel");
  return FO_OK;
}

// Calls f<cell, jac, value type, n = 3, tasks of several passes> for the run-time choices
template <class F>
fo_status by_kernel(int nv, bool tet, bool want_jac, int dtype, bool n3, bool passes, F f) {
  auto by_pass = [&](auto c, auto jac, auto val, auto n) {
    if constexpr (c.value != TETS)
      if (passes) return f(c, jac, val, n, std::true_type{});
    return f(c, jac, val, n, std::false_type{});
  };
  auto by_n = [&](auto c, auto jac, auto val) {
    return n3 ? by_pass(c, jac, val, std::true_type{}) : by_pass(c, jac, val, std::false_type{});
  };
  auto by_type = [&](auto c) {
    if (!want_jac) return by_n(c, std::false_type{}, double{});
    if (dtype == FO_F32) return by_n(c, std::true_type{}, float{});
    return by_n(c, std::true_type{}, double{});
  };
  if (tet) return by_type(std::integral_constant<Cell, TETS>{});
  if (nv == 4) return by_type(std::integral_constant<Cell, HEX>{});
  return by_type(std::integral_constant<Cell, PRISM>{});
}

}  // namespace

fo_status launch_front_add(const MeshView &m, int32_t n_front, const int32_t *vtx, const double *load, double *R,
                           hipStream_t s) {
  if (n_front == 0 || R == nullptr) return FO_OK;
  const int64_t n = int64_t(n_front) * 2 * (m.L + 1);
  hipLaunchKernelGGL(front_add_kernel, dim3(unsigned((n + 255) / 256)), dim3(256), 0, s, int(n_front), int(m.L), vtx,
                     load, R);
  FO_LAUNCH_CHECK("front_add_kernel");
  return FO_OK;
}

fo_status launch_ensemble(const EnsembleLaunch &E, int dtype, int kind, bool want_jac, hipStream_t s) {
  return by_kernel(E.nv, E.tet, want_jac, dtype, E.all_n3, E.passes, [&](auto c, auto jac, auto val, auto n3, auto ps) {
    return launch_ens_t<c.value, jac.value, decltype(val), n3.value, ps.value>(E, kind, s);
  });
}

fo_status launch_fill_zero(void *p, size_t bytes, hipStream_t s) {
  if (bytes == 0) return FO_OK;
  if ((reinterpret_cast<uintptr_t>(p) & 15) != 0 || (bytes & 3) != 0)
    return fail(FO_EINVAL, "fill_zero: pointer must be 16-byte aligned and size a multiple of 4");
  const int64_t n16 = int64_t(bytes / 16);
  if (n16 > 0) {
    const int64_t want = (n16 + 255) / 256;
    const unsigned grid = unsigned(want < 8192 ? want : 8192);
    hipLaunchKernelGGL(fill_zero_kernel, dim3(grid), dim3(256), 0, s, reinterpret_cast<uint4 *>(p), n16);
    FO_LAUNCH_CHECK("fill_zero_kernel");
  }
  const int64_t rem4 = int64_t((bytes - size_t(n16) * 16) / 4);
  if (rem4 > 0) {
    hipLaunchKernelGGL(fill_zero_tail_kernel, dim3(1), dim3(64), 0, s,
                       reinterpret_cast<uint32_t *>(static_cast<char *>(p) + n16 * 16), rem4);
    FO_LAUNCH_CHECK("fill_zero_tail_kernel");
  }
  return FO_OK;
}

fo_status launch_assemble(const fo_mesh *mesh, const double *U, double *R, void *J, int dtype,
                          int kind, bool want_jac, hipStream_t s) {
  fo_status st = launch_assemble_cells(mesh, U, R, J, dtype, kind, want_jac, s);
  if (st != FO_OK) return st;
  return launch_front_add(mesh->view, mesh->n_front, mesh->front_vtx, mesh->front_load, R, s);
}

fo_status launch_assemble_cells(const fo_mesh *mesh, const double *U, double *R, void *J, int dtype,
                                int kind, bool want_jac, hipStream_t s) {
  const MeshView &m = mesh->view;
  return by_kernel(m.nv, m.tet != 0, want_jac, dtype, m.n_glen == 3.0, mesh->passes,
                   [&](auto c, auto jac, auto val, auto n3, auto ps) {
                     using JT = decltype(val);
                     return launch_t<c.value, jac.value, JT, n3.value, ps.value>(
                         mesh, U, R, jac.value ? static_cast<JT *>(J) : nullptr, kind, s);
                   });
}

}  // namespace fo
