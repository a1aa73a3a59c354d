// Internal declarations of the two-level column semicoarsening preconditioner.
#pragma once

#include <string>
#include <vector>

#include "fo_internal.h"

namespace fo {

constexpr int kMdscCoarsestMax = 64;      // plane vertices solved by the dense inverse
// Below the first level, a level of at most this many vertices and all below it are one matrix formed
// at setup: its kernels are bound by their launches and load chains (14 us for a level of 215 and the
// coarsest solve, 4.7 us as a matrix, which takes 10 us to form).  Levels shrink about eightfold, and
// the matrix grows with the square: 8 MB at 512, 100 MB (20 us to read) at the level before that.
constexpr int kMdscDenseMax = 512;
constexpr int kMdscMaxLevels = 24;

// Host tables that link one plane level to the next (coarser) one.
struct PlaneTables {
  std::vector<int32_t> cptr, cidx;   // graph of the aggregates
  std::vector<int32_t> mptr, midx;   // members of each aggregate
  std::vector<int32_t> gptr, gidx;   // per coarse block: the fine blocks summed into it
};

int32_t aggregate_graph(const std::vector<int32_t> &ptr, const std::vector<int32_t> &idx, std::vector<int32_t> &agg);
void coarse_tables(const std::vector<int32_t> &ptr, const std::vector<int32_t> &idx, const std::vector<int32_t> &agg,
                   int32_t n_agg, PlaneTables &t);
bool graph_ok(int32_t n, const int32_t *ptr, const int32_t *idx, std::string &why);

// A smoothed level's largest Gershgorin row bound and its Chebyshev coefficients.
struct PlaneCheb {
  double g, inv_theta, c1, c2;
};

// One plane level on the device.  Blocks are 2x2, stored [2 c + d] (row component c, column
// component d); vectors hold 2 values per vertex.
struct PlaneLevel {
  int32_t n = 0, nnzb = 0;
  std::vector<int32_t> ptr_h, idx_h, agg_h;
  const int32_t *ptr = nullptr, *idx = nullptr;   // level 0: the mesh's neighbour lists
  int32_t *own_ptr = nullptr, *own_idx = nullptr;
  int32_t *diag = nullptr;      // [n] index of each vertex's diagonal block
  double *A = nullptr;          // [4 nnzb]
  double *Dinv = nullptr;       // [4 n]
  PlaneCheb *ch = nullptr;      // behind the object's flags
  int32_t *agg = nullptr;       // [n] aggregate of each vertex (smoothed levels)
  int32_t *mptr = nullptr, *midx = nullptr;   // members of the next level's vertices
  int32_t *gptr = nullptr, *gidx = nullptr;   // Galerkin gather lists for the next level
  double *b = nullptr, *x = nullptr;          // [2 n] right-hand side and iterate
  double *x2 = nullptr;         // [2 n] first iterate, on the first level then its second one
  double *d = nullptr;          // [2 n] degree-2 smoothing state (first level only)
  double *MT = nullptr;         // [2 n][2 n] column-major: this level and all below it (coarsest: the inverse)
};

// One plane level as the V-cycle kernels read it.  x1 is null where the level is not smoothed.
struct LevelDev {
  int32_t n;
  const int32_t *ptr, *idx, *agg, *mptr, *midx;
  const double *A, *Dinv;
  const PlaneCheb *ch;
  double *b, *x, *x1, *x2, *d;
};

}  // namespace fo

struct fo_mdsc {
  const fo_mesh *mesh = nullptr;
  int device = 0;
  std::vector<fo::PlaneLevel> lv;   // lv.back() is the coarsest
  int32_t *blk_row = nullptr;       // [nnzb of level 0] row vertex of each block
  int dense = 0;                    // first level solved by its MT
  float *fac = nullptr;             // column factors, the layout of the column preconditioner
  double *W = nullptr;              // [V][L+1][2][2] collapse weights (FP64, for the setup)
  float *W32 = nullptr;             // the same rounded to FP32 (restriction and prolongation)
  float *JP = nullptr;              // J P0 (FP32) by plane block e = (v, r): entry d of row q
                                    // of column v at (2 e + d) 2 (L+1) + q
  size_t jp_count = 0;
  int32_t *flag = nullptr;          // device status of the last setup, then the levels' ch
  int32_t *flag_host = nullptr;     // pinned
  bool ready = false;
};
