// Launchers of the linear-algebra kernels used by the Newton driver.
#pragma once

#include "fo_internal.h"

namespace fo {
fo_status spmv(const fo_mesh *mesh, const void *vals, int dtype, const double *x, double *y, hipStream_t s);
fo_status colblock_factor(const fo_mesh *mesh, const void *vals, int dtype, float *fac, hipStream_t s);
// The same factors and, from one pass over the column blocks, the collapse weights of the two-level
// preconditioner: W [V][L+1][2][2] and its FP32 rounding.
fo_status colblock_factor_weights(const fo_mesh *mesh, const void *vals, int dtype, float *fac, double *W, float *W32,
                                  hipStream_t s);
fo_status colblock_apply(const fo_mesh *mesh, const float *fac, const double *r, double *z, hipStream_t s);
// z = P0 y + M^{-1} (r - JP y): the column smoother after the plane correction of the two-level
// preconditioner (W32: FP32 collapse weights [V][L+1][2][2], JP: FP32 J P0 by column, y: [2 V])
fo_status colblock_apply_correction(const fo_mesh *mesh, const float *fac, const float *W32, const float *JP,
                                    const double *y, const double *r, double *z, hipStream_t s);
int multidot_blocks(int64_t n);
// out[0..nv-1] = V_i . w, out[nv] = w . w, out[nv + 1] = 1 / ||w - V h|| from the first two (1 if
// ||w - V h||^2 <= drop ||w||^2 with drop > 0; 0 if it is not positive with drop = 0).  partial:
// multidot_blocks(n) * (nv + 1) doubles, out: nv + 2; n and ld even, FO_EINVAL otherwise.  host: NULL,
// or pinned coherent memory of kDotsFlag + 1 doubles that receives out, then seq (an integer) at
// kDotsFlag.
constexpr int kDotsMax = 504, kDotsFlag = kDotsMax;
fo_status multidot(int64_t n, const double *V, int64_t ld, int nv, const double *w, double *partial,
                   double *out, double drop, double *host, uint64_t seq, hipStream_t s);
// ||w - V h|| from what multidot wrote for nv vectors: 0 where its square is not positive, infinite where
// the square overflowed (the device's scale is 0 there too)
double projected_norm(const double *out, int nv);
int dot2_blocks(int64_t n);
// out[0] = a . w, out[1] = w . w (partial: 2 dot2_blocks(n) doubles; n even, FO_EINVAL otherwise)
fo_status dot2(int64_t n, const double *a, const double *w, double *partial, double *out, hipStream_t s);
// out = scale[0] (w + sign * sum_i h_i V_i), scale NULL for 1, w NULL for 0, out may be w (n and ld
// even, FO_EINVAL otherwise)
fo_status multiaxpy(int64_t n, const double *V, int64_t ld, int nv, const double *h, const double *scale,
                    const double *w, double *out, double sign, hipStream_t s);
// x += alpha p, r -= alpha q with alpha = num[0] / den[0] read on the device
fo_status cg_step(int64_t n, const double *num, const double *den, const double *p, const double *q, double *x,
                  double *r, hipStream_t s);
fo_status axpby(int64_t n, double a, const double *x, double b, double *y, hipStream_t s);
fo_status xpay(int64_t n, const double *x, double a, const double *y, double *z, hipStream_t s);
}  // namespace fo
