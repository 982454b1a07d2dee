/* Vector operations of the reconstructions (recon.py) on the device of
 * `stream`.  FP32 arrays, FP64 sums added in a fixed order (deterministic);
 * `workspace` holds oat_recon_workspace() bytes, 8-byte aligned, and is free
 * again when the call's work on `stream` is done.  Status codes and
 * oat_last_error() as in oat.h. */
#ifndef OAT_RECON_H
#define OAT_RECON_H

#include <stddef.h>
#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

size_t oat_recon_workspace(void);

/* out[0] = sum_i x[i] y[i], products and sum in FP64 (n >= 1). */
int oat_dot(const float *x, const float *y, int64_t n, double *out, void *workspace, void *stream);

/* Smoothed isotropic total variation of a[nz][ny][nx], nx ny nz < 2^31, with
 * forward differences d (zero across the far faces), s = sqrt(|d a|^2 + eps2):
 * tv[0] = sum s, w = 1 / s, grad = d^T (w d a).  grad and w must not overlap a. */
int oat_tv(const float *a, int nx, int ny, int nz, float eps2, float *grad, float *w, double *tv,
           void *workspace, void *stream);

/* out[0] = sum w |d x|^2, the curvature along x of the quadratic that lies
 * above the total variation where w was taken. */
int oat_tv_curvature(const float *x, const float *w, int nx, int ny, int nz, double *out,
                     void *workspace, void *stream);

#ifdef __cplusplus
}
#endif

#endif /* OAT_RECON_H */
