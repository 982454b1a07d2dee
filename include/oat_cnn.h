/*
 * oat_cnn.h -- C ABI of the small 3-D convolution network used as a learned
 * preconditioner for the penalised least-squares reconstruction (training
 * and inference on gfx950).  The network and its use are not part of the
 * paper: they extend the PLS iteration of Sec. IV.A-B, whose gradient they
 * map to a search direction.
 *
 * Volumes are C-contiguous [C][D][H][W] (W fastest), one sample per call;
 * zero padding of one voxel on every face ("same" 3x3x3 convolution).
 * Activations may be stored in FP32 or BF16 (oat_dtype of oat.h); all
 * arithmetic accumulates in FP32.  Weights, biases, gradients and optimiser
 * state are FP32.  Weight layout: [C_out][C_in][3][3][3].
 *
 * Every pointer is a DEVICE pointer owned by the caller; calls are
 * asynchronous on `stream` (hipStream_t, NULL = default stream).  Channel
 * counts must be 1 or 16.  Returns an oat_status (oat.h); sizes and
 * pointers are checked on the host before any launch.
 */
#ifndef OAT_CNN_H
#define OAT_CNN_H

#include <stddef.h>
#include <stdint.h>

#include "oat.h"

#ifdef __cplusplus
extern "C" {
#endif

/* y[co] = b[co] + sum_ci sum_taps w[co][ci][tap] x[ci][v + tap - 1], then
 * y = max(y, 0) if relu != 0, then y = 0 wherever mask (same shape as y,
 * dtype ydt) is <= 0 if mask != NULL.  bias may be NULL (zero).  x and y
 * must not overlap. */
int oat_conv3d_forward(const void *x, oat_dtype xdt, int c_in, int d, int h, int w,
                       const float *weight, const float *bias, int c_out, void *y, oat_dtype ydt,
                       int relu, const void *mask, void *stream);

/* Bytes of device workspace oat_conv3d_backward_weight needs for this shape. */
size_t oat_conv3d_backward_weight_workspace(int c_in, int c_out, int d, int h, int w);

/* dweight[co][ci][tap] = sum_v dy[co][v] x[ci][v + tap - 1] (zero padding),
 * dbias[co] = sum_v dy[co][v]; both overwritten (dbias may be NULL).  The
 * sum is taken per tile of voxels into `workspace` and the tiles are added
 * in a fixed order, so the result is deterministic. */
int oat_conv3d_backward_weight(const void *x, oat_dtype xdt, const void *dy, oat_dtype dydt,
                               int c_in, int c_out, int d, int h, int w, float *dweight,
                               float *dbias, void *workspace, size_t workspace_bytes,
                               void *stream);

/* One Adam step on n parameters (FP32, in place):
 * m = b1 m + (1-b1) g, v = b2 v + (1-b2) g^2,
 * p -= lr (m / (1-b1^t)) / (sqrt(v / (1-b2^t)) + eps), t = step >= 1. */
int oat_adam_step(float *param, const float *grad, float *m, float *v, int64_t n, float lr,
                  float beta1, float beta2, float eps, int step, void *stream);

/* Mean squared error over n values: loss[0] = sum (y - t)^2 / n (FP64
 * accumulation, FP32 result); dy = 2 (y - t) / n in ydt.  `loss` is a device
 * float; `workspace` holds at least oat_mse_workspace() bytes. */
size_t oat_mse_workspace(void);
int oat_mse(const void *y, oat_dtype ydt, const void *target, oat_dtype tdt, int64_t n,
            float *loss, void *dy, void *workspace, void *stream);

/* The whole network z = x + C3(relu(C2(relu(C1(x))))), 3x3x3 kernels, 16
 * channels, on one volume [d][h][w] with BF16 activations, and its parameter
 * gradients.  C1 and C3 (one channel on one side) use the FP32 weights as they
 * are, C2 rounds its weights to BF16; sums are FP32.  Every layer's output is
 * rounded to BF16 once, C3's before x is added.
 *
 * oat_net_forward: x of xdt (rounded to BF16 if FP32), z BF16.  a1 and a2
 * receive the activations after C1 and C2, BF16, channel-last [d][h][w][16].
 * oat_net_backward: gradients of w1 [16][1][27], w2 [16][16][27],
 * w3 [1][16][27] and the biases for dz = dloss/dz (BF16), from the forward's x
 * (as BF16), a1 and a2; every gradient is overwritten; deterministic.
 *
 * a1, a2, workspace and the 16-value biases must be 16-byte aligned.  The
 * workspace holds oat_net_workspace(d, h, w, backward) bytes (0: sizes out of
 * range, d, h, w >= 1).  z must not overlap x. */
size_t oat_net_workspace(int d, int h, int w, int backward);
int oat_net_forward(const void *x, oat_dtype xdt, int d, int h, int w, const float *w1,
                    const float *b1, const float *w2, const float *b2, const float *w3,
                    const float *b3, void *a1, void *a2, void *z, void *workspace,
                    size_t workspace_bytes, void *stream);
int oat_net_backward(const void *x, const void *a1, const void *a2, const void *dz, int d, int h,
                     int w, const float *w2, const float *w3, float *dw1, float *dw2, float *dw3,
                     float *db1, float *db2, float *db3, void *workspace, size_t workspace_bytes,
                     void *stream);

#ifdef __cplusplus
}
#endif

#endif /* OAT_CNN_H */
