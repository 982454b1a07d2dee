// Vector operations of the reconstructions: FP64 inner products of FP32
// arrays, and the smoothed total variation with its gradient, weights and
// curvature, each in one pass over its arrays and one small kernel that adds
// the blocks' FP64 sums.
//
// As separate tensor operations (differences, squares, copies to FP64, sums)
// these were 330 launches and 1.3 ms of 10.4 ms in three iterations of a 96^3
// total-variation reconstruction.  Bound by launches at such sizes, by memory
// at large ones: a node's neighbours come from the caches, and recomputing the
// weights of its three previous neighbours costs less than a second pass.
#include <hip/hip_runtime.h>

#include "oat.h"
#include "oat_internal.hpp"
#include "oat_recon.h"

// FP32 operations as written (the sums and the gradient round as separate
// operations would).
#pragma clang fp contract(off)

namespace oat {

namespace {

constexpr int RECON_BLOCKS = 1024, RECON_THREADS = 256;

// Sum over the block in a fixed order, in thread 0.
__device__ __forceinline__ double block_sum(double v)
{
    __shared__ double part[RECON_THREADS / WAVE];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if (threadIdx.x % WAVE == 0) part[threadIdx.x / WAVE] = v;
    __syncthreads();
    double s = 0.0;
    for (int w = 0; w < RECON_THREADS / WAVE; ++w) s += part[w];
    return s;
}

__global__ void __launch_bounds__(RECON_THREADS)
sum_kernel(const double *__restrict__ part, int n, double *__restrict__ out)
{
    double v = 0.0;
    for (int i = threadIdx.x; i < n; i += RECON_THREADS) v += part[i];
    v = block_sum(v);
    if (threadIdx.x == 0) out[0] = v;
}

__global__ void __launch_bounds__(RECON_THREADS)
dot_kernel(const float *__restrict__ x, const float *__restrict__ y, int64_t n,
           double *__restrict__ part)
{
    double v = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * RECON_THREADS + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * RECON_THREADS)
        v = fma((double)x[i], (double)y[i], v);
    v = block_sum(v);
    if (threadIdx.x == 0) part[blockIdx.x] = v;
}

struct Diff {
    float x, y, z;
};

// Forward differences of a at node n = (x, y, z).
__device__ __forceinline__ Diff diff(const float *__restrict__ a, size_t n, int x, int y, int z,
                                     int nx, int ny, int nz)
{
    const float c = a[n];
    return Diff{x + 1 < nx ? a[n + 1] - c : 0.f, y + 1 < ny ? a[n + nx] - c : 0.f,
                z + 1 < nz ? a[n + (size_t)nx * ny] - c : 0.f};
}

__device__ __forceinline__ float norm2(const Diff &d) { return d.x * d.x + d.y * d.y + d.z * d.z; }

__global__ void __launch_bounds__(RECON_THREADS)
tv_kernel(const float *__restrict__ a, int nx, int ny, int nz, float eps2, float *__restrict__ grad,
          float *__restrict__ wout, double *__restrict__ part)
{
    const unsigned n_all = (unsigned)nx * ny * nz;
    const size_t sz = (size_t)nx * ny;
    double sum = 0.0;
    for (unsigned n = blockIdx.x * RECON_THREADS + threadIdx.x; n < n_all;
         n += gridDim.x * RECON_THREADS) {
        const unsigned row = n / nx;
        const int x = n - row * nx, z = row / ny, y = row - z * ny;
        const Diff d = diff(a, n, x, y, z, nx, ny, nz);
        const float s = sqrtf(norm2(d) + eps2), w = 1.f / s;
        // d^T of the weighted differences: from the previous neighbours' along
        // each axis, minus the node's own
        auto weight = [&](const Diff &p) { return 1.f / sqrtf(norm2(p) + eps2); };
        float g = 0.f;
        if (x > 0) {
            const Diff p = diff(a, n - 1, x - 1, y, z, nx, ny, nz);
            g += p.x * weight(p);
        }
        g -= d.x * w;
        if (y > 0) {
            const Diff p = diff(a, n - nx, x, y - 1, z, nx, ny, nz);
            g += p.y * weight(p);
        }
        g -= d.y * w;
        if (z > 0) {
            const Diff p = diff(a, n - sz, x, y, z - 1, nx, ny, nz);
            g += p.z * weight(p);
        }
        g -= d.z * w;
        grad[n] = g;
        wout[n] = w;
        sum += (double)s;
    }
    sum = block_sum(sum);
    if (threadIdx.x == 0) part[blockIdx.x] = sum;
}

__global__ void __launch_bounds__(RECON_THREADS)
tv_curvature_kernel(const float *__restrict__ a, const float *__restrict__ w, int nx, int ny, int nz,
                    double *__restrict__ part)
{
    const unsigned n_all = (unsigned)nx * ny * nz;
    double sum = 0.0;
    for (unsigned n = blockIdx.x * RECON_THREADS + threadIdx.x; n < n_all;
         n += gridDim.x * RECON_THREADS) {
        const unsigned row = n / nx;
        const int x = n - row * nx, z = row / ny, y = row - z * ny;
        sum += (double)w[n] * (double)norm2(diff(a, n, x, y, z, nx, ny, nz));
    }
    sum = block_sum(sum);
    if (threadIdx.x == 0) part[blockIdx.x] = sum;
}

int recon_fail(int code, const char *msg)
{
    set_last_error(msg);
    return code;
}

int blocks_for(int64_t n)
{
    const int64_t b = (n + RECON_THREADS - 1) / RECON_THREADS;
    return b < RECON_BLOCKS ? (int)b : RECON_BLOCKS;
}

// Adds the blocks' sums and reports the launches' status.
int finish(const char *name, void *workspace, int blocks, double *out, hipStream_t s)
{
    if (hipGetLastError() != hipSuccess) return recon_fail(OAT_ERR_DEVICE, name);
    hipLaunchKernelGGL(sum_kernel, dim3(1), dim3(RECON_THREADS), 0, s, (const double *)workspace,
                       blocks, out);
    return hipGetLastError() == hipSuccess ? OAT_OK : recon_fail(OAT_ERR_DEVICE, name);
}

// An element count below 2^31 less the grid, so that 32-bit indices do not wrap.
bool volume_ok(int nx, int ny, int nz)
{
    return nx >= 1 && ny >= 1 && nz >= 1 && (int64_t)nx * ny <= INT32_MAX &&
           (int64_t)nx * ny * nz <= INT32_MAX;
}

}  // namespace
}  // namespace oat

using namespace oat;

extern "C" {

size_t oat_recon_workspace(void) { return sizeof(double) * RECON_BLOCKS; }

int oat_dot(const float *x, const float *y, int64_t n, double *out, void *workspace, void *stream)
{
    if (!x || !y || !out || !workspace || n < 1)
        return recon_fail(OAT_ERR_ARG, "oat_dot: bad argument");
    const int blocks = blocks_for(n);
    hipLaunchKernelGGL(dot_kernel, dim3(blocks), dim3(RECON_THREADS), 0, (hipStream_t)stream, x, y, n,
                       (double *)workspace);
    return finish("oat_dot: launch failed", workspace, blocks, out, (hipStream_t)stream);
}

int oat_tv(const float *a, int nx, int ny, int nz, float eps2, float *grad, float *w, double *tv,
           void *workspace, void *stream)
{
    if (!a || !grad || !w || !tv || !workspace || a == grad || a == w || grad == w)
        return recon_fail(OAT_ERR_ARG, "oat_tv: bad argument");
    if (!volume_ok(nx, ny, nz)) return recon_fail(OAT_ERR_ARG, "oat_tv: bad volume sizes");
    const int blocks = blocks_for((int64_t)nx * ny * nz);
    hipLaunchKernelGGL(tv_kernel, dim3(blocks), dim3(RECON_THREADS), 0, (hipStream_t)stream, a, nx, ny,
                       nz, eps2, grad, w, (double *)workspace);
    return finish("oat_tv: launch failed", workspace, blocks, tv, (hipStream_t)stream);
}

int oat_tv_curvature(const float *x, const float *w, int nx, int ny, int nz, double *out,
                     void *workspace, void *stream)
{
    if (!x || !w || !out || !workspace)
        return recon_fail(OAT_ERR_ARG, "oat_tv_curvature: bad argument");
    if (!volume_ok(nx, ny, nz))
        return recon_fail(OAT_ERR_ARG, "oat_tv_curvature: bad volume sizes");
    const int blocks = blocks_for((int64_t)nx * ny * nz);
    hipLaunchKernelGGL(tv_curvature_kernel, dim3(blocks), dim3(RECON_THREADS), 0, (hipStream_t)stream,
                       x, w, nx, ny, nz, (double *)workspace);
    return finish("oat_tv_curvature: launch failed", workspace, blocks, out, (hipStream_t)stream);
}

}  // extern "C"
