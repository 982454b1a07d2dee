// The learned preconditioner z = x + C3(relu(C2(relu(C1(x))))) on gfx950, BF16
// activations: forward pass and parameter gradients as a handful of launches
// (include/oat_cnn.h).  The 16-channel activations are kept channel-last,
// [z][y][x][16]: a voxel is 32 bytes, so halo tiles load and results store in
// whole vectors, and a voxel's channels are the k values of an MFMA operand.
//
// Operand layout of v_mfma_f32_16x16x32_bf16: lane l holds row (A) or column
// (B) l % 16 and 8 k values of group g = l / 16; the result holds column l % 16
// and rows 4 g .. 4 g + 3.  Which k a group's slots stand for is free as long
// as A and B agree.
//
// The one-channel layers and their weights' gradients used to run on the VALU
// with FP32 weights.  Their FP32 weights are split here into three BF16 terms
// w = w1 + w2 + w3 (exact to 2^-27): BF16 products are exact in FP32, so the
// sums are as accurate as FP32 multiply-adds.  The 16 -> 16 layer rounds its
// weights to BF16, as in oat_conv3d_forward.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>
#include <type_traits>

#include "oat.h"
#include "oat_cnn.h"
#include "oat_internal.hpp"

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
typedef unsigned short u16;

__device__ __forceinline__ bf16x8 as_op(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }
__device__ __forceinline__ float bf_f(unsigned bits) { return __uint_as_float(bits << 16); }
__device__ __forceinline__ unsigned f_bf(float v)
{
    return (unsigned)__builtin_bit_cast(u16, (__bf16)v);   // round to nearest even
}
// Two values rounded to BF16 in one word.
__device__ __forceinline__ unsigned f_bf2(float lo, float hi)
{
    typedef __attribute__((ext_vector_type(2))) float f32x2;
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    return __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}
__device__ __forceinline__ f32x4 mfma(u32x4 a, u32x4 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_op(a), as_op(b), c, 0, 0, 0);
}

// The s-th BF16 term of w (s = 0, 1, 2).
__device__ __forceinline__ unsigned split_term(float w, int s)
{
    unsigned b = f_bf(w);
    for (int i = 0; i < s; ++i) {
        const float r = w - bf_f(b);
        w = fabsf(r) <= 0x1.fffffep127f ? r : 0.f;   // no remainder of a first term that is not finite
        b = f_bf(w);
    }
    return b;
}

// Infinities in a product with a split weight's terms, or with the zeros in
// unused slots, give NaN where the product with the weight itself is an
// infinity.  C1 forms the product with the first terms alone, too, in tiles whose
// values or weights are large enough for that, and lets it stand for the results
// that it does not leave finite; C3 and its gradient take a result that is not
// finite again from single products.
constexpr float MAX_F = 3.4028235e38f, LARGE_WEIGHT = 0x1p30f;
constexpr unsigned LARGE_BITS = 0x6c80;   // 2^90 as BF16
__device__ __forceinline__ f32x4 first_if_not_finite(f32x4 first, f32x4 all)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) all[r] = fabsf(first[r]) <= MAX_F ? all[r] : first[r];
    return all;
}

// One-channel input value as FP32, then BF16 bits (FP32 inputs are rounded).
__device__ __forceinline__ unsigned in_bits(const void *x, size_t i, int dt)
{
    return dt == 0 ? f_bf(((const float *)x)[i]) : (unsigned)((const u16 *)x)[i];
}

// ---------------------------------------------------------------------------
// 16 -> 16: weight fragments.  The taps of a row dy come as 5 k-blocks of two
// taps: (dz, dx = 0 | dx = 1) for dz = 0, 1, 2, then dx = 2 of dz = 0 | 1 and of
// dz = 2 twice, with half the weight each (exact; a zero weight would turn an
// infinity into NaN).  k slot 8 (g & 1) + j of tap half g >> 1 is channel
// 8 (g & 1) + j.  frag[dy * 5 + f][lane], row (output channel) lane % 16.
// ---------------------------------------------------------------------------
constexpr int NFRAG = 15;

__device__ __forceinline__ void block_tap(int f, int half, int &dz, int &dx)
{
    if (f < 3) {
        dz = f;
        dx = half;
    } else {
        dz = f == 3 ? half : 2;
        dx = 2;
    }
}

// flip: weights of the data backward, W'[o][i][t] = w[i][o][26 - t].
__device__ void write_fragments(const float *__restrict__ w, int flip, u32x4 *__restrict__ frag)
{
    for (int e = threadIdx.x; e < NFRAG * 64; e += blockDim.x) {
        const int lane = e & 63, dy = (e >> 6) / 5, f = (e >> 6) % 5;
        const int co = lane & 15, g = lane >> 4;
        int dz, dx;
        block_tap(f, g >> 1, dz, dx);
        u32x4 v = {0u, 0u, 0u, 0u};
        const int t = 9 * dz + 3 * dy + dx;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int ci = 8 * (g & 1) + j;
            const float a = flip ? w[(ci * 16 + co) * 27 + 26 - t] : w[(co * 16 + ci) * 27 + t];
            v[j >> 1] |= f_bf(f == 4 ? 0.5f * a : a) << (16 * (j & 1));
        }
        frag[e] = v;
    }
}

// Four channels (4 g ..) of a lane's voxel in a row of voxels: ReLU or mask
// (zero where mask <= 0), one rounding, one 8-byte store past the caches (a
// layer's output is larger than the L2 and read by the next launch: 222 -> 216 us
// for C1 at 256^3, 5% of the pass).  `row` and `mrow` are wave-uniform, `o` the lane's offset.
__device__ __forceinline__ void store4(u16 *__restrict__ row, unsigned o, f32x4 v, bool relu,
                                       const u16 *__restrict__ mrow)
{
    float f[4] = {v[0], v[1], v[2], v[3]};
    if (relu) {
#pragma unroll
        for (int r = 0; r < 4; ++r) f[r] = fmaxf(f[r], 0.f);
    }
    if (mrow) {
        const u32x2 m = *reinterpret_cast<const u32x2 *>(mrow + o);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const unsigned mw = m[r >> 1];
            if (!(__uint_as_float((r & 1) ? mw & 0xffff0000u : mw << 16) > 0.f)) f[r] = 0.f;
        }
    }
    __builtin_nontemporal_store(u32x2{f_bf2(f[0], f[1]), f_bf2(f[2], f[3])},
                                reinterpret_cast<u32x2 *>(row + o));
}

__device__ __forceinline__ int wave_index()
{
    return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
}

// ---------------------------------------------------------------------------
// 1 -> 16 (C1, and the data backward of C3 with flipped weights).  A tile of
// 32 x 8 x C1Z voxels, one or two planes a wave; B: column = voxel, k = tap (27 of 32), gathered from the
// halo tile in LDS; A: the weights' three terms.  Workgroup (0, 0, 0) also
// writes the 16 -> 16 fragments of the layer that follows.
// 158 us at 256^3 (3.4 TB/s of output, 4.7 with its reads; 298 us on the VALU):
// HBM at 90% of a copy's rate, VALU issue three quarters busy with the gather of
// the taps and the stores.
// ---------------------------------------------------------------------------
constexpr int C1X = 32, C1Y = 8, C1_THREADS = 256;
constexpr int C1P = C1X + 4, C1HY = C1Y + 2;   // LDS row pitch, halo rows

template <int C1Z>
__global__ void __launch_bounds__(C1_THREADS)
net_c1_kernel(const void *__restrict__ x, int xdt, int D, int H, int W, const float *__restrict__ w,
              int flip, const float *__restrict__ bias, u16 *__restrict__ y, int relu,
              const u16 *__restrict__ mask, const float *__restrict__ w16, u32x4 *__restrict__ frag)
{
    constexpr int C1HZ = C1Z + 2;
    __shared__ u16 xs[C1HZ * C1HY * C1P];
    __shared__ int wave_large[C1_THREADS / 64];
    static_assert(C1_THREADS / 64 == 4, "wave_large");
    const int x0 = blockIdx.x * C1X, y0 = blockIdx.y * C1Y, z0 = blockIdx.z * C1Z;
    const size_t plane = (size_t)H * W;
    unsigned top = 0;   // the largest |value| of this thread's, as bits, and |weight|
    float top_w = 0.f;
    for (int r = threadIdx.x >> 5; r < C1HZ * C1HY; r += C1_THREADS / 32) {
        const int gy = y0 - 1 + r % C1HY, gz = z0 - 1 + r / C1HY;
        const bool in = gy >= 0 && gy < H && gz >= 0 && gz < D;
        const size_t row = gz * plane + (size_t)gy * W;
#pragma unroll
        for (int xx = threadIdx.x & 31; xx < C1X + 2; xx += 32) {
            const int gx = x0 - 1 + xx;
            const unsigned v = (in && gx >= 0 && gx < W) ? in_bits(x, row + gx, xdt) : 0u;
            xs[r * C1P + xx] = (u16)v;
            top = max(top, v & 0x7fffu);
        }
    }
    const int wave = wave_index(), lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4;
    u32x4 a[3];
    int off[8];
#pragma unroll
    for (int s = 0; s < 3; ++s) a[s] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int t = 8 * g + j, tt = t < 27 ? t : 26;   // (the slots past 26 have zero weights)
        off[j] = ((tt / 9) * C1HY + (tt / 3) % 3) * C1P + tt % 3 + col;
        if (t < 27) {
            const float f = w[col * 27 + (flip ? 26 - t : t)];
            top_w = fmaxf(top_w, fabsf(f));
#pragma unroll
            for (int s = 0; s < 3; ++s) a[s][j >> 1] |= split_term(f, s) << (16 * (j & 1));
        }
    }
    f32x4 b4 = {0.f, 0.f, 0.f, 0.f};
    if (bias) b4 = *reinterpret_cast<const f32x4 *>(bias + 4 * g);
    if (frag && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0) write_fragments(w16, flip, frag);
    const uint64_t lanes = __ballot(top_w >= LARGE_WEIGHT || top >= LARGE_BITS);
    if (lane == 0) wave_large[wave] = lanes != 0;
    __syncthreads();
    const int large = wave_large[0] | wave_large[1] | wave_large[2] | wave_large[3];
    const unsigned vo = (unsigned)col * 16 + 4 * g;   // the lane's offset in a group's row
    // group k of the plane's 16 groups of 16 voxels along x
    auto group = [&](int lz, int k, auto with_large) {
        const u16 *xz = xs + lz * C1HY * C1P;
        const int ly = k >> 1, lx = (k & 1) * 16;
        u32x4 v;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            v[j] = (unsigned)xz[ly * C1P + lx + off[2 * j]] |
                   ((unsigned)xz[ly * C1P + lx + off[2 * j + 1]] << 16);
        f32x4 acc = mfma(a[2], v, b4);
        acc = mfma(a[1], v, acc);
        acc = mfma(a[0], v, acc);
        if (decltype(with_large)::value) {
            if (g == 3) v = u32x4{v[0], v[1] & 0xffffu, 0u, 0u};   // (slots past tap 26)
            acc = first_if_not_finite(mfma(a[0], v, b4), acc);
        }
        const size_t row = ((z0 + lz) * plane + (size_t)(y0 + ly) * W + x0 + lx) * 16;
        if (y0 + ly < H && x0 + lx + col < W) store4(y + row, vo, acc, relu, mask ? mask + row : nullptr);
    };
    if (__builtin_amdgcn_readfirstlane(large)) {
        for (int i = wave; i < C1Z * 2 * C1Y; i += C1_THREADS / 64)
            if (z0 + i / (2 * C1Y) < D) group(i / (2 * C1Y), i % (2 * C1Y), std::true_type());
        return;
    }
    for (int lz = wave; lz < C1Z && z0 + lz < D; lz += C1_THREADS / 64) {
#pragma unroll
        for (int k = 0; k < 2 * C1Y; ++k) group(lz, k, std::false_type());
    }
}

// ---------------------------------------------------------------------------
// 16 -> 16.  A workgroup takes a column of 32 x 8 voxels and marches along z, a
// wave 16 x 4 of each plane: A = weights (rows co), B = voxels.  Four halo
// planes sit in LDS: the three of the current step and the next one, whose
// loads are issued before the step's products and stored after them, so memory
// and matrix cores overlap and a step has one barrier (tiles of 16 x 8 x 8
// loaded, then computed: 505 us at 256^3; marching 374, with wave-uniform rows
// and stores past the caches 285, which is 3.8 TB/s).  An input row's operands are read once
// and serve the three output rows that it touches: 30 LDS operands for 60
// MFMAs.  A plane is two halves of 8 channels, 16 bytes a voxel: 16 lanes read
// 256 consecutive bytes.
// ---------------------------------------------------------------------------
constexpr int C2X = 32, C2Y = 8, C2_THREADS = 256, C2R = 4;   // C2R rows a wave
constexpr int C2HX = C2X + 2, C2HY = C2Y + 2, C2HV = C2HX * C2HY, C2SLOT = 2 * C2HV;
constexpr int C2L = (2 * C2HV + C2_THREADS - 1) / C2_THREADS;   // 16-byte loads a thread and plane

__global__ void __launch_bounds__(C2_THREADS) __attribute__((amdgpu_waves_per_eu(3, 3)))
net_c2_kernel(const u16 *__restrict__ x, int D, int H, int W, const u32x4 *__restrict__ frag,
              const float *__restrict__ bias, u16 *__restrict__ y, int relu,
              const u16 *__restrict__ mask, int zr)
{
    __shared__ u32x4 xs[4 * C2SLOT];
    const int x0 = blockIdx.x * C2X, y0 = blockIdx.y * C2Y, z0 = blockIdx.z * zr, z1 = min(D, z0 + zr);
    const size_t plane = (size_t)H * W;
    const int wave = wave_index(), lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4;
    int src[C2L];   // voxel in the plane, -1 outside the volume
#pragma unroll
    for (int k = 0; k < C2L; ++k) {
        const int i = threadIdx.x + k * C2_THREADS, v = i >> 1;
        const int gx = x0 - 1 + v % C2HX, gy = y0 - 1 + v / C2HX;
        src[k] = (i < C2SLOT && gx >= 0 && gx < W && gy >= 0 && gy < H) ? gy * W + gx : -1;
    }
    u32x4 d[C2L];
    auto load = [&](int z) {
#pragma unroll
        for (int k = 0; k < C2L; ++k) {
            d[k] = u32x4{0u, 0u, 0u, 0u};
            if (src[k] >= 0 && z >= 0 && z < D)
                d[k] = *reinterpret_cast<const u32x4 *>(x + (z * plane + src[k]) * 16 + (threadIdx.x & 1) * 8);
        }
    };
    auto store = [&](int z) {
        u32x4 *dst = xs + (z & 3) * C2SLOT + (threadIdx.x & 1) * C2HV + (threadIdx.x >> 1);
#pragma unroll
        for (int k = 0; k < C2L; ++k)
            if (threadIdx.x + k * C2_THREADS < C2SLOT) dst[k * (C2_THREADS / 2)] = d[k];
    };
    for (int z = z0 - 1; z <= z0 + 1; ++z) {
        load(z);
        store(z);
    }
    u32x4 a[NFRAG];
#pragma unroll
    for (int i = 0; i < NFRAG; ++i) a[i] = frag[i * 64 + lane];
    f32x4 b4 = {0.f, 0.f, 0.f, 0.f};
    if (bias) b4 = *reinterpret_cast<const f32x4 *>(bias + 4 * g);
    __syncthreads();
    const int yw = (wave >> 1) * C2R;   // first output row of the wave
    const int at = (g & 1) * C2HV + yw * C2HX + (wave & 1) * 16 + col;
    const int gx = x0 + (wave & 1) * 16 + col;
    const unsigned vo = (unsigned)col * 16 + 4 * g;
    for (int z = z0; z < z1; ++z) {
        if (z + 1 < z1) load(z + 2);
        // operands of input row 0: blocks 0 .. 2 (plane z - 1 + f, dx = g >> 1),
        // block 3 (plane z - 1 + (g >> 1), dx = 2), block 4 (plane z + 1, dx = 2)
        const u32x4 *p[5];
#pragma unroll
        for (int f = 0; f < 3; ++f) p[f] = xs + ((z - 1 + f) & 3) * C2SLOT + at + (g >> 1);
        p[3] = xs + ((z - 1 + (g >> 1)) & 3) * C2SLOT + at + 2;
        p[4] = xs + ((z + 1) & 3) * C2SLOT + at + 2;
        f32x4 acc[C2R];
#pragma unroll
        for (int r = 0; r < C2R; ++r) acc[r] = b4;
#pragma unroll
        for (int yi = 0; yi < C2R + 2; ++yi)
#pragma unroll
            for (int f = 0; f < 5; ++f) {
                const u32x4 v = p[f][yi * C2HX];
#pragma unroll
                for (int dy = 0; dy < 3; ++dy) {
                    const int r = yi - dy;
                    if (r >= 0 && r < C2R) acc[r] = mfma(a[dy * 5 + f], v, acc[r]);
                }
            }
        if (gx < W)
#pragma unroll
            for (int r = 0; r < C2R; ++r) {
                const size_t row = (z * plane + (size_t)(y0 + yw + r) * W + x0 + (wave & 1) * 16) * 16;
                if (y0 + yw + r < H) store4(y + row, vo, acc[r], relu, mask ? mask + row : nullptr);
            }
        if (z + 1 < z1) store(z + 2);
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// 16 -> 1 with the skip: z = x + r, r = C3(a) rounded to BF16 as a stored
// layer would be.  A column of 32 x 16 voxels marches along z.  Per input
// plane the matrix cores form Y[tap][voxel] = sum_ci w[ci][tap] a[voxel][ci]
// once per halo voxel (k = channel, twice: the slots 16 .. 31 carry the second
// weight term), into LDS; every thread then adds the 27 shifted values to the
// three output planes that the input plane touches.  221 us at 256^3 (a
// 2.7 TB/s read; 1648 us on the VALU from LDS tiles), a third of it LDS and a
// fifth MFMA time; columns of 32 x 8 took 250 us, a second plane of loads in
// flight 234.
// ---------------------------------------------------------------------------
constexpr int C3X = 32, C3Y = 16, C3_THREADS = C3X * C3Y, C3_WAVES = C3_THREADS / 64;
constexpr int C3HX = C3X + 2, C3HY = C3Y + 2, C3HV = C3HX * C3HY;
constexpr int C3G = (C3HV + 15) / 16;            // groups of 16 voxels
constexpr int C3P = C3G * 16 + 4;                // row pitch of Y: 4 rows apart are 16 banks apart
constexpr int C3GW = (C3G + C3_WAVES - 1) / C3_WAVES;

// C3 at one voxel from single FP32 products: the value where the split weights'
// sum is not finite.
__device__ __attribute__((noinline)) float c3_value(const u16 *__restrict__ a, int D, int H, int W,
                                                    const float *__restrict__ w, float bias, int x, int y, int z)
{
    float sum = bias;
    for (int ci = 0; ci < 16 && sum == sum; ++ci)
        for (int t = 0; t < 27; ++t) {
            const int px = x + t % 3 - 1, py = y + t / 3 % 3 - 1, pz = z + t / 9 - 1;
            const bool in = px >= 0 && px < W && py >= 0 && py < H && pz >= 0 && pz < D;
            sum = fmaf(w[ci * 27 + t], in ? bf_f(a[(((size_t)pz * H + py) * W + px) * 16 + ci]) : 0.f, sum);
        }
    return sum;
}

__global__ void __launch_bounds__(C3_THREADS) __attribute__((amdgpu_waves_per_eu(4, 4)))
net_c3_kernel(const u16 *__restrict__ a, const void *__restrict__ x, int xdt, int D, int H, int W,
              const float *__restrict__ w, const float *__restrict__ bias, u16 *__restrict__ z, int zr)
{
    __shared__ float ys[27 * C3P];
    const int x0 = blockIdx.x * C3X, y0 = blockIdx.y * C3Y, z0 = blockIdx.z * zr;
    const int z1 = min(D, z0 + zr);
    const size_t plane = (size_t)H * W;
    const int wave = wave_index(), lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4;
    // weights: [tap tile][terms 1 and 2 | term 3]
    u32x4 wt[2][2];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            wt[m][p] = u32x4{0u, 0u, 0u, 0u};
            const int t = 16 * m + col;
            if (t < 27 && (p == 0 || g < 2))
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    wt[m][p][j >> 1] |= split_term(w[(8 * (g & 1) + j) * 27 + t], p == 0 ? g >> 1 : 2)
                                        << (16 * (j & 1));
        }
    // this wave's halo voxels: groups wave, wave + 8, ...
    int idx[C3GW];        // offset in the plane, -1 outside the volume
#pragma unroll
    for (int k = 0; k < C3GW; ++k) {
        const int v = (wave + k * C3_WAVES) * 16 + col;
        const int gx = x0 - 1 + v % C3HX, gy = y0 - 1 + v / C3HX;
        idx[k] = (v < C3HV && gx >= 0 && gx < W && gy >= 0 && gy < H) ? gy * W + gx : -1;
    }
    const int lx = threadIdx.x % C3X, ly = threadIdx.x / C3X;
    const int gx = x0 + lx, gy = y0 + ly;
    const float b0 = bias ? bias[0] : 0.f;
    const float *yr = ys + ly * C3HX + lx;
    float acc[3] = {b0, b0, b0};   // output planes zi - 1, zi, zi + 1 of input plane zi
    u32x4 v[C3GW];
    auto load = [&](int zi) {
#pragma unroll
        for (int k = 0; k < C3GW; ++k) {
            v[k] = u32x4{0u, 0u, 0u, 0u};
            if (idx[k] >= 0 && zi >= 0 && zi < D)
                v[k] = *reinterpret_cast<const u32x4 *>(a + (zi * plane + idx[k]) * 16 + (g & 1) * 8);
        }
    };
    load(z0 - 1);
    for (int zi = z0 - 1; zi <= z1; ++zi) {
#pragma unroll
        for (int k = 0; k < C3GW; ++k) {
            const int grp = wave + k * C3_WAVES;
            if (grp >= C3G) break;
            f32x4 r0 = {0.f, 0.f, 0.f, 0.f}, r1 = r0;
            r0 = mfma(wt[0][1], v[k], r0);
            r1 = mfma(wt[1][1], v[k], r1);
            r0 = mfma(wt[0][0], v[k], r0);
            r1 = mfma(wt[1][0], v[k], r1);
            float *dst = ys + grp * 16 + col;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                dst[(4 * g + r) * C3P] = r0[r];
                if (16 + 4 * g + r < 27) dst[(16 + 4 * g + r) * C3P] = r1[r];
            }
        }
        if (zi < z1) load(zi + 1);   // in flight while the sums run
        __syncthreads();
#pragma unroll
        for (int dz = 0; dz < 3; ++dz) {
            float s = acc[2 - dz];
#pragma unroll
            for (int t = 0; t < 9; ++t) s += yr[(9 * dz + t) * C3P + (t / 3) * C3HX + t % 3];
            acc[2 - dz] = s;
        }
        __syncthreads();
        const int zo = zi - 1;
        if (zo >= z0 && gx < W && gy < H) {
            const size_t o = zo * plane + (size_t)gy * W + gx;
            float r = acc[0];
            if (!(fabsf(r) <= MAX_F)) r = c3_value(a, D, H, W, w, b0, gx, gy, zo);
            z[o] = (u16)f_bf(bf_f(in_bits(x, o, xdt)) + bf_f(f_bf(r)));
        }
        acc[0] = acc[1];
        acc[1] = acc[2];
        acc[2] = b0;
    }
}

// ---------------------------------------------------------------------------
// Weight gradients: sums over voxels, the k of the MFMAs.  Channel-last tiles
// become operands (row or column = channel, k = voxels) by transposed LDS reads:
// ds_read_b64_tr_b16 gives lane i of a group of 16 channel i of the 4 voxels
// whose 4 x 16 values the group's lanes address.  A step takes the 32 voxels of
// two rows: slots 0 .. 3 of group g are voxels 4 g .. 4 g + 3 of the first row,
// slots 4 .. 7 those of the second.  Workgroups keep their sums in registers
// over all their tiles and write one partial each; the partials are added in
// workgroup order (deterministic).
// ---------------------------------------------------------------------------
constexpr int GX = 16, GY = 8, GZ = 4, G_THREADS = 256;
// workgroups that share the tiles: as many as the LDS lets the device hold
constexpr int G16_GRID = 768, G1_GRID = 1280;
constexpr int GHX = GX + 2, GHY = GY + 2, GHZ = GZ + 2, GHV = GHX * GHY * GHZ, GV = GX * GY * GZ;
constexpr int NJ1 = 16 * 27 + 16, NJ2 = 16 * 16 * 27 + 16, NJ3 = 16 * 27 + 1;   // C1, C2, C3

__device__ __forceinline__ u32x2 tr_read(const u16 *p)
{
    const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) s16x4 *)p);
    return __builtin_bit_cast(u32x2, v);
}

// A 16-channel halo or core tile, 32 bytes a voxel, zero outside the volume:
// into registers, and from there to LDS, so that the next tile's loads are in
// flight during the current one's products.
template <int NX, int NY, int NZ>
struct TileCl {
    static constexpr int N = 2 * NX * NY * NZ, L = (N + G_THREADS - 1) / G_THREADS;
    u32x4 d[L];
    __device__ __forceinline__ void load(const u16 *__restrict__ src, int D, int H, int W, int x0, int y0,
                                         int z0)
    {
#pragma unroll
        for (int k = 0; k < L; ++k) {
            const int i = threadIdx.x + k * G_THREADS, v = i >> 1;
            const int xx = v % NX, r = v / NX, yy = r % NY, zz = r / NY;
            const int gx = x0 + xx, gy = y0 + yy, gz = z0 + zz;
            d[k] = u32x4{0u, 0u, 0u, 0u};
            if (i < N && gx >= 0 && gx < W && gy >= 0 && gy < H && gz >= 0 && gz < D)
                d[k] = *reinterpret_cast<const u32x4 *>(src + (((size_t)gz * H + gy) * W + gx) * 16 +
                                                        (i & 1) * 8);
        }
    }
    __device__ __forceinline__ void store(u32x4 *dst) const
    {
#pragma unroll
        for (int k = 0; k < L; ++k)
            if (threadIdx.x + k * G_THREADS < N) dst[threadIdx.x + k * G_THREADS] = d[k];
    }
};

__device__ __forceinline__ void tile_origin(int tile, int tx, int ty, int &x0, int &y0, int &z0)
{
    x0 = tile % tx * GX;
    y0 = tile / tx % ty * GY;
    z0 = tile / (tx * ty) * GZ;
}

// C2: dW[co][ci][tap] = sum_v dy[v][co] x[v + tap][ci]; wave w takes taps w,
// w + 4, ..., and wave 3 the bias (a tap whose x is 1).
__global__ void __launch_bounds__(G_THREADS)
net_wgrad16_kernel(const u16 *__restrict__ x, const u16 *__restrict__ dy, int D, int H, int W, int tx,
                   int ty, int tiles, float *__restrict__ part)
{
    __shared__ u32x4 xs[2 * GHV], gs[2 * GV];
    const int wave = wave_index(), lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4;
    // address of this lane's 8 bytes of a transposed read at voxel 0
    const u16 *xl = reinterpret_cast<const u16 *>(xs) + (4 * g + (col >> 2)) * 16 + (col & 3) * 4;
    const u16 *gl = reinterpret_cast<const u16 *>(gs) + (4 * g + (col >> 2)) * 16 + (col & 3) * 4;
    f32x4 acc[7];
    int toff[7];
#pragma unroll
    for (int k = 0; k < 7; ++k) {
        const int t = min(wave + 4 * k, 26);
        acc[k] = f32x4{0.f, 0.f, 0.f, 0.f};
        toff[k] = (((t / 9) * GHY + (t / 3) % 3) * GHX + t % 3) * 16;
    }
    TileCl<GHX, GHY, GHZ> xt;
    TileCl<GX, GY, GZ> gt;
    auto load = [&](int tile) {
        int x0, y0, z0;
        tile_origin(tile, tx, ty, x0, y0, z0);
        xt.load(x, D, H, W, x0 - 1, y0 - 1, z0 - 1);
        gt.load(dy, D, H, W, x0, y0, z0);
    };
    load(blockIdx.x);
    for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        __syncthreads();
        xt.store(xs);
        gt.store(gs);
        __syncthreads();
        if (tile + (int)gridDim.x < tiles) load(tile + gridDim.x);
#pragma unroll 2
        for (int s = 0; s < GV / 32; ++s) {   // rows 2 s and 2 s + 1 of the tile
            const int lz = s / (GY / 2), ly = s % (GY / 2) * 2;
            const u32x2 a0 = tr_read(gl + (lz * GY + ly) * GX * 16),
                        a1 = tr_read(gl + (lz * GY + ly + 1) * GX * 16);
            const u32x4 av = {a0[0], a0[1], a1[0], a1[1]};
            const u16 *xr = xl + (lz * GHY + ly) * GHX * 16;
#pragma unroll
            for (int k = 0; k < 7; ++k) {
                const u32x2 b0 = tr_read(xr + toff[k]), b1 = tr_read(xr + toff[k] + GHX * 16);
                u32x4 bv = {b0[0], b0[1], b1[0], b1[1]};
                if (k == 6 && wave == 3) bv = u32x4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
                acc[k] = mfma(av, bv, acc[k]);
            }
        }
    }
    float *dst = part + (size_t)blockIdx.x * NJ2;
#pragma unroll
    for (int k = 0; k < 7; ++k) {
        const int t = wave + 4 * k;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (t < 27)
                dst[((4 * g + r) * 16 + col) * 27 + t] = acc[k][r];
            else if (col == 0)
                dst[16 * 16 * 27 + 4 * g + r] = acc[k][r];
        }
    }
}

// sum_v s[v][ch] t[v + tap] over a workgroup's tiles, both voxels inside the
// volume; ends at the first NaN.
__device__ __attribute__((noinline)) float pair_sum(const u16 *__restrict__ sv, const u16 *__restrict__ tv,
                                                    int D, int H, int W, int tx, int ty, int tiles, int ch,
                                                    int tap)
{
    float sum = 0.f;
    for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        int x0, y0, z0;
        tile_origin(tile, tx, ty, x0, y0, z0);
        for (int v = 0; v < GV && sum == sum; ++v) {
            const int gx = x0 + v % GX, gy = y0 + v / GX % GY, gz = z0 + v / (GX * GY);
            const int px = gx + tap % 3 - 1, py = gy + tap / 3 % 3 - 1, pz = gz + tap / 9 - 1;
            if (gx < W && gy < H && gz < D && px >= 0 && px < W && py >= 0 && py < H && pz >= 0 && pz < D)
                sum = fmaf(bf_f(sv[(((size_t)gz * H + gy) * W + gx) * 16 + ch]),
                           bf_f(tv[((size_t)pz * H + py) * W + px]), sum);
        }
    }
    return sum;
}

// One-channel layers: P[ch][tap] = sum_v s[v][ch] t[v + tap].  C1: s = dy, t = x
// (with the bias, sum_v s[v][ch], as tap 27); C3: s = x, t = dy and tap 26 - tap
// (with the bias, sum_v t[v]).  A: rows = taps, from three copies of t's tile
// shifted by dx, so that runs of 4 voxels are aligned; B: s, transposed.
template <bool C3>
__global__ void __launch_bounds__(G_THREADS)
net_wgrad1_kernel(const u16 *__restrict__ sv, const u16 *__restrict__ tv, int D, int H, int W, int tx,
                  int ty, int tiles, float *__restrict__ part)
{
    __shared__ u32x4 ss[2 * GV];
    __shared__ __attribute__((aligned(16))) u16 ts[3][GHZ * GHY][GX];
    __shared__ float red[4][2][64][4];
    __shared__ float bred[4];
    const int wave = wave_index(), lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4;
    const u16 *sl = reinterpret_cast<const u16 *>(ss) + (4 * g + (col >> 2)) * 16 + (col & 3) * 4;
    f32x4 acc[2];
    const u16 *tp[2];
    bool one[2], none[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        const int t = min(16 * m + col, 26);
        acc[m] = f32x4{0.f, 0.f, 0.f, 0.f};
        tp[m] = &ts[t % 3][(t / 9) * GHY + (t / 3) % 3][4 * g];
        one[m] = 16 * m + col == 27;
        none[m] = 16 * m + col > 27;
    }
    float bsum = 0.f;
    TileCl<GX, GY, GZ> st;
    constexpr int TL = (GHV + G_THREADS - 1) / G_THREADS;
    u16 tl[TL];
    auto load = [&](int tile) {
        int x0, y0, z0;
        tile_origin(tile, tx, ty, x0, y0, z0);
        st.load(sv, D, H, W, x0, y0, z0);
#pragma unroll
        for (int k = 0; k < TL; ++k) {
            const int i = threadIdx.x + k * G_THREADS;
            const int xx = i % GHX, r = i / GHX, yy = r % GHY, zz = r / GHY;
            const int gx = x0 - 1 + xx, gy = y0 - 1 + yy, gz = z0 - 1 + zz;
            tl[k] = 0;
            if (i < GHV && gx >= 0 && gx < W && gy >= 0 && gy < H && gz >= 0 && gz < D)
                tl[k] = tv[((size_t)gz * H + gy) * W + gx];
        }
    };
    load(blockIdx.x);
    for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        __syncthreads();
        st.store(ss);
#pragma unroll
        for (int k = 0; k < TL; ++k) {
            const int i = threadIdx.x + k * G_THREADS;
            if (i >= GHV) break;
            const int xx = i % GHX, r = i / GHX, yy = r % GHY, zz = r / GHY;
#pragma unroll
            for (int dx = 0; dx < 3; ++dx)
                if (xx - dx >= 0 && xx - dx < GX) ts[dx][r][xx - dx] = tl[k];
            if (C3 && xx > 0 && xx <= GX && yy > 0 && yy <= GY && zz > 0 && zz <= GZ) bsum += bf_f(tl[k]);
        }
        __syncthreads();
        if (tile + (int)gridDim.x < tiles) load(tile + gridDim.x);
#pragma unroll
        for (int k = 0; k < GV / 32 / 4; ++k) {
            const int s = wave * (GV / 32 / 4) + k, lz = s / (GY / 2), ly = s % (GY / 2) * 2;
            const u32x2 b0 = tr_read(sl + (lz * GY + ly) * GX * 16),
                        b1 = tr_read(sl + (lz * GY + ly + 1) * GX * 16);
            const u32x4 bv = {b0[0], b0[1], b1[0], b1[1]};
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const u16 *p = tp[m] + (lz * GHY + ly) * GX;
                const u32x2 a0 = *reinterpret_cast<const u32x2 *>(p),
                            a1 = *reinterpret_cast<const u32x2 *>(p + GX);
                u32x4 av = {a0[0], a0[1], a1[0], a1[1]};
                if (one[m]) av = u32x4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
                if (none[m]) av = u32x4{0u, 0u, 0u, 0u};
                acc[m] = mfma(av, bv, acc[m]);
            }
        }
    }
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wave][m][lane][r] = acc[m][r];
    if (C3) {
        for (int o = 32; o > 0; o >>= 1) bsum += __shfl_xor(bsum, o);
        if (lane == 0) bred[wave] = bsum;
    }
    __syncthreads();
    float *dst = part + (size_t)blockIdx.x * (C3 ? NJ3 : NJ1);
    for (int i = threadIdx.x; i < 512; i += G_THREADS) {
        const int r = i & 3, l = (i >> 2) & 63, m = i >> 8;
        const int t = 16 * m + 4 * (l >> 4) + r, ch = l & 15;
        float v = (red[0][m][l][r] + red[1][m][l][r]) + (red[2][m][l][r] + red[3][m][l][r]);
        // an infinite activation times the zeros around t is no part of C3's sum
        if (C3 && t < 27 && !(fabsf(v) <= MAX_F))
            v = pair_sum(sv, tv, D, H, W, tx, ty, tiles, ch, t);
        if (t < 27)
            dst[ch * 27 + (C3 ? 26 - t : t)] = v;
        else if (!C3 && t == 27)
            dst[16 * 27 + ch] = v;
    }
    if (C3 && threadIdx.x == 0) dst[16 * 27] = (bred[0] + bred[1]) + (bred[2] + bred[3]);
}

// Gradients from the workgroups' partials, added in a fixed order: 64 columns and
// 16 runs of workgroups per block, then the runs.
struct NetGrads {
    float *dw1, *dw2, *dw3, *db1, *db2, *db3;
};
constexpr int SUM1 = (NJ1 + 63) / 64, SUM2 = (NJ2 + 63) / 64, SUM3 = (NJ3 + 63) / 64;
__global__ void __launch_bounds__(1024)
net_wgrad_sum_kernel(const float *__restrict__ p1, const float *__restrict__ p2,
                     const float *__restrict__ p3, int n1, int n2, NetGrads o)
{
    __shared__ float red[16][64];
    int b = blockIdx.x;
    const int layer = b < SUM2 ? 2 : (b < SUM2 + SUM1 ? 1 : 3);
    b -= layer == 2 ? 0 : (layer == 1 ? SUM2 : SUM2 + SUM1);
    const int nj = layer == 1 ? NJ1 : (layer == 2 ? NJ2 : NJ3);
    const int nw = layer == 2 ? 16 * 16 * 27 : 16 * 27, n = layer == 2 ? n2 : n1;
    const float *__restrict__ part = layer == 1 ? p1 : (layer == 2 ? p2 : p3);
    const int c = threadIdx.x & 63, run = threadIdx.x >> 6, j = b * 64 + c;
    const int per = (n + 15) / 16, i0 = run * per, i1 = min(n, i0 + per);
    float s = 0.f;
    if (j < nj) {
        int i = i0;
        for (; i + 8 <= i1; i += 8) {   // eight loads in flight, added in order
            float v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = part[(size_t)(i + k) * nj + j];
#pragma unroll
            for (int k = 0; k < 8; ++k) s += v[k];
        }
        for (; i < i1; ++i) s += part[(size_t)i * nj + j];
    }
    red[run][c] = s;
    __syncthreads();
    if (run > 0 || j >= nj) return;
    for (int r = 1; r < 16; ++r) s += red[r][c];
    float *dw = layer == 1 ? o.dw1 : (layer == 2 ? o.dw2 : o.dw3);
    float *db = layer == 1 ? o.db1 : (layer == 2 ? o.db2 : o.db3);
    if (j < nw)
        dw[j] = s;
    else
        db[j - nw] = s;
}

constexpr int C2_WGS = 1536;   // two rounds of the three workgroups a CU holds
constexpr size_t PART_BYTES = sizeof(float) * ((size_t)G16_GRID * NJ2 + (size_t)G1_GRID * (NJ1 + NJ3));
constexpr size_t FRAG_BYTES = (sizeof(u32x4) * NFRAG * 64 + 255) / 256 * 256;

int net_fail(int code, const char *msg)
{
    oat::set_last_error(msg);
    return code;
}

int net_launched(const char *who)
{
    const hipError_t e = hipGetLastError();
    if (e == hipSuccess) return OAT_OK;
    oat::set_last_error((std::string(who) + ": " + hipGetErrorName(e)).c_str());
    return OAT_ERR_DEVICE;
}

unsigned up(int n, int t) { return (unsigned)((n + t - 1) / t); }

// Sizes that the kernels' 32-bit plane offsets and grids hold.
bool net_size_ok(int d, int h, int w)
{
    return d >= 1 && h >= 1 && w >= 1 && (long long)h * w < (1ll << 31) &&
           (long long)up(w, GX) * up(h, GY) * up(d, GZ) < (1ll << 31) && up(h, C1Y) <= 65535 &&
           up(d, 4) <= 65535;
}


// Tiles of 8 planes halve a workgroup's set-up (weight terms, halo) per voxel:
// 186 -> 172 us at 256^3; of 4 where 8 would leave fewer than 8 workgroups a CU.
void launch_c1(const void *x, int xdt, int d, int h, int w, const float *wt, int flip, const float *bias,
               u16 *y, int relu, const u16 *mask, const float *w16, u32x4 *frag, hipStream_t s)
{
    auto go = [&](auto kernel, int planes) {
        hipLaunchKernelGGL(kernel, dim3(up(w, C1X), up(h, C1Y), up(d, planes)), dim3(C1_THREADS), 0, s, x,
                           xdt, d, h, w, wt, flip, bias, y, relu, mask, w16, frag);
    };
    (long long)up(w, C1X) * up(h, C1Y) * up(d, 8) >= 2048 ? go(net_c1_kernel<8>, 8) : go(net_c1_kernel<4>, 4);
}

// Planes per column of a marching kernel: the most that leave `want` workgroups.
int column_planes(long long columns, int d, int want)
{
    int zr = 32;
    while (zr > 4 && columns * up(d, zr) < want) zr /= 2;
    return zr;
}

void launch_c2(const u16 *x, int d, int h, int w, const u32x4 *frag, const float *bias, u16 *y, int relu,
               const u16 *mask, hipStream_t s)
{
    const int zr = column_planes((long long)up(w, C2X) * up(h, C2Y), d, C2_WGS);
    hipLaunchKernelGGL(net_c2_kernel, dim3(up(w, C2X), up(h, C2Y), up(d, zr)), dim3(C2_THREADS), 0, s, x, d,
                       h, w, frag, bias, y, relu, mask, zr);
}

bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }

}  // namespace

extern "C" {

size_t oat_net_workspace(int d, int h, int w, int backward)
{
    if (!net_size_ok(d, h, w)) return 0;
    const size_t n = (size_t)d * h * w;
    return FRAG_BYTES + (backward ? 2 * 32 * n + PART_BYTES : 0);
}

int oat_net_forward(const void *x, oat_dtype xdt, int d, int h, int w, const float *w1, const float *b1,
                    const float *w2, const float *b2, const float *w3, const float *b3, void *a1,
                    void *a2, void *z, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!x || !w1 || !b1 || !w2 || !b2 || !w3 || !b3 || !a1 || !a2 || !z || !workspace)
        return net_fail(OAT_ERR_ARG, "oat_net_forward: null pointer");
    if (!net_size_ok(d, h, w)) return net_fail(OAT_ERR_ARG, "oat_net_forward: bad volume sizes");
    if (xdt != OAT_F32 && xdt != OAT_BF16) return net_fail(OAT_ERR_DTYPE, "oat_net_forward: unknown dtype");
    if (x == z || a1 == a2) return net_fail(OAT_ERR_ARG, "oat_net_forward: buffers alias");
    if (!aligned16(a1) || !aligned16(a2) || !aligned16(workspace) || !aligned16(b1) || !aligned16(b2))
        return net_fail(OAT_ERR_ARG, "oat_net_forward: buffers must be 16-byte aligned");
    if (workspace_bytes < oat_net_workspace(d, h, w, 0))
        return net_fail(OAT_ERR_ARG, "oat_net_forward: workspace too small");
    const hipStream_t s = (hipStream_t)stream;
    u32x4 *frag = (u32x4 *)workspace;
    launch_c1(x, (int)xdt, d, h, w, w1, 0, b1, (u16 *)a1, 1, nullptr, w2, frag, s);
    launch_c2((const u16 *)a1, d, h, w, frag, b2, (u16 *)a2, 1, nullptr, s);
    const int zr = column_planes((long long)up(w, C3X) * up(h, C3Y), d, 512);
    hipLaunchKernelGGL(net_c3_kernel, dim3(up(w, C3X), up(h, C3Y), up(d, zr)), dim3(C3_THREADS), 0, s,
                       (const u16 *)a2, x, (int)xdt, d, h, w, w3, b3, (u16 *)z, zr);
    return net_launched("oat_net_forward");
}

int oat_net_backward(const void *x, const void *a1, const void *a2, const void *dz, int d, int h, int w,
                     const float *w2, const float *w3, float *dw1, float *dw2, float *dw3, float *db1,
                     float *db2, float *db3, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!x || !a1 || !a2 || !dz || !w2 || !w3 || !dw1 || !dw2 || !dw3 || !db1 || !db2 || !db3 || !workspace)
        return net_fail(OAT_ERR_ARG, "oat_net_backward: null pointer");
    if (!net_size_ok(d, h, w)) return net_fail(OAT_ERR_ARG, "oat_net_backward: bad volume sizes");
    if (!aligned16(a1) || !aligned16(a2) || !aligned16(workspace))
        return net_fail(OAT_ERR_ARG, "oat_net_backward: buffers must be 16-byte aligned");
    if (workspace_bytes < oat_net_workspace(d, h, w, 1))
        return net_fail(OAT_ERR_ARG, "oat_net_backward: workspace too small");
    const hipStream_t s = (hipStream_t)stream;
    const size_t n = (size_t)d * h * w;
    u32x4 *frag = (u32x4 *)workspace;
    u16 *d2 = (u16 *)((char *)workspace + FRAG_BYTES), *d1 = d2 + 16 * n;
    float *p2 = (float *)(d1 + 16 * n), *p1 = p2 + (size_t)G16_GRID * NJ2, *p3 = p1 + (size_t)G1_GRID * NJ1;
    const int tx = (int)up(w, GX), ty = (int)up(h, GY), tiles = tx * ty * (int)up(d, GZ);
    const int g16 = std::min(tiles, G16_GRID), g1 = std::min(tiles, G1_GRID);
    // d2 = C3^T dz through relu(a2); its 16 -> 16 fragments are those of C2^T
    launch_c1(dz, (int)OAT_BF16, d, h, w, w3, 1, nullptr, d2, 0, (const u16 *)a2, w2, frag, s);
    hipLaunchKernelGGL(net_wgrad1_kernel<true>, dim3(g1), dim3(G_THREADS), 0, s, (const u16 *)a2,
                       (const u16 *)dz, d, h, w, tx, ty, tiles, p3);
    launch_c2(d2, d, h, w, frag, nullptr, d1, 0, (const u16 *)a1, s);
    hipLaunchKernelGGL(net_wgrad16_kernel, dim3(g16), dim3(G_THREADS), 0, s, (const u16 *)a1,
                       (const u16 *)d2, d, h, w, tx, ty, tiles, p2);
    hipLaunchKernelGGL(net_wgrad1_kernel<false>, dim3(g1), dim3(G_THREADS), 0, s, (const u16 *)d1,
                       (const u16 *)x, d, h, w, tx, ty, tiles, p1);
    const NetGrads o{dw1, dw2, dw3, db1, db2, db3};
    hipLaunchKernelGGL(net_wgrad_sum_kernel, dim3(SUM1 + SUM2 + SUM3), dim3(1024), 0, s,
                       (const float *)p1, (const float *)p2, (const float *)p3, g1, g16, o);
    return net_launched("oat_net_backward");
}

}  // extern "C"
