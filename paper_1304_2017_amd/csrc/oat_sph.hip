// Spherical-voxel imaging model on gfx950 (Sec. II.B.2): H_sph of
// Eq. (dis_sph) with p0 of Eq. (p0f), and its adjoint, Eq. (sphbwd), for
// point-like transducers (the surface integral over S_q divided by S_q is the
// value at r_q) and an ideal EIR:
//   u[q, l] = p0(f_l) sum_n alpha_n exp(-j 2 pi f_l d_qn / c0) / (2 pi d_qn),
//   f_l = f_min + l df,   d_qn = |r_q - r_n|.
// A transducer sees every voxel through one band-limited function of the
// distance, so the sums over frequencies are formed once per transducer, not
// once per voxel: the distance axis is cut into intervals, and
// exp(-j 2 pi f d / c0) on an interval is a polynomial in the position t
// within it (sph_band).  H_sph bins the voxels' weights a t^m into
// moments per interval and transforms those; H_sph^T tabulates each
// transducer's function as FP32 polynomials and evaluates one per (voxel,
// transducer).  The polynomials' errors, as a share of a term, stay below
// 4e-8 rms over the band (H_sph, degree 5; 1 to 2e-8 of the output, whose
// rounding to FP32 is 2.5e-8; degree 7 where the plain sums have no other error
// than that) and 7e-9 (H_sph^T, degree 7, whose tables are rounded to FP32).
// Measured at 64^3 / 2048 transducers / 256 frequencies against the plain sums:
// H_sph of an iterate 29.0 -> 1.49 ms, of a phantom (4.7% of its voxels set)
// 1.75 -> 0.31 ms, H_sph^T 18.2 -> 0.75 ms.
//
// The plain sums over every (transducer, frequency, voxel) term (sph_fwd_kernel,
// sph_adj_kernel) remain for the smallest problems, for H_sph^T of one frequency
// and for H_sph where a transducer's moments exceed the LDS: distances and phases
// in FP64 (a phase of hundreds of turns must keep ~1e-7 turn), an accurate sincos
// of the phase's fractional turn followed by short recurrences along l (an FP64
// rotation by an FP64 step in the forward kernel, FP32 Horner's rule in the
// adjoint), sums in FP64.
#include <algorithm>
#include <cmath>
#include <mutex>
#include <vector>

#include "oat_dtype.hpp"
#include "oat_geom.hpp"
#include "oat_internal.hpp"

#pragma clang fp contract(off)

namespace oat {

namespace {

// Interval polynomials of a frequency band (sph_band): intervals per mm and
// their length, distance from a transducer's centre within which its nodes
// see every voxel, intervals per transducer and per voxel tile (of half
// diagonal `half`), phase per frequency (rad per MHz), Chebyshev nodes and
// the inverse of their Vandermonde matrix.
struct SphBand {
    double inv, step, reach, half, y_per_f, n_want;
    double t[4], e[4][4];
    int n, w;
};

constexpr int SPH_THREADS = 256;
constexpr int SPH_FB = 32;       // frequencies per thread (forward)
constexpr int SPH_TILE = 256;    // voxels staged per LDS tile (forward)
constexpr int SPH_SHARE = 1024;  // (transducer, voxel) values shared per step (forward)
constexpr int SPH_ANCHOR = 16;   // frequencies per Horner block (adjoint)
constexpr int SPH_VQ = 4096;     // staged u p0* values per adjoint tile (32 KB: 4 groups per CU)
constexpr int SPH_NV = 2;        // consecutive voxels per adjoint thread
constexpr int SPH_P = 8;         // polynomial coefficients per interval (adjoint)
constexpr int SPH_M = 6;         // moments per interval (forward): 6, or
constexpr int SPH_M8 = 8;        // 8 where the plain sums have no error but rounding
// 64-bit words per interval of moments in LDS (odd: spreads banks)
constexpr int sph_mrow(int m) { return m + 1; }
constexpr int SPH_MTHREADS = 1024;
// Terms up to which half the threads take a transducer's: more workgroups at once
// hide the clearing and storing of the moments, which such calls consist of (a 5%
// phantom of 28^3 / 2048, 32 frequencies: 78 -> 72 us; every voxel set: 198 -> 202,
// at 64^3 1573 -> 1653).
constexpr int SPH_FEW = 24576;
// Intervals up to which 17 to 32 frequencies take two shares a wave: their moments
// come in vector loads then, two addresses a wave, which bind in long shares (64 x
// 13 x 47 / 1329 / 27, 915 intervals: 72 us for 65).
constexpr int SPH_SUB_N = 768;
constexpr int SPH_RUN = 1 << 20;         // terms summed in integers at a time
constexpr int SPH_TX = 16, SPH_TZ = 8;   // voxel tile of the table adjoint: 16 x 16 x 8
constexpr int SPH_TVOX = SPH_TX * SPH_TX * SPH_TZ;
constexpr int SPH_STAGE = 40960;         // bytes of staged polynomials: 4 workgroups per CU
constexpr long long SPH_PASS = 1ll << 24;   // voxels listed per forward pass (16 bytes each)
constexpr size_t SPH_MOMENTS = size_t(1) << 30;   // bytes of moments held at a time (forward)

__device__ __forceinline__ double frac_turn(double x) { return x - floor(x); }

// Node n of the [nz][ny][nx] grid in FP64.
__device__ __forceinline__ void node_pos(const Problem &P, long long n, double &x, double &y,
                                         double &z)
{
    const long long ix = n % P.nx, iy = (n / P.nx) % P.ny, iz = n / ((long long)P.nx * P.ny);
    x = P.x0 + (double)ix * P.dxd;
    y = P.y0 + (double)iy * P.dxd;
    z = P.z0 + (double)iz * P.dxd;
}

// Partial sums of one voxel chunk.  Thread: transducer q = blockIdx.x * QB +
// t / LB, frequencies l0 = (t % LB) * SPH_FB ... + SPH_FB - 1.
// part[chunk][q][l] = sum over the chunk's voxels (FP64 complex, no p0).
__global__ void __launch_bounds__(SPH_THREADS)
sph_fwd_kernel(Problem P, const void *__restrict__ img, int img_dt, int n_f, double f_min,
               double df, int LB, long long chunk_len, double2 *__restrict__ part)
{
    static_assert(SPH_TILE == SPH_THREADS && SPH_THREADS % 64 == 0, "one voxel per thread per tile");
    __shared__ double sx[SPH_TILE], sy[SPH_TILE], sz[SPH_TILE];
    __shared__ float sa[SPH_TILE];
    __shared__ int wcnt[SPH_THREADS / 64];
    __shared__ double stau[SPH_SHARE], sw[SPH_SHARE];
    __shared__ double2 sstep[SPH_SHARE];
    const int QB = SPH_THREADS / LB;
    const int t = threadIdx.x;
    const int q = blockIdx.x * QB + t / LB;
    const int l0 = (t % LB) * SPH_FB;
    const bool active = (t / LB) < QB && q < P.nq && l0 < n_f;
    const long long N = (long long)P.nx * P.ny * P.nz;
    const long long n0 = (long long)blockIdx.y * chunk_len, n1 = min(N, n0 + chunk_len);
    const double inv_c0 = 1.0 / P.c0d;
    const double fa = f_min + df * (double)l0;   // first frequency of the thread
    double ar[SPH_FB], ai[SPH_FB];
#pragma unroll
    for (int i = 0; i < SPH_FB; ++i) ar[i] = ai[i] = 0.0;
    for (long long base = n0; base < n1; base += SPH_TILE) {
        // Stage the tile's non-zero voxels (their terms are the only
        // non-zero ones), compacted in voxel order: wave ballots give each
        // voxel its rank, so the sums keep the order of the voxels.
        __syncthreads();
        const long long n = base + t;
        const float a_n = n < n1 ? load_val(img, (size_t)n, img_dt) : 0.f;
        const bool keep = a_n != 0.f;
        const uint64_t bal = __ballot(keep);
        const int wv = t >> 6, ln = t & 63;
        if (ln == 0) wcnt[wv] = __popcll(bal);
        __syncthreads();
        int off = 0, cnt = 0;
#pragma unroll
        for (int w = 0; w < SPH_THREADS / 64; ++w) {
            const int c = wcnt[w];
            off += w < wv ? c : 0;
            cnt += c;
        }
        if (keep) {
            const int pos = off + __popcll(bal & ((1ull << ln) - 1ull));
            double x, y, z;
            node_pos(P, n, x, y, z);
            sx[pos] = x;
            sy[pos] = y;
            sz[pos] = z;
            sa[pos] = a_n;
        }
        // Per (transducer, voxel, face node) values shared by the
        // transducer's LB threads, formed once for SUB (voxel, node) items at
        // a time: tau = d/c0, the weight a w_node/(2 pi d) and the frequency
        // step exp(-j 2 pi df tau); items run voxel-major.
        const int NS = P.sph_ns;
        const int SUB = min(SPH_TILE * NS, SPH_SHARE / QB);
        for (int s0 = 0; s0 < cnt * NS; s0 += SUB) {
            const int m = min(SUB, cnt * NS - s0);
            __syncthreads();
            for (int idx = t; idx < QB * m; idx += SPH_THREADS) {
                // item (voxel jj, face node fs) of transducer qq
                const int ql = idx / m, it = s0 + idx % m;
                const int jj = it / NS, fs = it - jj * NS;
                const int qq = blockIdx.x * QB + ql;
                double tq = 0.0, wq = 0.0, cz = 1.0, szs = 0.0;
                if (qq < P.nq) {
                    const double4 fp = P.sph_pts[(size_t)qq * NS + fs];
                    const double vx = sx[jj] - fp.x, vy = sy[jj] - fp.y, vz = sz[jj] - fp.z;
                    const double dd = sqrt(fma(vz, vz, fma(vy, vy, vx * vx)));
                    tq = dd * inv_c0;
                    wq = (double)sa[jj] * fp.w / (6.283185307179586 * dd);
                    sincos_turns_d(frac_turn(df * tq), cz, szs);
                }
                stau[idx] = tq;
                sw[idx] = wq;
                sstep[idx] = make_double2(cz, -szs);   // exp(-j dtheta)
            }
            __syncthreads();
            if (!active) continue;
            const int row = (t / LB) * m;
            for (int jj = 0; jj < m; ++jj) {
                const double tau = stau[row + jj], w = sw[row + jj];
                const double2 zs = sstep[row + jj];
                float c, sn;
                sincos_turns((float)frac_turn(fa * tau), c, sn);
                // w exp(-j theta) = w (c, -sn), stepped by exp(-j dtheta) in
                // FP64 (as fast as FP32 here, and no conversions per term)
                double er = w * (double)c, ei = -(w * (double)sn);
                const double zr = zs.x, zi = zs.y;
#pragma unroll
                for (int i = 0; i < SPH_FB; ++i) {
                    ar[i] += er;
                    ai[i] += ei;
                    const double nr = fma(er, zr, -(ei * zi)), ni = fma(er, zi, ei * zr);
                    er = nr;
                    ei = ni;
                }
            }
        }
    }
    if (active) {
        double2 *dst = part + ((size_t)blockIdx.y * P.nq + q) * n_f;
        for (int i = 0; i < SPH_FB && l0 + i < n_f; ++i) dst[l0 + i] = make_double2(ar[i], ai[i]);
    }
}

// p0(f) of Eq. (p0f) with beta c0^3 / Cp = Gamma c0, ideal EIR; 0 at f = 0.
__device__ __forceinline__ double2 sph_p0(const Problem &P, double f)
{
    if (f == 0.0) return make_double2(0.0, 0.0);
    const double x = 3.141592653589793 * f * P.dxd / P.c0d;
    const double br = P.dxd / (2.0 * P.c0d) * cos(x) - sin(x) / (6.283185307179586 * f);
    return make_double2(0.0, -P.gammad * P.c0d / f * br);
}

// u[q][l] = p0(f_l) * sum over chunks (in chunk order) of part, as complex FP32.
__global__ void __launch_bounds__(SPH_THREADS)
sph_fwd_reduce_kernel(Problem P, const double2 *__restrict__ part, int nchunk, int n_f,
                      double f_min, double df, float2 *__restrict__ u)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long total = (long long)P.nq * n_f;
    if (i >= total) return;
    const int l = (int)(i % n_f);
    double sr = 0.0, si = 0.0;
    for (int c = 0; c < nchunk; ++c) {
        const double2 v = part[(size_t)c * total + i];
        sr += v.x;
        si += v.y;
    }
    const double2 p0 = sph_p0(P, f_min + df * (double)l);
    u[i] = make_float2((float)(p0.x * sr - p0.y * si), (float)(p0.x * si + p0.y * sr));
}

// SPH_NV consecutive voxels per thread:
//   out[n] = Re sum_q sum_l v[q,l] exp(+j 2 pi f_l d_qn / c0) / (2 pi d_qn),
//   v[q,l] = u[q,l] conj(p0(f_l)), staged per transducer in LDS.
// The frequencies are taken in blocks of SPH_ANCHOR.  Within a block,
// sum_i v[l0+i] z^i with z = exp(+j 2 pi df d/c0) is formed by Horner's rule
// in FP32 (S <- S z + v, four FMAs per term); the block's anchor
// A = exp(+j 2 pi f_l0 d/c0) comes from an FP64 recurrence (the first anchor
// and the block step are FP64 sin/cos of fractional turns), and Re(A S) is
// added in FP64.  One staged read serves the thread's voxels.
template <int IMG_DT>
__global__ void __launch_bounds__(SPH_THREADS)
sph_adj_kernel(Problem P, const float2 *__restrict__ u, int n_f, double f_min, double df,
               void *__restrict__ img, double *__restrict__ slice_sum, int q_per_slice)
{
    extern __shared__ float2 sv[];   // [qt][n_fp]: rows padded with zeros to whole blocks
    constexpr int NV = SPH_NV;
    const long long N = (long long)P.nx * P.ny * P.nz;
    const long long nb = ((long long)blockIdx.x * blockDim.x + threadIdx.x) * NV;
    double x[NV], y[NV], z[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        x[v] = y[v] = z[v] = 0.0;
        if (nb + v < N) node_pos(P, nb + v, x[v], y[v], z[v]);
    }
    const double inv_c0 = 1.0 / P.c0d;
    const double dfa = df * SPH_ANCHOR;
    const int n_fp = (n_f + SPH_ANCHOR - 1) / SPH_ANCHOR * SPH_ANCHOR;
    const int qt = max(1, SPH_VQ / n_fp);   // transducers per LDS tile (32 KB)
    const int NS = P.sph_ns;                // face nodes per transducer
    double acc[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[v] = 0.0;
    // Transducers of this slice (blockIdx.y); with one slice, all of them.
    const int qb = (int)blockIdx.y * q_per_slice, qe = min(P.nq, qb + q_per_slice);
    for (int q0 = qb; q0 < qe; q0 += qt) {
        const int nq = min(qt, qe - q0);
        __syncthreads();
        for (int k = threadIdx.x; k < nq * n_fp; k += blockDim.x) {
            const int jq = k / n_fp, l = k % n_fp;
            float2 val = make_float2(0.f, 0.f);   // zero terms pad the last block
            if (l < n_f) {
                const float2 w = u[(size_t)(q0 + jq) * n_f + l];
                const double2 p = sph_p0(P, f_min + df * (double)l);   // w * conj(p0)
                val = make_float2((float)(w.x * p.x + w.y * p.y), (float)(w.y * p.x - w.x * p.y));
            }
            sv[k] = val;
        }
        __syncthreads();
        if (nb >= N) continue;
        for (int jf = 0; jf < nq * NS; ++jf) {
            // transducer j, face node fs
            const int j = jf / NS, fs = jf - j * NS;
            const double4 fp = P.sph_pts[(size_t)(q0 + j) * NS + fs];
            float zr[NV], zi[NV];
            double ar[NV], ai[NV], gr[NV], gi[NV], rd[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const double vx = x[v] - fp.x, vy = y[v] - fp.y, vz = z[v] - fp.z;
                const double dd = sqrt(fma(vz, vz, fma(vy, vy, vx * vx)));
                const double tau = dd * inv_c0;
                sincos_turns((float)frac_turn(df * tau), zr[v], zi[v]);
                sincos_turns_d(frac_turn(f_min * tau), ar[v], ai[v]);
                sincos_turns_d(frac_turn(dfa * tau), gr[v], gi[v]);
                rd[v] = fp.w / (6.283185307179586 * dd);
            }
            const float2 *vq = sv + j * n_fp;
            double part[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) part[v] = 0.0;
            for (int l0 = 0; l0 < n_fp; l0 += SPH_ANCHOR) {
                float sr[NV], si[NV];
#pragma unroll
                for (int v = 0; v < NV; ++v) sr[v] = si[v] = 0.f;
#pragma unroll
                for (int i = SPH_ANCHOR - 1; i >= 0; --i) {
                    const float2 w = vq[l0 + i];
#pragma unroll
                    for (int v = 0; v < NV; ++v) {
                        const float nr = fmaf(sr[v], zr[v], fmaf(-si[v], zi[v], w.x));
                        const float ni = fmaf(sr[v], zi[v], fmaf(si[v], zr[v], w.y));
                        sr[v] = nr;
                        si[v] = ni;
                    }
                }
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    part[v] = fma(ar[v], (double)sr[v], fma(-ai[v], (double)si[v], part[v]));
                    const double tr = ar[v] * gr[v] - ai[v] * gi[v];
                    ai[v] = ar[v] * gi[v] + ai[v] * gr[v];
                    ar[v] = tr;
                }
            }
#pragma unroll
            for (int v = 0; v < NV; ++v) acc[v] = fma(part[v], rd[v], acc[v]);
        }
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        if (nb + v >= N) continue;
        if (slice_sum)
            slice_sum[(size_t)blockIdx.y * N + nb + v] = acc[v];
        else
            store_val(img, (size_t)(nb + v), IMG_DT, (float)acc[v]);
    }
}

// img[n] = sum over the slices, in slice order, of slice_sum[slice][n].
__global__ void __launch_bounds__(SPH_THREADS)
sph_adj_sum_kernel(const double *__restrict__ slice_sum, int slices, long long N,
                   void *__restrict__ img, int img_dt)
{
    const long long n = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= N) return;
    double acc = 0.0;
    for (int sl = 0; sl < slices; ++sl) acc += slice_sum[(size_t)sl * N + n];
    store_val(img, (size_t)n, img_dt, (float)acc);
}

// ---------------------------------------------------------------------------
// Interval polynomials.  Interval i of the distance axis is centred at
// i / inv mm; a transducer at distance r from the origin uses the intervals
// sph_first(r) .. + n - 1, which cover every distance to a node.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int sph_first(const Problem &P, const SphBand &B, int q)
{
    const double x = P.det[q].r[0], y = P.det[q].r[1], z = P.det[q].r[2];
    return (int)floor((sqrt(fma(z, z, fma(y, y, x * x))) - B.reach) * B.inv) - 1;
}

// Coefficients a_m, m < NP, of exp(+-j y t) on t in [-1/2, 1/2], y = 2 pi f
// step / c0: the polynomials that equal cos(y t) (even m) and sin(y t) (odd
// m) at the NP Chebyshev nodes +-t_k.
template <int NP>
__device__ __forceinline__ void sph_basis(const SphBand &B, double f, double a[NP])
{
    constexpr int H = NP / 2;
    double c[H], sn[H];
#pragma unroll
    for (int k = 0; k < H; ++k) {
        sincos(B.y_per_f * f * B.t[k], &sn[k], &c[k]);
        sn[k] /= B.t[k];
    }
#pragma unroll
    for (int m = 0; m < H; ++m) {
        a[2 * m] = a[2 * m + 1] = 0.0;
#pragma unroll
        for (int k = 0; k < H; ++k) {
            a[2 * m] = fma(B.e[m][k], c[k], a[2 * m]);
            a[2 * m + 1] = fma(B.e[m][k], sn[k], a[2 * m + 1]);
        }
    }
}

// Distance d and its reciprocal from the squared distance: the FP32
// reciprocal square root and one FP64 step, the series of (1 - 2 e)^(-1/2),
// e < 2e-7, to e^2 (FULL: to the last places of FP64) or to e (1e-14, where the
// position in the interval is rounded to FP32 next; FULL there: 784 us for 755 at
// 64^3 / 2048 / 256).
template <bool FULL>
__device__ __forceinline__ void sph_dist(double r2, double &d, double &rd)
{
    const double y = (double)__builtin_amdgcn_rsqf((float)r2);
    const double p = r2 * y, e = fma(-p, 0.5 * y, 0.5), c = FULL ? fma(1.5 * e, e, e) : e;
    d = fma(p, c, p);
    rd = fma(y, c, y);
}

// --- H_sph -----------------------------------------------------------------
// Voxels per block of the list.  A block's entries go thread by thread, each
// thread's voxels a quarter of the block apart: neighbours in the list are then
// not neighbours in the image, whose equal distances would meet in the same moments
// (voxels in order: 31 x 54 x 41 / 76 / 84 with 9 face nodes 326 us, 284; 64^3 / 512 /
// 64 499, 413; eight voxels a thread 237 and 433, but 4 us more for the list of a
// phantom).
constexpr int SPH_LIST = 4 * SPH_THREADS;

// A thread's values of the block's voxels n0 .. n1 - 1; returns the block's
// count of non-zero ones, and in wcnt each wave's.
__device__ __forceinline__ int sph_block_values(const void *__restrict__ img, int img_dt, long long n0,
                                                long long n1, float v[SPH_LIST / SPH_THREADS], int *wcnt)
{
    const int wave = threadIdx.x >> 6;
    int cnt = 0;
#pragma unroll
    for (int i = 0; i < SPH_LIST / SPH_THREADS; ++i) {
        const long long n = n0 + (long long)blockIdx.x * SPH_LIST + i * SPH_THREADS + threadIdx.x;
        v[i] = n < n1 ? load_val(img, (size_t)n, img_dt) : 0.f;
        cnt += __popcll(__ballot(v[i] != 0.f));
    }
    if ((threadIdx.x & 63) == 0) wcnt[wave] = cnt;
    __syncthreads();
    cnt = 0;
    for (int w = 0; w < SPH_THREADS / 64; ++w) cnt += wcnt[w];
    return cnt;
}

// blk[block] = (non-zero voxels, bits of the largest |value|) of the blocks of
// the voxels n0 .. n1 - 1.
__global__ void __launch_bounds__(SPH_THREADS)
sph_count_kernel(const void *__restrict__ img, int img_dt, long long n0, long long n1,
                 int2 *__restrict__ blk)
{
    __shared__ int wcnt[SPH_THREADS / 64];
    __shared__ unsigned wmax[SPH_THREADS / 64];
    float v[SPH_LIST / SPH_THREADS];
    const int cnt = sph_block_values(img, img_dt, n0, n1, v, wcnt);
    unsigned m = 0;
#pragma unroll
    for (int i = 0; i < SPH_LIST / SPH_THREADS; ++i) m = max(m, __float_as_uint(v[i]) & 0x7fffffffu);
    for (int o = 32; o > 0; o >>= 1) m = max(m, (unsigned)__shfl_xor((int)m, o));
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < SPH_THREADS / 64; ++w) m = max(m, wmax[w]);
        blk[blockIdx.x] = make_int2(cnt, (int)m);
    }
}

// The non-zero voxels n0 .. n1 - 1 as (ix, iy, iz, value bits), block by block,
// each block's in a fixed order: parts of the list, and their sums, are the
// same on every call.  hdr: their number, bits of the largest |value|.
__global__ void __launch_bounds__(SPH_THREADS)
sph_list_kernel(Problem P, const void *__restrict__ img, int img_dt, long long n0, long long n1,
                const int2 *__restrict__ blk, int *__restrict__ hdr, int4 *__restrict__ list)
{
    constexpr int NW = SPH_THREADS / 64;
    __shared__ int wcnt[NW], wsum[NW];
    __shared__ unsigned wmax[NW];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    // the blocks before this one (the last block looks at all of them)
    const int upto = blockIdx.x + 1 < gridDim.x ? blockIdx.x : gridDim.x;
    int before = 0;
    unsigned m = 0;
    for (int i = threadIdx.x; i < upto; i += SPH_THREADS) {
        const int2 c = blk[i];
        before += i < (int)blockIdx.x ? c.x : 0;
        m = max(m, (unsigned)c.y);
    }
    for (int o = 32; o > 0; o >>= 1) {
        before += __shfl_xor(before, o);
        m = max(m, (unsigned)__shfl_xor((int)m, o));
    }
    if (lane == 0) {
        wsum[wave] = before;
        wmax[wave] = m;
    }
    float v[SPH_LIST / SPH_THREADS];
    const int cnt = sph_block_values(img, img_dt, n0, n1, v, wcnt);
    int pos = 0;
    for (int w = 0; w < NW; ++w) {
        pos += wsum[w];
        m = max(m, wmax[w]);
    }
    if (blockIdx.x + 1 == gridDim.x && threadIdx.x == 0) {
        hdr[0] = pos + cnt;
        hdr[1] = (int)m;
    }
    for (int w = 0; w < wave; ++w) pos += wcnt[w];
#pragma unroll
    for (int i = 0; i < SPH_LIST / SPH_THREADS; ++i)   // the lanes before this one
        pos += __popcll(__ballot(v[i] != 0.f) & ((1ull << lane) - 1ull));
#pragma unroll
    for (int i = 0; i < SPH_LIST / SPH_THREADS; ++i)
        if (v[i] != 0.f) {
            const long long n = n0 + (long long)blockIdx.x * SPH_LIST + i * SPH_THREADS + threadIdx.x;
            const long long xy = (long long)P.nx * P.ny;
            const int iz = (int)(n / xy), r = (int)(n - iz * xy), iy = r / P.nx;
            list[pos++] = make_int4(r - iy * P.nx, iy, iz, (int)__float_as_uint(v[i]));
        }
}

// The same list and header of at most SPH_ONE voxels from one workgroup: one
// launch for two, which at such sizes are 4 us each of a call of 20 to 100 (up to
// 32768 voxels this way: 10 us longer at 32^3).
constexpr int SPH_ONE = 8192, SPH_ONE_THREADS = 1024;
__global__ void __launch_bounds__(SPH_ONE_THREADS)
sph_list_one_kernel(Problem P, const void *__restrict__ img, int img_dt, int N, int *__restrict__ hdr,
                    int4 *__restrict__ list)
{
    constexpr int PER = 8, NW = SPH_ONE_THREADS / 64;
    __shared__ int wcnt[2][NW];
    __shared__ unsigned wmax[NW];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    int base = 0, buf = 0;
    unsigned m = 0;
    for (int b0 = 0; b0 < N; b0 += PER * SPH_ONE_THREADS, buf ^= 1) {
        float v[PER];
        int cnt = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int n = b0 + i * SPH_ONE_THREADS + threadIdx.x;
            v[i] = n < N ? load_val(img, (size_t)n, img_dt) : 0.f;
        }
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            cnt += __popcll(__ballot(v[i] != 0.f));
            m = max(m, __float_as_uint(v[i]) & 0x7fffffffu);
        }
        if (lane == 0) wcnt[buf][wave] = cnt;
        __syncthreads();
        int pos = base;
        for (int w = 0; w < NW; ++w) {
            const int c = wcnt[buf][w];
            pos += w < wave ? c : 0;
            base += c;
        }
#pragma unroll
        for (int i = 0; i < PER; ++i) pos += __popcll(__ballot(v[i] != 0.f) & ((1ull << lane) - 1ull));
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (v[i] != 0.f) {
                const int n = b0 + i * SPH_ONE_THREADS + threadIdx.x;
                const int row = n / P.nx, iz = row / P.ny;
                list[pos++] = make_int4(n - row * P.nx, row - iz * P.ny, iz, (int)__float_as_uint(v[i]));
            }
    }
    for (int o = 32; o > 0; o >>= 1) m = max(m, (unsigned)__shfl_xor((int)m, o));
    if (lane == 0) wmax[wave] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < NW; ++w) m = max(m, wmax[w]);
        hdr[0] = base;
        hdr[1] = (int)m;
    }
}

// Parts in use of the `parts` that a call provides for the moments of n
// listed terms: enough to fill the device, not more than the terms are worth
// (every part costs sph_synth_kernel another pass over the intervals).
__device__ __forceinline__ int sph_parts(long long n, int parts, int fixed)
{
    return fixed ? parts : (int)max(1ll, min((long long)parts, n >> 14));
}

// Few listed terms: the synthesis then sums over the terms themselves, and the
// moments are not formed.  most: as many as the intervals, a third where there are
// enough blocks to fill the device (a term's own exponentials are three times an
// interval's operations: 56 x 16 x 16 / 976 / 139, 154 us for 102); 0 where the
// voxels come in several passes.
__device__ __forceinline__ bool sph_direct(int total, int ns, int most)
{
    return (long long)total * ns <= most;
}

// Moments of one transducer (q = q0 + blockIdx.x) over a part of the listed
// voxels (blockIdx.y of sph_parts): M[part][q - q0][i][m] = sum over the (voxel, face
// node) terms in interval i of w t^m, w = value x node weight / (2 pi d),
// added to the earlier contents if `add`.  The LDS sums are 64-bit integers,
// so they do not depend on the order of a run's terms: every |w t^m| is below
// 2^k / S with k + log2(terms) <= 62, k <= 50 (adding 1.5 2^52 rounds a term
// to an integer in the low bits).  A run is at most SPH_RUN terms, so k >= 42
// whatever the image: the runs are added in FP64, and the roundings of N terms
// together stay near sqrt(N) 2^-43 of the largest, 3e-9 of the output for 2^30
// terms of which one is large (all of them in one run: 1e-5).  A value that
// is not finite makes the moments NaN.
// Bound by the LDS atomics, NM a term at about 12 cycles per wave (two
// thirds of it bank conflicts of random intervals): 1466 us at 64^3 / 2048.
template <int NM>
__global__ void __launch_bounds__(SPH_MTHREADS)
sph_moment_kernel(Problem P, SphBand B, const int4 *__restrict__ list, const int *__restrict__ hdr,
                  int q0, double *__restrict__ M, int add, int fixed, int most)
{
    constexpr int MROW = sph_mrow(NM);
    extern __shared__ unsigned long long mom[];   // [n][MROW]
    const int q = q0 + (int)blockIdx.x, NS = P.sph_ns;
    const int total = hdr[0];
    const unsigned amax = (unsigned)hdr[1];
    const int parts = sph_parts((long long)total * NS, gridDim.y, fixed);
    if ((int)blockIdx.y >= parts || (most > 0 && sph_direct(total, NS, most))) return;
    const int len = (total + parts - 1) / parts;
    const int i0 = (int)blockIdx.y * len, i1 = min(total, i0 + len);
    const int run = min(max(len, 1), SPH_RUN / NS);
    const int first = sph_first(P, B, q);
    const bool bad = amax >= 0x7f800000u;
    // |w| <= |value| / (2 pi d), d >= the transducer's distance - reach
    const double x = P.det[q].r[0], y = P.det[q].r[1], z = P.det[q].r[2];
    const double dmin = sqrt(fma(z, z, fma(y, y, x * x))) - B.reach;
    int e = 0;
    (void)frexp((double)__uint_as_float(amax) / (6.283185307179586 * dmin), &e);
    const int kb = min(62 - (32 - __clz(run * NS - 1)), 50) - e;
    const double S = ldexp(1.0, kb);
    const double unscale = bad ? __longlong_as_double(0x7ff8000000000000ll) : ldexp(1.0, -kb);
    const double ws = S / 6.283185307179586;
    double *dst = M + ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * B.n * NM;
    for (int r0 = i0; r0 == i0 || r0 < i1; r0 += run) {
        const int r1 = min(i1, r0 + run);
        for (int j = threadIdx.x; j < B.n * MROW; j += (int)blockDim.x) mom[j] = 0ull;
        __syncthreads();
        for (int idx = r0 + threadIdx.x; idx < r1; idx += (int)blockDim.x) {
            const int4 en = list[idx];
            const double vx = fma((double)en.x, P.dxd, P.x0), vy = fma((double)en.y, P.dxd, P.y0),
                         vz = fma((double)en.z, P.dxd, P.z0);
            const double av = (double)__uint_as_float((unsigned)en.w) * ws;
            for (int fs = 0; fs < NS; ++fs) {
                const double4 fp = P.sph_pts[(size_t)q * NS + fs];
                const double dx = vx - fp.x, dy = vy - fp.y, dz = vz - fp.z;
                double d, rd;
                sph_dist<true>(fma(dz, dz, fma(dy, dy, dx * dx)), d, rd);
                const double sp = d * B.inv, k = rint(sp), t = sp - k;
                // (in range by the triangle inequality; the minimum keeps the
                // LDS access inside the rows whatever the values are)
                const unsigned i = min((unsigned)((int)k - first), (unsigned)(B.n - 1));
                unsigned long long *row = mom + i * MROW;
                double v = av * (fp.w * rd);
#pragma unroll
                for (int m = 0; m < NM; ++m) {
                    // the magic constant's low word is zero: one 32-bit subtract
                    const long long bits = __double_as_longlong(v + 0x1.8p52);
                    const unsigned hi = (unsigned)(bits >> 32) - 0x43380000u;
                    atomicAdd(row + m, ((unsigned long long)hi << 32) | (unsigned)bits);
                    v *= t;
                }
            }
        }
        __syncthreads();
        for (int j = threadIdx.x; j < B.n * NM; j += (int)blockDim.x) {
            const int i = j / NM;
            const double v = (double)(long long)mom[i * (MROW - NM) + j] * unscale;
            dst[j] = add || r0 > i0 ? dst[j] + v : v;
        }
        __syncthreads();
    }
}

// u[q][l] = p0(f_l) sum_i exp(-j theta_i) (sum_even m - j sum_odd m) a_m(f_l) M[i][m],
// theta_i = 2 pi f_l (first + i) step / c0; `parts` moment sets are summed.
// A lane takes LF frequencies (64 apart), the wave-uniform moments come
// through the scalar cache (LF frequencies share a load); the sum over a
// wave's intervals is Horner's rule in exp(-j 2 pi f step / c0), FP64, times
// one accurate phase.  The waves split the intervals evenly and are added in
// wave order.  Where sph_direct holds (images with few voxels set), the shares are
// of the terms, each with its own exponential (phantoms of 34 x 15 x 55 / 931 / 77
// and 35 x 22 x 45 / 243 / 263: the calls 101 -> 30 and 60 -> 50 us).  SUB > 1 (at
// most 64 / SUB frequencies): a wave's lanes are SUB such shares, so that none is
// idle (a 5% phantom of 12^3 / 2048, 16 frequencies: the call 47 -> 31 us).  Bound
// by FP64 VALU issue: 10 operations per (interval, frequency); 259 us at 64^3 /
// 2048 / 256.
template <int NM, int LF, int SUB>
__global__ void __launch_bounds__(LF == 1 ? 1024 : 256)
sph_synth_kernel(Problem P, SphBand B, const double *__restrict__ M, const int *__restrict__ hdr,
                 const int4 *__restrict__ list, int q0, int max_parts, int fixed, int most, int n_f,
                 double f_min, double df, float2 *__restrict__ u)
{
    static_assert(SUB == 1 || LF == 1, "shares of a wave have one frequency a lane");
    constexpr int F = 64 / SUB;
    extern __shared__ double2 red[];   // [shares][LF * F]
    const int q = q0 + (int)blockIdx.x, NS = (blockDim.x >> 6) * SUB;
    const int lane = threadIdx.x & (F - 1);
    // (uniform with one share a wave: the moments' loads are scalar)
    const int sh = SUB > 1 ? (int)threadIdx.x / F : __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lb = blockIdx.y * 64 * LF;
    const int parts = sph_parts((long long)hdr[0] * P.sph_ns, max_parts, fixed);
    const double tau = B.step / P.c0d;   // us per interval
    const int share = (B.n + NS - 1) / NS, ia = min(B.n, sh * share), ib = min(B.n, ia + share);
    const int first = sph_first(P, B, q);
    double tr[LF], ti[LF];
#pragma unroll
    for (int v = 0; v < LF; ++v) tr[v] = ti[v] = 0.0;
    if (most > 0 && sph_direct(hdr[0], P.sph_ns, most)) {
        // (d / c0, w) of every term in LDS, a share's terms one after the other
        const int terms = hdr[0] * P.sph_ns;
        double2 *term = red + (size_t)NS * LF * F;
        for (int k = threadIdx.x; k < terms; k += blockDim.x) {
            const int4 en = list[k / P.sph_ns];
            const double4 fp = P.sph_pts[(size_t)q * P.sph_ns + k % P.sph_ns];
            const double dx = fma((double)en.x, P.dxd, P.x0) - fp.x, dy = fma((double)en.y, P.dxd, P.y0) - fp.y,
                         dz = fma((double)en.z, P.dxd, P.z0) - fp.z;
            double d, rd;
            sph_dist<true>(fma(dz, dz, fma(dy, dy, dx * dx)), d, rd);
            term[k] = make_double2(d / P.c0d, (double)__uint_as_float((unsigned)en.w) * fp.w * rd *
                                                  0.15915494309189535);
        }
        __syncthreads();
        for (int k = sh; k < terms; k += NS) {
            const double2 t = term[k];
#pragma unroll
            for (int v = 0; v < LF; ++v) {
                const double f = f_min + df * (double)min(lb + v * 64 + lane, n_f - 1);
                double c, s;
                sincos_turns_d(frac_turn(f * t.x), c, s);
                tr[v] = fma(t.y, c, tr[v]);
                ti[v] = fma(-t.y, s, ti[v]);
            }
        }
#pragma unroll
        for (int v = 0; v < LF; ++v) red[(sh * LF + v) * F + lane] = make_double2(tr[v], ti[v]);
    } else {
        double a[LF][NM], zc[LF], zs[LF];
#pragma unroll
        for (int v = 0; v < LF; ++v) {
            const double f = f_min + df * (double)min(lb + v * 64 + lane, n_f - 1);
            sph_basis<NM>(B, f, a[v]);
            sincos_turns_d(frac_turn(f * tau), zc[v], zs[v]);
        }
        for (int c = 0; c < parts; ++c) {
            const double *__restrict__ row = M + (((size_t)c * gridDim.x + blockIdx.x) * B.n + ib) * NM;
            double sr[LF], si[LF];
#pragma unroll
            for (int v = 0; v < LF; ++v) sr[v] = si[v] = 0.0;
#pragma unroll 2
            for (int i = ib; i > ia; --i) {
                row -= NM;
#pragma unroll
                for (int v = 0; v < LF; ++v) {
                    // S <- (even - j odd) + S (zc - j zs)
                    double r = fma(sr[v], zc[v], fma(si[v], zs[v], a[v][0] * row[0]));
                    double m = fma(si[v], zc[v], fma(-sr[v], zs[v], -(a[v][1] * row[1])));
#pragma unroll
                    for (int k = 2; k < NM; k += 2) {
                        r = fma(a[v][k], row[k], r);
                        m = fma(-a[v][k + 1], row[k + 1], m);
                    }
                    sr[v] = r;
                    si[v] = m;
                }
            }
#pragma unroll
            for (int v = 0; v < LF; ++v) {
                tr[v] += sr[v];
                ti[v] += si[v];
            }
        }
#pragma unroll
        for (int v = 0; v < LF; ++v) {
            // times exp(-j theta) of the share's first interval
            const double f = f_min + df * (double)min(lb + v * 64 + lane, n_f - 1);
            double c, s;
            sincos_turns_d(frac_turn(f * tau * (double)(first + ia)), c, s);
            red[(sh * LF + v) * F + lane] = make_double2(fma(tr[v], c, ti[v] * s), fma(ti[v], c, -(tr[v] * s)));
        }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < F * LF && lb + t < n_f; t += blockDim.x) {
        double2 r = red[t];
        for (int w = 1; w < NS; ++w) {
            r.x += red[w * LF * F + t].x;
            r.y += red[w * LF * F + t].y;
        }
        const double2 p0 = sph_p0(P, f_min + df * (double)(lb + t));
        u[(size_t)q * n_f + lb + t] = make_float2((float)(p0.x * r.x - p0.y * r.y),
                                                  (float)(p0.x * r.y + p0.y * r.x));
    }
}

// --- H_sph^T ---------------------------------------------------------------
// ab[m] = a_m(f) beta with p0(f) = j beta.
__device__ __forceinline__ void sph_adj_basis(const Problem &P, const SphBand &B, double f,
                                              double *__restrict__ ab)
{
    const double beta = sph_p0(P, f).y;
    double a[SPH_P];
    sph_basis<SPH_P>(B, f, a);
#pragma unroll
    for (int m = 0; m < SPH_P; ++m) ab[m] = a[m] * beta;
}

__global__ void __launch_bounds__(64)
sph_adj_basis_kernel(Problem P, SphBand B, int n_f, double f_min, double df,
                     double *__restrict__ ab)
{
    const int l = blockIdx.x * 64 + threadIdx.x;
    if (l < n_f) sph_adj_basis(P, B, f_min + df * (double)l, ab + (size_t)l * SPH_P);
}

// Transducers of a table batch: the offsets b0 .. b1 - 1 of every slice of
// qps transducers; table row (slice, offset).
struct SphBatch {
    int qps, b0, b1;
};

// Interval polynomials of F_q(d) = Re sum_l u[q][l] conj(p0(f_l))
// exp(+j 2 pi f_l d / c0) of the batch's transducers: table[row][i] holds the
// coefficients of t^0 .. t^7 (two float4).
// A lane takes two intervals (they share the loads of the row of u and of the
// basis), a workgroup one transducer; FP64 up to the final rounding.  Small grids,
// bound by latency: OWN forms the basis in the workgroup, a launch less, and SH
// groups of threads share the frequencies, their sums added in order (20^3 voxels,
// 16 transducers, 200 frequencies: 15 us, 45 for the two launches).
constexpr int SPH_TTHREADS = 128;
template <int SH, bool OWN>
__global__ void __launch_bounds__(SPH_TTHREADS *SH)
sph_table_kernel(Problem P, SphBand B, SphBatch bt, const float2 *__restrict__ u,
                 const double *__restrict__ ab, int n_f, double f_min, double df,
                 float4 *__restrict__ table)
{
    extern __shared__ double tl[];   // OWN: basis [n_f][SPH_P]; SH > 1: sums [SH - 1][2 SPH_P][threads]
    const int per = bt.b1 - bt.b0, slice = blockIdx.y / per, off = bt.b0 + blockIdx.y % per;
    const int q = slice * bt.qps + off;
    const int lane = threadIdx.x % SPH_TTHREADS;
    const int sh = SH > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / SPH_TTHREADS) : 0;
    const int i0 = blockIdx.x * 2 * SPH_TTHREADS + lane;
    if (off >= bt.qps || q >= P.nq) return;   // (the whole workgroup)
    if (OWN) {
        for (int l = threadIdx.x; l < n_f; l += SPH_TTHREADS * SH)
            sph_adj_basis(P, B, f_min + df * (double)l, tl + l * SPH_P);
        __syncthreads();
    }
    const int share = (n_f + SH - 1) / SH, la = sh * share, lb = min(n_f, la + share);
    double zc[2], zs[2], c[2], s[2], k[2][SPH_P];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const double tau = B.step / P.c0d * (double)(sph_first(P, B, q) + i0 + h * SPH_TTHREADS);
        sincos_turns_d(frac_turn(df * tau), zc[h], zs[h]);
        sincos_turns_d(frac_turn((f_min + df * (double)la) * tau), c[h], s[h]);
#pragma unroll
        for (int m = 0; m < SPH_P; ++m) k[h][m] = 0.0;
    }
    const float2 *__restrict__ row = u + (size_t)q * n_f;
#pragma unroll 2
    for (int l = la; l < lb; ++l) {
        const double ux = (double)row[l].x, uy = (double)row[l].y;
        double a[SPH_P];
#pragma unroll
        for (int m = 0; m < SPH_P; ++m) a[m] = OWN ? tl[l * SPH_P + m] : ab[(size_t)l * SPH_P + m];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            // u conj(p0) exp(j theta) = beta (A - j D); times cos(y t) +
            // j sin(y t), the real part is beta (A cos + D sin)
            const double A = fma(uy, c[h], ux * s[h]), D = fma(ux, c[h], -(uy * s[h]));
#pragma unroll
            for (int m = 0; m < SPH_P; m += 2) {
                k[h][m] = fma(a[m], A, k[h][m]);
                k[h][m + 1] = fma(a[m + 1], D, k[h][m + 1]);
            }
            const double nc = fma(c[h], zc[h], -(s[h] * zs[h]));
            s[h] = fma(c[h], zs[h], s[h] * zc[h]);
            c[h] = nc;
        }
    }
    if (SH > 1) {
        __syncthreads();   // the basis is read
        double *part = tl + (size_t)(sh - 1) * 2 * SPH_P * SPH_TTHREADS + lane;
        if (sh > 0)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int m = 0; m < SPH_P; ++m) part[(h * SPH_P + m) * SPH_TTHREADS] = k[h][m];
        __syncthreads();
        if (sh > 0) return;
        for (int w = 0; w < SH - 1; ++w)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int m = 0; m < SPH_P; ++m)
                    k[h][m] += tl[((size_t)(w * 2 + h) * SPH_P + m) * SPH_TTHREADS + lane];
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int i = i0 + h * SPH_TTHREADS;
        if (i >= B.n) break;
        float4 *dst = table + ((size_t)blockIdx.y * B.n + i) * 2;
        dst[0] = make_float4((float)k[h][0], (float)k[h][1], (float)k[h][2], (float)k[h][3]);
        dst[1] = make_float4((float)k[h][4], (float)k[h][5], (float)k[h][6], (float)k[h][7]);
    }
}

// Sums over a slice's transducers of the batch (blockIdx.y) for the voxels
// of tile tile0 + blockIdx.x: a thread takes a column of 8 voxels along z.
// The B.w intervals that a tile can touch are staged in LDS, `qt`
// transducers at a time, 48 bytes apart (32 would meet half the banks).
// Per (voxel, node): the distance in FP64, in units of intervals, its
// interval, a polynomial in FP32, the sum in FP64.  With `part` the sums go
// there ([slice][tile][voxel], continuing the earlier batches' if `add`),
// else to the image.
// Bound by VALU issue: about 30 instructions per (voxel, node).
template <bool FACE>
__global__ void __launch_bounds__(SPH_THREADS)
sph_eval_kernel(Problem P, SphBand B, SphBatch bt, const float4 *__restrict__ table, int qt,
                long long tile0, void *__restrict__ img, int img_dt, double *__restrict__ part,
                int add)
{
    extern __shared__ float4 st[];   // [qt][w][3], then each one's first interval and row offset
    int2 *sfirst = reinterpret_cast<int2 *>(st + (size_t)qt * 3 * B.w);
    const int ntx = (P.nx + SPH_TX - 1) / SPH_TX, nty = (P.ny + SPH_TX - 1) / SPH_TX;
    const long long tile = tile0 + blockIdx.x;
    const int bx = (int)(tile % ntx), by = (int)(tile / ntx % nty), bz = (int)(tile / ((long long)ntx * nty));
    const int tx = threadIdx.x % SPH_TX, ty = threadIdx.x / SPH_TX;
    const int ix = bx * SPH_TX + tx, iy = by * SPH_TX + ty, iz = bz * SPH_TZ;
    const double x = fma((double)ix, P.dxd, P.x0) * B.inv, y = fma((double)iy, P.dxd, P.y0) * B.inv,
                 z = fma((double)iz, P.dxd, P.z0) * B.inv, dz = P.dxd * B.inv;
    // tile centre (its far columns may lie outside the grid: harmless, the
    // staged range covers the whole tile)
    const double cx = fma(bx * SPH_TX + 0.5 * (SPH_TX - 1), P.dxd, P.x0),
                 cy = fma(by * SPH_TX + 0.5 * (SPH_TX - 1), P.dxd, P.y0),
                 cz = fma(iz + 0.5 * (SPH_TZ - 1), P.dxd, P.z0);
    const int NS = FACE ? P.sph_ns : 1;
    double acc[SPH_TZ];
    double *pp = part ? part + (((size_t)blockIdx.y * gridDim.x + blockIdx.x) * SPH_TVOX) + threadIdx.x
                      : nullptr;
#pragma unroll
    for (int v = 0; v < SPH_TZ; ++v) acc[v] = add ? pp[v * SPH_THREADS] : 0.0;
    const int per = bt.b1 - bt.b0;
    const int qs = (int)blockIdx.y * bt.qps;
    const int cnt = min(min(bt.b1, bt.qps), P.nq - qs) - bt.b0;   // transducers of this batch
    for (int j0 = 0; j0 < cnt; j0 += qt) {
        const int nj = min(qt, cnt - j0);
        __syncthreads();
        for (int j = threadIdx.x; j < nj; j += SPH_THREADS) {
            const int q = qs + bt.b0 + j0 + j, row0 = sph_first(P, B, q);
            const double vx = cx - P.det[q].r[0], vy = cy - P.det[q].r[1], vz = cz - P.det[q].r[2];
            const int lo = (int)floor((sqrt(fma(vz, vz, fma(vy, vy, vx * vx))) - B.half) * B.inv) - 1;
            sfirst[j] = make_int2(max(lo, row0), max(lo - row0, 0));
        }
        __syncthreads();
        for (int j = 0; j < nj; ++j) {
            const int off = __builtin_amdgcn_readfirstlane(sfirst[j].y);
            const float4 *__restrict__ src = table + (((size_t)blockIdx.y * per + j0 + j) * B.n + off) * 2;
            float4 *dst = st + (size_t)j * 3 * B.w;
            const int n2 = 2 * min(B.w, B.n - off);
            for (int k = threadIdx.x; k < n2; k += SPH_THREADS) dst[k + (k >> 1)] = src[k];
        }
        __syncthreads();
        for (int j = 0; j < nj; ++j) {
            const int q = qs + bt.b0 + j0 + j;
            const int first = __builtin_amdgcn_readfirstlane(sfirst[j].x);
            const float4 *__restrict__ row = st + (size_t)j * 3 * B.w;
            for (int fs = 0; fs < NS; ++fs) {
                const double4 fp = P.sph_pts[(size_t)q * NS + fs];
                const double vx = fma(-fp.x, B.inv, x), vy = fma(-fp.y, B.inv, y),
                             vz0 = fma(-fp.z, B.inv, z);
                const double rxy = fma(vy, vy, vx * vx);
#pragma unroll
                for (int v = 0; v < SPH_TZ; ++v) {
                    const double vz = fma((double)v, dz, vz0);
                    double sp, rd;
                    sph_dist<false>(fma(vz, vz, rxy), sp, rd);
                    const double k = rint(sp);
                    const float t = (float)(sp - k);
                    // (in range by the choice of w; the minimum keeps the
                    // access inside the row whatever the values are)
                    const unsigned i = min((unsigned)((int)k - first), (unsigned)(B.w - 1));
                    const float4 *c = row + __umul24(i, 3);
                    const float4 lo = c[0], hi = c[1];
                    float r = fmaf(t, fmaf(t, fmaf(t, hi.w, hi.z), hi.y), hi.x);
                    r = fmaf(t, fmaf(t, fmaf(t, fmaf(t, r, lo.w), lo.z), lo.y), lo.x);
                    if (FACE) rd *= fp.w;
                    acc[v] = fma((double)r, rd, acc[v]);
                }
            }
        }
    }
    if (part) {
#pragma unroll
        for (int v = 0; v < SPH_TZ; ++v) pp[v * SPH_THREADS] = acc[v];
        return;
    }
    if (ix >= P.nx || iy >= P.ny) return;
#pragma unroll
    for (int v = 0; v < SPH_TZ; ++v)
        if (iz + v < P.nz)
            store_val(img, ((size_t)(iz + v) * P.ny + iy) * P.nx + ix, img_dt,
                      (float)(acc[v] * (B.inv * 0.15915494309189535)));
}

// Image values of ntile tiles from tile0 on: the slices' sums in slice order.
__global__ void __launch_bounds__(SPH_THREADS)
sph_eval_sum_kernel(Problem P, SphBand B, const double *__restrict__ part, int slices,
                    long long tile0, void *__restrict__ img, int img_dt)
{
    const int ntx = (P.nx + SPH_TX - 1) / SPH_TX, nty = (P.ny + SPH_TX - 1) / SPH_TX;
    const long long tile = tile0 + blockIdx.x;
    const int ix = (int)(tile % ntx) * SPH_TX + threadIdx.x % SPH_TX,
              iy = (int)(tile / ntx % nty) * SPH_TX + threadIdx.x / SPH_TX,
              iz = (int)(tile / ((long long)ntx * nty)) * SPH_TZ + blockIdx.y;
    if (ix >= P.nx || iy >= P.ny || iz >= P.nz) return;
    double s = 0.0;
    for (int sl = 0; sl < slices; ++sl)
        s += part[((size_t)sl * gridDim.x + blockIdx.x) * SPH_TVOX + blockIdx.y * SPH_THREADS +
                  threadIdx.x];
    store_val(img, ((size_t)iz * P.ny + iy) * P.nx + ix, img_dt,
              (float)(s * (B.inv * 0.15915494309189535)));
}

}  // namespace

hipError_t sph_scratch_address(int device, double **out)
{
    static std::mutex mu;
    static std::vector<double *> addr;   // per device ordinal; null until allocated
    std::lock_guard<std::mutex> lock(mu);
    if (device < 0) return hipErrorInvalidDevice;
    if ((size_t)device >= addr.size()) addr.resize((size_t)device + 1, nullptr);
    if (!addr[(size_t)device]) {
        double *p = nullptr;
        const hipError_t e = hipMalloc((void **)&p, SPH_SCRATCH_BYTES);
        if (e != hipSuccess) return e;
        addr[(size_t)device] = p;
    }
    *out = addr[(size_t)device];
    return hipSuccess;
}

// Interval grid of a band: x = pi f_max step / c0 is the largest half-phase of
// an interval; the error of polynomials with np coefficients is about
// 2 (x/2)^np / np!.
static SphBand sph_band(const Problem &P, int n_f, double f_min, double df, int np, double x)
{
    SphBand B{};
    const double lo[3] = {P.x0, P.y0, P.z0};
    const int n[3] = {P.nx, P.ny, P.nz};
    double r2 = 0.0;
    for (int a = 0; a < 3; ++a) {
        const double m = std::max(std::fabs(lo[a]), std::fabs(lo[a] + (n[a] - 1) * P.dxd));
        r2 += m * m;
    }
    const double f_max = f_min + df * (n_f - 1), rf = P.sph_rf;
    B.reach = std::sqrt(r2) + rf + 1e-9 * (std::sqrt(r2) + rf);
    // at least one interval per reach, so a zero band stays finite
    B.inv = std::max(M_PI * f_max / (x * P.c0d), 1.0 / std::max(B.reach, P.dxd));
    B.step = 1.0 / B.inv;
    B.n_want = 2.0 * B.reach * B.inv + 5.0;
    B.y_per_f = 2.0 * M_PI * B.step / P.c0d;
    B.half = P.dxd * 0.5 * std::sqrt(2.0 * (SPH_TX - 1) * (SPH_TX - 1) + (SPH_TZ - 1) * (SPH_TZ - 1)) *
                 (1.0 + 1e-9) + rf;
    const double w_want = 2.0 * B.half * B.inv + 5.0;
    B.n = (int)std::min(B.n_want, 1e9);
    B.w = (int)std::min(std::min(w_want, B.n_want), 1e9);
    // inverse of the Vandermonde matrix in t_k^2: rows are the Lagrange
    // polynomials' coefficients
    const int h = np / 2;
    double u[4];
    for (int k = 0; k < h; ++k) {
        B.t[k] = 0.5 * std::cos(M_PI * (2 * k + 1) / (2.0 * np));
        u[k] = B.t[k] * B.t[k];
    }
    for (int k = 0; k < h; ++k) {
        double c[4] = {1.0, 0.0, 0.0, 0.0}, den = 1.0;
        for (int j = 0, deg = 0; j < h; ++j) {
            if (j == k) continue;
            ++deg;
            for (int m = deg; m > 0; --m) c[m] = c[m - 1] - u[j] * c[m];
            c[0] *= -u[j];
            den *= u[k] - u[j];
        }
        for (int m = 0; m < h; ++m) B.e[m][k] = c[m] / den;
    }
    return B;
}

// Voxel parts of the moments: enough workgroups for two per CU.
static int sph_moment_parts(const Problem &P)
{
    return std::max(1, std::min(16, 256 / P.nq));
}

// Largest half-phase of the moments' intervals.  Their error grows as (x f /
// f_max)^6: 0.4 for a band that starts near 0, less (down to 0.32) for a
// narrow one, so that its rms over the frequencies is the same.
static double sph_fwd_phase(int n_f, double f_min, double df)
{
    const double f_max = f_min + df * (n_f - 1);
    double m = 0.0;   // mean of (f / f_max)^12
    if (!(f_max > 0.0)) return 0.4;
    if (n_f <= 64) {
        for (int l = 0; l < n_f; ++l) m += std::pow((f_min + df * l) / f_max, 12.0) / n_f;
    } else {
        const double r = f_min / f_max;
        m = r < 0.999 ? (1.0 - std::pow(r, 13.0)) / (13.0 * (1.0 - r)) : 1.0;
    }
    return 0.4 * std::pow(1.0 / (13.0 * m), 1.0 / 12.0);
}

// Moments per interval of H_sph.  Six, at half-phases up to 0.4 (two workgroups'
// LDS per CU at 64^3 and (0, 5] MHz; 0.3: 1.96 ms (one workgroup per CU), 0.33:
// 1.58, 0.4: 1.55, 0.45: 1.55; eight at 0.5: 2.13): their error, 1 to 2e-8 of the
// output, is below that of the plain sums, whose runs of SPH_FB frequencies
// start from FP32 exponentials (together with the outputs' rounding of 2.5e-8, 3
// to 5e-8 against 7 to 11e-8).  A run that starts at or near the frequency 0
// starts exactly, and leaves the plain sums nothing but that rounding: eight
// moments at 0.5 add as little (40 x 37 x 33 voxels, 16 frequencies from 0 to 4.7
// MHz: 2.54e-8 either way, six moments 3.30e-8).  A few frequencies of a second
// run leave them ahead of six moments (19 x 58 x 43, 36 frequencies: 2.81e-8 against
// 3.07e-8; 40: 3.48e-8 against 3.11e-8).
static int sph_moments(const SphBand &B, const Problem &P, int n_f, double f_min)
{
    return n_f <= SPH_FB + 8 && f_min * B.reach < 0.25 * P.c0d ? SPH_M8 : SPH_M;
}

// The moment path is taken when a transducer's moments fit the LDS and its work
// is less, in VALU operations: about 10 per moment of a (voxel, node) term and 2
// per moment, interval and frequency, against 6 per frequency of whole blocks of
// SPH_FB, and 40, of the dense sum.  (The images' zero voxels are skipped on both
// paths.)  A few terms take the plain sums' two launches (1 voxel: 12 us, 17 with
// the moments').
static bool sph_fwd_fast(const Problem &P, int n_f, double f_min, double df, SphBand &B, int &nm)
{
    B = sph_band(P, n_f, f_min, df, SPH_M, sph_fwd_phase(n_f, f_min, df));
    nm = sph_moments(B, P, n_f, f_min);
    if (nm == SPH_M8) B = sph_band(P, n_f, f_min, df, SPH_M8, 0.5);
    const double terms = (double)P.nx * P.ny * P.nz * P.sph_ns;
    if (terms < 32 || B.n_want * sph_mrow(nm) * 8 > 150e3) return false;
    const double parts = std::max(1.0, std::min((double)sph_moment_parts(P), terms / 16384));
    const int blocks = (n_f + SPH_FB - 1) / SPH_FB;
    return terms * 10 * nm + B.n_want * n_f * 2 * nm * parts < terms * (6.0 * SPH_FB * blocks + 40);
}

// Transducer slices of the dense adjoint: a grid of fewer than 1024
// workgroups (a small image) takes the transducers in up to 4 slices along
// grid y, so the device holds more waves; their FP64 partial images are then
// added in slice order.
static int sph_adj_slices(const Problem &P)
{
    const long long N = (long long)P.nx * P.ny * P.nz;
    const long long blocks = ((N + SPH_NV - 1) / SPH_NV + SPH_THREADS - 1) / SPH_THREADS;
    if (blocks >= 1024) return 1;
    long long sl = 1024 / blocks;
    if (sl > 4) sl = 4;
    if (sl > P.nq) sl = P.nq;
    return (int)sl;
}

// H_sph^T: interval half-phases up to 0.65 (error 6e-9 of a term, below the
// FP32 rounding of the tables).  The table path is taken where its work is
// less, in VALU operations: 18 per (interval, frequency) and 40 a (voxel,
// node) term, against 4 per frequency and 100 of the dense sum (12^3 voxels, 64
// transducers, 16 frequencies: 22 against 24 us, and an error of 5e-8 against
// 7e-7).  A single frequency takes the plain sums, which hold nothing but u p0* in
// FP32 (40 x 37 x 33 voxels, 3 MHz: 3.7e-8 of the output, the tables 5.0e-8; from
// two frequencies on Horner's FP32 steps make theirs the larger error).
static bool sph_adj_fast(const Problem &P, int n_f, double f_min, double df, SphBand &B)
{
    B = sph_band(P, n_f, f_min, df, SPH_P, 0.65);
    const double terms = (double)P.nx * P.ny * P.nz * P.sph_ns;
    if (n_f == 1 || B.w > 3072 || B.n_want * 32 > 8e6) return false;
    return B.n_want * n_f * 18 + terms * 40 < terms * (4.0 * n_f + 100);
}

// The list's header (256 bytes) and its blocks' counts.
static size_t sph_list_bytes(long long N)
{
    return 256 + (sizeof(int2) * (size_t)((std::min(N, SPH_PASS) + SPH_LIST - 1) / SPH_LIST) + 255) / 256 * 256;
}

// Transducers whose moments are held at a time, and the moments' bytes.
static int sph_moment_batch(const Problem &P, const SphBand &B, int nm, size_t &bytes)
{
    const size_t row = sizeof(double) * nm * (size_t)sph_moment_parts(P) * B.n;
    const int qb = (int)std::max<size_t>(1, std::min<size_t>(SPH_MOMENTS / row, (size_t)P.nq));
    bytes = row * qb;
    return qb;
}

size_t sph_workspace_bytes(const Problem &P, int n_f, double f_min, double df)
{
    SphBand B;
    int nm;
    if (!sph_fwd_fast(P, n_f, f_min, df, B, nm))
        return sizeof(double2) * (size_t)SPH_CHUNKS * P.nq * n_f;
    const long long N = (long long)P.nx * P.ny * P.nz;
    size_t moments;
    (void)sph_moment_batch(P, B, nm, moments);
    return sph_list_bytes(N) + sizeof(int4) * (size_t)std::min(N, SPH_PASS) + moments;
}

template <int NM>
static hipError_t launch_sph_moments(const Problem &P, const SphBand &B, const void *img, int img_dt,
                                     float2 *u, int n_f, double f_min, double df, char *work,
                                     hipStream_t s)
{
    const long long N = (long long)P.nx * P.ny * P.nz;
    int *hdr = (int *)work;
    int2 *blk = (int2 *)(work + 256);
    int4 *list = (int4 *)(work + sph_list_bytes(N));
    double *M = (double *)(list + std::min(N, SPH_PASS));
    const int parts = sph_moment_parts(P), fixed = N > SPH_PASS ? 1 : 0;
    size_t bytes;
    const int qb = sph_moment_batch(P, B, NM, bytes);
    const int threads_m = N * P.sph_ns <= SPH_FEW ? SPH_MTHREADS / 2 : SPH_MTHREADS;
    for (int q0 = 0; q0 < P.nq; q0 += qb) {
        const int nq = std::min(qb, P.nq - q0);
        const long long blocks = (long long)nq * ((n_f + 63) / 64);
        const int most = fixed ? 0 : (blocks >= 768 ? B.n / 3 : B.n);
        for (long long n0 = 0; n0 < N; n0 += SPH_PASS) {
            const long long n1 = std::min(N, n0 + SPH_PASS);
            // (one pass: its list serves every batch of transducers)
            if (N <= SPH_ONE && q0 == 0) {
                hipLaunchKernelGGL(sph_list_one_kernel, dim3(1), dim3(SPH_ONE_THREADS), 0, s, P, img, img_dt,
                                   (int)N, hdr, list);
            } else if (fixed || q0 == 0) {
                const dim3 blocks((unsigned)((n1 - n0 + SPH_LIST - 1) / SPH_LIST)), threads(SPH_THREADS);
                hipLaunchKernelGGL(sph_count_kernel, blocks, threads, 0, s, img, img_dt, n0, n1, blk);
                hipLaunchKernelGGL(sph_list_kernel, blocks, threads, 0, s, P, img, img_dt, n0, n1, blk, hdr,
                                   list);
            }
            hipLaunchKernelGGL(sph_moment_kernel<NM>, dim3(nq, parts), dim3(threads_m),
                               sizeof(unsigned long long) * sph_mrow(NM) * B.n, s, P, B, list, hdr, q0, M,
                               n0 > 0 ? 1 : 0, fixed, most);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        auto synth = [&](auto kernel, int lf, int nw) {
            hipLaunchKernelGGL(kernel, dim3(nq, (n_f + 64 * lf - 1) / (64 * lf)), dim3(64 * nw),
                               sizeof(double2) * (size_t)(64 * lf * nw + most), s, P, B, M, hdr, list, q0,
                               parts, fixed, most, n_f, f_min, df, u);
        };
        // Frequencies share the loads of the moments where enough waves are
        // left without it; few blocks split the intervals over more waves, each
        // of which pays for the basis of its frequencies (5% phantoms: 24^3 / 209 /
        // 81, 418 blocks: 4 waves 40, 8 34, 16 38 us; 200 blocks 37, 30, 28; 800
        // blocks 38, 41, 54; shares of a wave, 12^3 / 500 / 16: 18, 20, 24).  Where
        // the voxels come in parts there is a set of moments for each (64^3 / 64 /
        // 256, every voxel set, 256 blocks: 8 waves 178, 16 133).
        const bool sets = parts > 1;
        const int nw = blocks >= (sets ? 1024 : 768) ? 4 : (blocks >= (sets ? 512 : 256) ? 8 : 16);
        if (n_f <= 16) synth(sph_synth_kernel<NM, 1, 4>, 1, sets ? 8 : 4);
        else if (n_f <= 32 && B.n <= SPH_SUB_N) synth(sph_synth_kernel<NM, 1, 2>, 1, sets ? 8 : 4);
        else if (blocks >= 2048 && n_f > 128) synth(sph_synth_kernel<SPH_M, 4, 1>, 4, 4);
        else if (blocks >= 2048 && n_f > 64) synth(sph_synth_kernel<SPH_M, 2, 1>, 2, 4);
        else synth(sph_synth_kernel<NM, 1, 1>, 1, nw);
    }
    return hipGetLastError();
}

hipError_t launch_sph_project(const Problem &P, const void *img, int img_dt, float2 *u, int n_f,
                              double f_min, double df, double2 *part, hipStream_t s)
{
    const long long N = (long long)P.nx * P.ny * P.nz;
    SphBand B;
    int nm;
    if (sph_fwd_fast(P, n_f, f_min, df, B, nm))
        return (nm == SPH_M8 ? launch_sph_moments<SPH_M8> : launch_sph_moments<SPH_M>)(
            P, B, img, img_dt, u, n_f, f_min, df, (char *)part, s);
    // n_f <= SPH_THREADS * SPH_FB (checked by the caller): a transducer's
    // frequency blocks fit one workgroup.
    const int LB = (n_f + SPH_FB - 1) / SPH_FB;
    const int QB = SPH_THREADS / LB;
    const long long chunk_len = (N + SPH_CHUNKS - 1) / SPH_CHUNKS;
    const int nchunk = (int)((N + chunk_len - 1) / chunk_len);
    dim3 grid((P.nq + QB - 1) / QB, nchunk);
    hipLaunchKernelGGL(sph_fwd_kernel, grid, dim3(SPH_THREADS), 0, s, P, img, img_dt, n_f, f_min,
                       df, LB, chunk_len, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const long long total = (long long)P.nq * n_f;
    hipLaunchKernelGGL(sph_fwd_reduce_kernel, dim3((unsigned)((total + SPH_THREADS - 1) / SPH_THREADS)),
                       dim3(SPH_THREADS), 0, s, P, part, nchunk, n_f, f_min, df, u);
    return hipGetLastError();
}

// Work split of the table adjoint: tiles of 16 x 16 x 8 voxels, taken
// 1024 at a time; fewer tiles than that take the transducers in `slices`
// slices of at least 8 (4 where that makes no more than 16: 12^3 / 64 / 16
// frequencies, the evaluation 12.7 -> 7.9 us).  The tables of a batch of `per`
// transducers of every slice, and the partial sums, stay within the fixed scratch.
struct SphAdjPlan {
    long long tiles;
    int chunk, slices, qps, per;
    size_t basis_b, table_b, part_b;
};
static SphAdjPlan sph_adj_plan(const Problem &P, const SphBand &B, int n_f)
{
    SphAdjPlan A{};
    A.tiles = (long long)((P.nx + SPH_TX - 1) / SPH_TX) * ((P.ny + SPH_TX - 1) / SPH_TX) *
              ((P.nz + SPH_TZ - 1) / SPH_TZ);
    A.chunk = (int)std::min<long long>(A.tiles, 1024);
    A.basis_b = (sizeof(double) * SPH_P * (size_t)n_f + 255) / 256 * 256;
    // tables held at a time (sph_adj_fast keeps a row below 8 MB, the grid
    // holds 65535 of them)
    const size_t row = sizeof(float4) * 2 * (size_t)B.n;
    const int most = (int)std::min<size_t>((SPH_SCRATCH_BYTES - (size_t(17) << 20)) / row, 65535);
    const int least = std::max(4, std::min(8, (P.nq + 15) / 16));
    A.slices = std::max(1, std::min({1024 / A.chunk, (P.nq + least - 1) / least, most}));
    A.qps = (P.nq + A.slices - 1) / A.slices;
    A.slices = (P.nq + A.qps - 1) / A.qps;
    A.per = std::max(1, std::min(most / A.slices, A.qps));
    A.table_b = (row * A.per * A.slices + 255) / 256 * 256;
    const bool direct = A.slices == 1 && A.per >= A.qps;
    A.part_b = direct ? 0 : sizeof(double) * (size_t)A.slices * A.chunk * SPH_TVOX;
    return A;
}

size_t sph_adj_workspace_bytes(const Problem &P, int n_f, double f_min, double df)
{
    SphBand B;
    if (sph_adj_fast(P, n_f, f_min, df, B)) {
        const SphAdjPlan A = sph_adj_plan(P, B, n_f);
        return A.basis_b + A.table_b + A.part_b;
    }
    const int S = sph_adj_slices(P);
    return S > 1 ? sizeof(double) * (size_t)S * P.nx * P.ny * P.nz : 0;
}

static hipError_t launch_sph_table_adjoint(const Problem &P, const SphBand &B, const float2 *u,
                                           int n_f, double f_min, double df, void *img, int img_dt,
                                           char *work, hipStream_t s)
{
    const SphAdjPlan A = sph_adj_plan(P, B, n_f);
    double *ab = (double *)work;
    float4 *table = (float4 *)(work + A.basis_b);
    double *part = A.part_b ? (double *)(work + A.basis_b + A.table_b) : nullptr;
    const int qt = std::max(1, SPH_STAGE / (48 * B.w));
    const size_t shm = (sizeof(float4) * 3 * B.w + sizeof(int2)) * (size_t)qt;
    const int batches = (A.qps + A.per - 1) / A.per;
    const unsigned gx = (B.n + 2 * SPH_TTHREADS - 1) / (2 * SPH_TTHREADS);
    const bool small = (long long)gx * A.slices * A.per <= 1024 && n_f <= 512;
    if (!small)
        hipLaunchKernelGGL(sph_adj_basis_kernel, dim3((n_f + 63) / 64), dim3(64), 0, s, P, B, n_f, f_min,
                           df, ab);
    for (long long t0 = 0; t0 < A.tiles; t0 += A.chunk) {
        const unsigned nt = (unsigned)std::min<long long>(A.chunk, A.tiles - t0);
        for (int k = 0; k < batches; ++k) {
            const SphBatch bt{A.qps, k * A.per, std::min(A.qps, (k + 1) * A.per)};
            auto tab = [&](auto kernel, int sh, size_t lds) {
                hipLaunchKernelGGL(kernel, dim3(gx, A.slices * (bt.b1 - bt.b0)), dim3(SPH_TTHREADS * sh), lds,
                                   s, P, B, bt, u, ab, n_f, f_min, df, table);
            };
            if (batches > 1 || t0 == 0) {   // one batch: the tables serve every chunk
                const size_t basis = sizeof(double) * SPH_P * n_f;
                const size_t sums = sizeof(double) * 3 * 2 * SPH_P * SPH_TTHREADS;
                if (!small) tab(sph_table_kernel<1, false>, 1, 0);
                else if (n_f < 32) tab(sph_table_kernel<1, true>, 1, basis);
                else tab(sph_table_kernel<4, true>, 4, std::max(basis, sums));
            }
            auto eval = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, dim3(nt, A.slices), dim3(SPH_THREADS), shm, s, P, B, bt,
                                   table, qt, t0, img, img_dt, part, k > 0 ? 1 : 0);
            };
            P.sph_ns > 1 ? eval(sph_eval_kernel<true>) : eval(sph_eval_kernel<false>);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        if (part)
            hipLaunchKernelGGL(sph_eval_sum_kernel, dim3(nt, SPH_TZ), dim3(SPH_THREADS), 0, s, P, B,
                               part, A.slices, t0, img, img_dt);
    }
    return hipGetLastError();
}

hipError_t launch_sph_backproject(const Problem &P, const float2 *u, int n_f, double f_min,
                                  double df, void *img, int img_dt, double *work, hipStream_t s)
{
    SphBand B;
    if (sph_adj_fast(P, n_f, f_min, df, B))
        return work ? launch_sph_table_adjoint(P, B, u, n_f, f_min, df, img, img_dt, (char *)work, s)
                    : hipErrorInvalidValue;
    const long long N = (long long)P.nx * P.ny * P.nz;
    const int n_fp = (n_f + SPH_ANCHOR - 1) / SPH_ANCHOR * SPH_ANCHOR;
    const int qt = (SPH_VQ / n_fp) > 1 ? SPH_VQ / n_fp : 1;
    const size_t shm = sizeof(float2) * (size_t)qt * n_fp;
    const long long threads = (N + SPH_NV - 1) / SPH_NV;
    const int S = sph_adj_slices(P);
    if (S > 1 && !work) return hipErrorInvalidValue;
    const int qps = (P.nq + S - 1) / S;
    double *slice_sum = S > 1 ? work : nullptr;
    dim3 grid((unsigned)((threads + SPH_THREADS - 1) / SPH_THREADS), (unsigned)S);
    if (img_dt == 0)
        hipLaunchKernelGGL(sph_adj_kernel<0>, grid, dim3(SPH_THREADS), shm, s, P, u, n_f, f_min, df,
                           img, slice_sum, qps);
    else
        hipLaunchKernelGGL(sph_adj_kernel<1>, grid, dim3(SPH_THREADS), shm, s, P, u, n_f, f_min, df,
                           img, slice_sum, qps);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || S == 1) return e;
    hipLaunchKernelGGL(sph_adj_sum_kernel, dim3((unsigned)((N + SPH_THREADS - 1) / SPH_THREADS)),
                       dim3(SPH_THREADS), 0, s, slice_sum, S, N, img, img_dt);
    return hipGetLastError();
}

}  // namespace oat
