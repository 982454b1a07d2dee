// Host check of FBP's unclamped sample index (fbp_kernel with HELD): where
// fbp_window_holds says that no clamp is needed, the index that the kernel forms
// in FP32, tile-relative, with its tolerance added, lies in 1 .. win - 2 (the
// decision at an integer may step it down by one) for voxels of whole tiles, the
// part beyond the grid included.  The kernel's operations are repeated in FP32;
// its square root and reciprocal square root are also taken up to 2 and 1.5 units
// in the last place off either way.  Checked per tile and transducer: the tile's
// corners, its voxel nearest the transducer (between them the extremes of the
// distance) and eight more; every voxel with "all".
//
// Input on stdin: nx ny nz dx x0 y0 z0 c0 dt t0 K Q, then Q lines x y z (mm).
// Prints "OK <held> <indices> <least> <win - 2 - most>" or the first failure.
#define __host__
#define __device__
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <vector>

#include "oat_fbp_window.hpp"

using namespace oat;

static float ulps(float v, float n) { return v + n * (std::nextafterf(v, INFINITY) - v); }

int main(int argc, char **argv)
{
    const bool all = argc > 1 && !std::strcmp(argv[1], "all");
    int n[3], K, Q;
    double dx, o[3], c0, dt, t0;
    if (std::scanf("%d %d %d %lf %lf %lf %lf %lf %lf %lf %d %d", &n[0], &n[1], &n[2], &dx, &o[0], &o[1], &o[2],
                   &c0, &dt, &t0, &K, &Q) != 12) {
        std::printf("FAIL bad header\n");
        return 1;
    }
    std::vector<double> uq(3 * (size_t)Q);
    double reach = 0.0;
    for (int q = 0; q < Q; ++q)
        for (int a = 0; a < 3; ++a) {
            double r;
            if (std::scanf("%lf", &r) != 1) {
                std::printf("FAIL bad transducer %d\n", q);
                return 1;
            }
            uq[3 * q + a] = (r - o[a]) / dx;
            reach = std::max(reach, std::fabs(uq[3 * q + a]));
        }
    reach += std::max(n[0], std::max(n[1], n[2])) + 16;
    const double sg = dx / (c0 * dt);
    if (!fbp_window_holds(reach, sg, t0 / dt)) {
        std::printf("OK 0 0 0 0\n");
        return 0;
    }
    const float sigma = (float)sg, tau = (float)(t0 / dt), hd = fbp_half_diag();
    const int win = fbp_window(sigma);
    const int T[3] = {FBP_TX, FBP_TY, FBP_TZ};
    long indices = 0, least = 1L << 40, room = 1L << 40;
    unsigned rnd = 12345;
    for (int bz = 0; bz * T[2] < n[2]; ++bz)
        for (int by = 0; by * T[1] < n[1]; ++by)
            for (int bx = 0; bx * T[0] < n[0]; ++bx) {
                const int lo[3] = {bx * T[0], by * T[1], bz * T[2]};
                float c[3];
                for (int a = 0; a < 3; ++a) c[a] = (float)lo[a] + 0.5f * (float)(T[a] - 1);
                for (int q = 0; q < Q; ++q) {
                    const double *u = &uq[3 * (size_t)q];
                    const float wx = c[0] - (float)u[0], wy = c[1] - (float)u[1], wz = c[2] - (float)u[2];
                    const float root = sqrtf(wx * wx + wy * wy + wz * wz);
                    auto voxel = [&](int tx, int ty, int tz) {
                        for (int d = -2; d <= 2; d += 2) {
                            const float dc = ulps(root, (float)d);
                            const int k0 = fbp_first_sample(dc, sigma, tau);
                            const float tol = fmaf(4e-7f, (dc + hd + 1.f) * sigma,
                                                   6.2e-8f * (2.f * hd * sigma + (float)win));
                            const float kx = (float)((u[0] - (double)c[0]) * sg), ky = (float)((u[1] - (double)c[1]) * sg);
                            const float kz = (float)((double)tol - (t0 / dt + (double)k0));
                            const double z = ((double)(lo[2] + tz) - u[2]) * sg;
                            const float z2 = (float)(z * z);
                            const float fx = (float)((tx - 0.5 * (T[0] - 1)) * sg), fy = (float)((ty - 0.5 * (T[1] - 1)) * sg);
                            const float vx = fx - kx, vy = fy - ky;
                            const float r2 = fmaf(vy, vy, vx * vx) + z2;
                            const float rs = (float)(1.0 / std::sqrt((double)r2));
                            for (int e = -1; e <= 1; ++e) {
                                const long li = (long)std::floor(fmaf(r2, ulps(rs, 1.5f * e), kz));
                                least = std::min(least, li);
                                room = std::min(room, (long)win - 2 - li);
                                ++indices;
                            }
                        }
                    };
                    if (all) {
                        for (int tz = 0; tz < T[2]; ++tz)
                            for (int ty = 0; ty < T[1]; ++ty)
                                for (int tx = 0; tx < T[0]; ++tx) voxel(tx, ty, tz);
                    } else {
                        for (int k = 0; k < 8; ++k)
                            voxel((k & 1) * (T[0] - 1), (k >> 1 & 1) * (T[1] - 1), (k >> 2) * (T[2] - 1));
                        int g[3];
                        for (int a = 0; a < 3; ++a)
                            g[a] = (int)std::min(std::max(std::floor(u[a] - lo[a] + 0.5), 0.0), (double)(T[a] - 1));
                        voxel(g[0], g[1], g[2]);
                        for (int k = 0; k < 8; ++k) {
                            rnd = rnd * 1664525u + 1013904223u;
                            voxel(rnd >> 8 & 15, rnd >> 12 & 15, rnd >> 16 & 7);
                        }
                    }
                    if (least < 1 || room < 0) {
                        std::printf("FAIL tile (%d,%d,%d) transducer %d: least %ld, room %ld, win %d\n", bx, by, bz,
                                    q, least, room, win);
                        return 1;
                    }
                }
            }
    std::printf("OK 1 %ld %ld %ld\n", indices, least, room);
    return 0;
}
