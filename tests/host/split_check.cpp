// Host check of the work splits of G and G^T (seg_fwd_grid, adj_grid) over
// brick counts, transducer counts and shell windows: the slices cover every
// transducer once, grids and LDS stay inside the device's limits, whole-window
// slices are whole and others divide a window, and the brick sums of G^T's
// slices stay below a bound whatever the number of transducers.
// Prints "OK <checked>" or the first failure.
#include <cstdio>

#include "oat_internal.hpp"

using namespace oat;

static long checked = 0;

static bool covers(int slices, int per, int nq)
{
    return per >= 1 && slices >= 1 && (long long)slices * per >= nq && (long long)(slices - 1) * per < nq;
}

static bool check(int nbricks, int nq, int window)
{
    ++checked;
    const FwdGrid f = seg_fwd_grid(nbricks, nq, window);
    bool ok = covers(f.slices, f.per, nq) && f.slices <= 65535;
    const long long rows = f.parts > 0 ? f.per : 16;
    ok = ok && (f.parts == 0 || (f.per <= FWD_SPLIT_Q && f.parts >= 1 && f.parts <= 16));
    // two words a node of the box, the rows' shell sums, the waves' first rings, and 1 KB of the rest
    ok = ok && 8ll * BOX_WORDS + (rows * 8 + 16 * 4) * window + 1024 <= 160 * 1024;
    if (!ok) {
        std::printf("FAIL G: %d bricks, %d transducers, window %d: %d slices of %d in %d parts\n", nbricks, nq,
                    window, f.slices, f.per, f.parts);
        return false;
    }
    const AdjGrid a = adj_grid(nbricks, nq);
    ok = covers(a.slices, a.per, nq) && a.slices <= 65535 && a.parts >= 1 && a.parts <= 16;
    ok = ok && (a.per % ADJ_WINDOW == 0 || ADJ_WINDOW % a.per == 0);
    // at most 8192 workgroups, or the 8 whole-window slices of large grids
    ok = ok && ((long long)a.slices * nbricks <= 8192 || a.slices <= 8);
    if (!ok)
        std::printf("FAIL G^T: %d bricks, %d transducers: %d slices of %d in %d parts\n", nbricks, nq, a.slices,
                    a.per, a.parts);
    return ok;
}

int main()
{
    const int windows[] = {3, 17, 40, 69, 70, 104, 208, 255, 256};
    for (long long b = 1; b <= 4000000; b = b < 300 ? b + 1 : b + b / 7)
        for (long long q = 1; q <= 700000000; q = q < 300 ? q + 1 : q + q / 5)
            for (int w : windows) {
                // plans hold fewer than 2^31 samples, of at least `window` a transducer
                if (q * w >= (1ll << 31)) continue;
                if (!check((int)b, (int)q, w)) return 1;
            }
    std::printf("OK %ld\n", checked);
    return 0;
}
