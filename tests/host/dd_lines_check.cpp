// Lines per workgroup of the double-double transforms (dd_lines), at every length,
// over line counts and CU counts.  Prints "ok" if every launch is within the limits
// its kernels assume and no allowed shape of a launch of few workgroups leaves fewer
// lines on the fullest CU, or as few in larger workgroups.
#include <cstdio>
#include <initializer_list>

#include "../../paper_2504_19410_amd/csrc/fsa_dd.hpp"

using namespace fsa;

int main() {
    int bad = 0;
    for (int cus : {1, 64, 256, 304})
        for (int P = 16; P <= kDDMaxP; P *= 2) {
            const int n = dd_line_threads(P);
            if (n < 1 || n > kDDThreads || (n & (n - 1)) != 0 || P % n != 0) ++bad;
            if (P / n > kDDMaxP / kDDThreads) ++bad;  // the fused pass's kept products
            for (long lines = 1; lines < 200000; lines += lines < 3000 ? 1 : 997) {
                const int W = dd_lines(P, lines, cus);
                const long groups = (lines + W - 1) / W;
                if (W < 1 || (W & (W - 1)) != 0 || W * n > kDDThreads) ++bad;
                if (2 * W * P * 16 > 65536) ++bad;  // LDS bytes of the tile
                auto on_one = [&](int w) { return ((lines + w - 1) / w + cus - 1) / cus * w; };
                bool few = true;  // every larger shape has fewer than four groups per CU
                for (int w = kDDThreads / n; w >= 1 && w * n >= 64; w /= 2) {
                    if (few && (on_one(w) < on_one(W) || (on_one(w) == on_one(W) && w > W))) ++bad;
                    few = few && (lines + w - 1) / w < 4 * cus;
                }
            }
        }
    std::printf(bad ? "bad %d\n" : "ok\n", bad);
    return bad != 0;
}
