// Lines per workgroup of the double-double transforms (dd_lines), at every length,
// over line counts and CU counts.  Prints "ok" if every launch is within the limits
// its kernels assume and a launch that cannot give every CU a workgroup takes no
// more than one wave's lines in each.
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
                if (groups < cus && W > 1 && W * n > 64) ++bad;
                // and no fewer lines than that needs
                if (2 * W * n <= kDDThreads && (lines + 2 * W - 1) / (2 * W) >= cus) ++bad;
            }
        }
    std::printf(bad ? "bad %d\n" : "ok\n", bad);
    return bad != 0;
}
