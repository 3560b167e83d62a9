// The even walk of pass C (fsa_walk.hpp): every workgroup takes a contiguous run,
// the runs follow each other without gaps and their lengths differ by at most one,
// none empty while there are as many items as workgroups.  Exit status 0 = pass.
#include <cstdio>

#include "../../paper_2504_19410_amd/csrc/fsa_walk.hpp"

using namespace fsa;

int main() {
    for (int G = 1; G <= 2048; G = G < 64 ? G + 1 : G + 16)
        for (int items = G; items <= 40000; items += items < 700 ? 1 : 211) {
            int at = 0, lo = items, hi = 0;
            for (int g = 0; g < G; ++g) {
                const Walk w = Walk::make<kWalkEven>(items, G, g);
                const int n = w.last - w.first;
                if (w.first != at || w.stride != 1 || n < 1) {
                    std::printf("items %d G %d g %d: %d .. %d step %d\n", items, G, g, w.first,
                                w.last, w.stride);
                    return 1;
                }
                at = w.last;
                lo = n < lo ? n : lo;
                hi = n > hi ? n : hi;
            }
            if (at != items || hi - lo > 1) {
                std::printf("items %d G %d: end %d, runs of %d .. %d\n", items, G, at, lo, hi);
                return 1;
            }
        }
    // the last item of the largest launch: no overflow on the way
    const int big = 2147483647 / 2;
    if (Walk::make<kWalkEven>(big, 2048, 2047).last != big) return 1;
    std::printf("OK\n");
    return 0;
}
