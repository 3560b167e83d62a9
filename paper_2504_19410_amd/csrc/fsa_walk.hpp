// Work walks of the persistent pass kernels: which work items each
// workgroup of a grid visits, in what order.  Plain C++ with host/device
// qualifiers, so that the CPU tests can check that every mode visits every
// item exactly once.
#pragma once

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#else
#define __host__
#define __device__
#define __forceinline__ inline
#endif

namespace fsa {

// The work items one workgroup visits, in order: first, first + stride, ...
// below last (uniform over the group).
//   Default: a contiguous chunk per workgroup.
//   XCD (for tiles whose rows are narrower than a 128-byte cache line, so
// that neighbouring tiles share lines): the dispatcher deals workgroups to
// the 8 XCDs in turn (workgroup g runs on XCD g mod 8), and each XCD has its
// own L2.  Each XCD takes a contiguous eighth of the items, which its
// workgroups visit side by side (workgroup g, the s-th of its XCD, takes
// items s, s + G/8, ... of that eighth): neighbouring tiles are in flight at
// the same time under one L2, so a shared line is read from memory once
// instead of once per tile.
//   PAIR (same case): the two tiles 2j and 2j + 1, which share every 128-byte
// line they touch when a tile row is 64 bytes, go to two workgroups of one
// XCD (g and g + 8) that run side by side, each stepping two items at a time
// through the pair chunk of the two; the pairs take contiguous chunks like
// the default, so only two workgroups ever read one line at once.
//   EVEN (pass C): contiguous chunks that differ by at most one item.  Chunks of
// equal size leave workgroups without any: the bins of an axis are one more than
// a power of two, so the work is often just over a whole number of items per
// workgroup (33024 pencils at 128^3 on 1024 workgroups of 16: 2.02, of which
// chunks of 3 keep a third of the workgroups idle).  Pass C is bound by the
// arithmetic its waves overlap: at 96^3, 128^3 and 192^3 FP64 24.3 -> 20.4,
// 36 -> 33 and 120 -> 116 us, at 512 x 64 x 64 48 -> 42, at 128^3 FP32 21.4 ->
// 19.2.  The passes bound by memory gain nothing from more waves (B) or lose
// a little (D at 256^3 FP64: 175 -> 181 us).
enum WalkMode { kWalkChunk = 0, kWalkXcd = 1, kWalkPair = 2, kWalkEven = 3 };
struct Walk {
    int first, last, stride;
    // the walk of workgroup g of a grid of G workgroups over `items` items
    template <int MODE>
    __host__ __device__ __forceinline__ static Walk make(int items, int G, int g) {
        if (MODE == kWalkPair && G >= 16 && (G & 15) == 0) {
            const int pairs = (items + 1) >> 1, np = G >> 1;
            const int x = g & 7, s = g >> 3, q = s >> 1, b = s & 1;
            const int c = (pairs + np - 1) / np, pg = q * 8 + x;
            const int lo = 2 * pg * c + b, hi = 2 * (pg * c + c);
            return Walk{lo, hi < items ? hi : items, 2};
        }
        if (MODE == kWalkXcd && G >= 8 && (G & 7) == 0) {
            const int per = (items + 7) / 8, x = g & 7, s = g >> 3;
            const int lo = x * per, hi = lo + per < items ? lo + per : items;
            return Walk{lo + s, hi, G >> 3};
        }
        if (MODE == kWalkEven) {
            const int c = items / G, r = items - c * G;
            const int first = g * c + (g < r ? g : r);
            return Walk{first, first + c + (g < r ? 1 : 0), 1};
        }
        const int c = (items + G - 1) / G;
        const int first = g * c;
        return Walk{first, first + c < items ? first + c : items, 1};
    }
};

}  // namespace fsa
