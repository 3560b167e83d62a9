// fsa_dd.hip -- the extended-precision (double-double) mode: tensor build and
// evaluation, Coulomb kernels (Table 1), grids N_j = 2^a <= 1024.
//
// The paper runs its method in quadruple precision to reach errors near
// 1e-34 once the tensor is generated in high precision (Sec. 5.1, Table 2).
// gfx950 has no FP128; double-double (hi + lo, 106 bits, fsa_dd.hpp) is the
// closest native format.  The method is the same as in FP32/FP64:
//   tensor  T^[p] = (DCT-I(T(1))[p] + W(|k_p|)) / prod P_j  on the octant
//           (the DCT-I as the real part of the DFT of the even extension),
//           T(1) = prod h_j U^eps(|n h|), U^eps = erf(r/eps)/(4 pi r) (3D) or
//           erf(r/eps)/(2 pi r) (2D), W = (1 - e^{-k^2 eps^2/4})/k^2 (3D) or
//           erf(k eps/2)/k (2D);
//   passes  the 2x zero-padded convolution, forward FFTs along the axes from
//           the last to axis 1, the fused forward FFT x T^ x inverse FFT
//           along axis 0, inverse FFTs back; input zero padding and output
//           crop folded into the loads and stores.
// rho and phi are real, so the last axis keeps only its bins 0 .. N_last (the
// others are conjugates), and its transforms take two rows in one complex FFT.
// A workgroup transforms W neighbouring lines (dd_lines) with a radix-4 FFT in LDS:
// every wave is full and the strided axes are read in runs of W values.  A thread
// stays with one line, so its addresses cost one division each.  The arithmetic
// bounds it (a double-double addition is 20 FP64 operations, a product 10): 64^3
// took 344 us on the whole complex spectrum with one line per workgroup of P / 4
// threads (half a wave at P = 128), 156 us this way; its fused pass 180 us, now 77.
// Arrays of reals are interleaved (hi, lo) pairs; complex values are
// (re.hi, re.lo, im.hi, im.lo).
#include <hip/hip_runtime.h>

#include "fsa_dd.hpp"
#include "fsa_internal.hpp"

namespace fsa {

namespace {

struct cdd {
    dd re, im;
};

__device__ __forceinline__ cdd cadd(cdd a, cdd b) { return cdd{a.re + b.re, a.im + b.im}; }
__device__ __forceinline__ cdd csub(cdd a, cdd b) { return cdd{a.re - b.re, a.im - b.im}; }
__device__ __forceinline__ cdd cmul(cdd a, cdd b) {
    return cdd{a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
__device__ __forceinline__ cdd cconj(cdd a) { return cdd{a.re, -a.im}; }

// Thread tid's place in its workgroup's W lines: a line has dd_line_threads(P)
// threads, neighbours of one line (rows, contiguous) or of W lines side by side
// (strided axes, where neighbouring lines are neighbours in memory).
struct DDThread {
    int w, t, n;  // line; first element; threads per line (a power of two)
    __device__ __forceinline__ DDThread(bool rows, int W, int P) {
        n = dd_line_threads(P);
        const int tid = (int)threadIdx.x;
        const int logn = 31 - __clz(n), logw = 31 - __clz(W);
        w = rows ? tid >> logn : tid & (W - 1);
        t = rows ? tid & (n - 1) : tid >> logw;
    }
};

// tw[m] = exp(-2 pi i m / P), m < P/2
__global__ void k_dd_twiddle(cdd* __restrict__ tw, int P) {
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= P / 2) return;
    dd s, c;
    dd_sincos_turn((double)m / (double)P, &s, &c);
    tw[m] = cdd{c, -s};
}

struct DDGeom {
    int d;
    int N[3], P[3];
    double L[3];
    double eps;
    int kind;
};

__device__ void octant_index(long i, const int* D, int d, int* a) {
    a[0] = (int)(i % D[0]);
    long r = i / D[0];
    a[1] = d > 1 ? (int)(r % D[1]) : 0;
    a[2] = d > 2 ? (int)(r / D[1]) : 0;
}

// T(1) on the octant (axis 0 innermost), FP64-free: every step in DD.
__global__ void k_dd_sample(dd* __restrict__ out, DDGeom g) {
    int D[3] = {g.N[0] + 1, g.d > 1 ? g.N[1] + 1 : 1, g.d > 2 ? g.N[2] + 1 : 1};
    const long n = (long)D[0] * D[1] * D[2];
    const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (i >= n) return;
    int a[3];
    octant_index(i, D, g.d, a);
    dd r2 = dd_of(0.0), hprod = dd_of(1.0);
    for (int j = 0; j < g.d; ++j) {
        const dd h = dd_of(2.0 * g.L[j]) / dd_of((double)g.N[j]);
        hprod = hprod * h;
        const dd x = h * (double)a[j];
        r2 = r2 + x * x;
    }
    const dd eps = dd_of(g.eps);
    const dd sqpi = dd_sqrt(dd_pi());
    dd u;
    if (r2.hi == 0.0) {
        // limits of erf(r/eps)/(c r): 2/(sqrt(pi) eps c)
        u = g.kind == FSA_COULOMB_3D ? dd_of(1.0) / (dd_pi() * sqpi * eps * 2.0)
                                     : dd_of(1.0) / (dd_pi() * sqpi * eps);
    } else {
        const dd r = dd_sqrt(r2);
        const dd e = dd_erf(r / eps);
        u = g.kind == FSA_COULOMB_3D ? e / (dd_pi() * r * 4.0) : e / (dd_pi() * r * 2.0);
    }
    out[i] = hprod * u;
}

// T^ = (DCT(T1) + W(|k|)) / prod P_j
__global__ void k_dd_finalize(const dd* __restrict__ dct, dd* __restrict__ out, DDGeom g) {
    int D[3] = {g.N[0] + 1, g.d > 1 ? g.N[1] + 1 : 1, g.d > 2 ? g.N[2] + 1 : 1};
    const long n = (long)D[0] * D[1] * D[2];
    const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (i >= n) return;
    int a[3];
    octant_index(i, D, g.d, a);
    dd k2 = dd_of(0.0);
    double prodP = 1.0;
    for (int j = 0; j < g.d; ++j) {
        const dd k = dd_pi() * (double)a[j] / (2.0 * g.L[j]);
        k2 = k2 + k * k;
        prodP *= (double)g.P[j];
    }
    const dd eps = dd_of(g.eps);
    dd w;
    if (g.kind == FSA_COULOMB_3D) {
        w = k2.hi == 0.0 ? eps * eps * 0.25 : -dd_expm1(-(k2 * eps * eps * 0.25)) / k2;
    } else {
        const dd sqpi = dd_sqrt(dd_pi());
        if (k2.hi == 0.0) {
            w = eps / sqpi;
        } else {
            const dd k = dd_sqrt(k2);
            w = dd_erf(k * eps * 0.5) / k;
        }
    }
    out[i] = (dct[i] + w) / prodP;  // prod P_j is a power of two: exact
}

// ---------------------------------------------------------------------------
// Evaluation: W lines per workgroup, radix-4 steps in LDS.
// ---------------------------------------------------------------------------

// The W lines of a workgroup in LDS, real and imaginary parts apart (a wave's
// 16-byte accesses are neighbours): value t of line w at w P + t.
struct DDTile {
    dd *re, *im;
    __device__ __forceinline__ cdd get(int i) const { return cdd{re[i], im[i]}; }
    __device__ __forceinline__ void put(int i, cdd v) const {
        re[i] = v.re;
        im[i] = v.im;
    }
};

// In-place decimation in time on every line x[w P, (w + 1) P) (bit-reversed
// order in, natural order out); tw[m] = exp(-2 pi i m / P), m < P/2.  The
// radix-2 stages run in
// pairs (len/2, len) as one radix-4 step per group of four points, with one
// exchange through LDS per pair, after a leading radix-2 stage when log2 P is
// odd or a radix-4 step without twiddles when it is even: points i0, i0 + q, i0 + 2q, i0 + 3q (q = len/4, j = i0 mod len < q)
// take the len/2 stage's twiddle w_len^(2j) on the odd points of each half,
// then the len stage's w_len^j on the second half, times -i (forward) or +i
// (inverse) for the upper pair.
template <bool INV>
__device__ void dd_fft_lds(const DDTile& x, int W, int P, int logP, const cdd* __restrict__ tw) {
    int len = 4;
    if (logP & 1) {
        for (int b = threadIdx.x; b < W * (P / 2); b += blockDim.x) {
            const cdd u = x.get(2 * b), v = x.get(2 * b + 1);
            x.put(2 * b, cadd(u, v));
            x.put(2 * b + 1, csub(u, v));
        }
        __syncthreads();
        len = 8;
    } else {  // groups of four points: every twiddle is 1
        for (int b = threadIdx.x; b < W * (P / 4); b += blockDim.x) {
            const cdd a0 = x.get(4 * b), a1 = x.get(4 * b + 1);
            const cdd a2 = x.get(4 * b + 2), a3 = x.get(4 * b + 3);
            const cdd b0 = cadd(a0, a1), b1 = csub(a0, a1);
            const cdd b2 = cadd(a2, a3), u3 = csub(a2, a3);
            const cdd t3 = INV ? cdd{-u3.im, u3.re} : cdd{u3.im, -u3.re};
            x.put(4 * b, cadd(b0, b2));
            x.put(4 * b + 2, csub(b0, b2));
            x.put(4 * b + 1, cadd(b1, t3));
            x.put(4 * b + 3, csub(b1, t3));
        }
        __syncthreads();
        len = 16;
    }
    for (int lq = (logP & 1) ? 1 : 2; len <= P; len <<= 2, lq += 2) {
        const int q = len >> 2, step = P / len;  // q = 2^lq divides P / 4
        for (int b = threadIdx.x; b < W * (P / 4); b += blockDim.x) {
            const int g = b >> lq, j = b & (q - 1);
            const int i0 = g * len + j;
            const cdd w2 = INV ? cconj(tw[2 * j * step]) : tw[2 * j * step];
            const cdd wa = INV ? cconj(tw[j * step]) : tw[j * step];
            const cdd a0 = x.get(i0), a1 = cmul(x.get(i0 + q), w2);
            const cdd a2 = x.get(i0 + 2 * q), a3 = cmul(x.get(i0 + 3 * q), w2);
            const cdd b0 = cadd(a0, a1), b1 = csub(a0, a1);
            const cdd b2 = cadd(a2, a3), b3 = csub(a2, a3);
            const cdd t2 = cmul(b2, wa);
            const cdd u3 = cmul(b3, wa);
            const cdd t3 = INV ? cdd{-u3.im, u3.re} : cdd{u3.im, -u3.re};
            x.put(i0, cadd(b0, t2));
            x.put(i0 + 2 * q, csub(b0, t2));
            x.put(i0 + q, cadd(b1, t3));
            x.put(i0 + 3 * q, csub(b1, t3));
        }
        __syncthreads();
    }
}

__device__ __forceinline__ int bitrev(int t, int logP) {
    return (int)(__brev((unsigned)t) >> (32 - logP));
}

// DCT-I along axis ax of the octant (D_j = N_j + 1 points per axis), as the
// real part of the length-2N DFT of each line's even extension (x[m] for
// m <= N, x[2N - m] above): sum_m c_m x[m] cos(pi p m / N), c_0 = c_N = 1,
// else 2.  W lines (a power of two) per workgroup; tw: the axis' twiddles of
// length 2N.
__global__ __launch_bounds__(kDDThreads) void k_dd_dct(const dd* __restrict__ in,
                                                     dd* __restrict__ out, DDGeom g, int ax,
                                                     long lines, int W,
                                                     const cdd* __restrict__ tw) {
    extern __shared__ dd lds[];
    const int D0 = g.N[0] + 1, D1 = g.d > 1 ? g.N[1] + 1 : 1;
    const int N = g.N[ax], P = 2 * N;
    const DDTile x{lds, lds + W * P};
    int logP = 0;
    while ((1 << logP) < P) ++logP;
    const long stride = ax == 0 ? 1 : ax == 1 ? D0 : (long)D0 * D1;
    auto base = [&](long l) {
        if (ax == 0) return l * D0;                                       // l = a2 D1 + a1
        if (ax == 1) return (l / D0) * (long)D1 * D0 + l % D0;            // l = a2 D0 + a0
        return l;                                                         // l = a1 D0 + a0
    };
    const DDThread th(ax == 0, W, P);
    const long l = (long)blockIdx.x * W + th.w;
    const bool act = l < lines;
    const long b = act ? base(l) : 0;
    for (int t = th.t; t < P; t += th.n) {
        const int m = t <= N ? t : P - t;
        x.put(th.w * P + bitrev(t, logP), cdd{act ? in[b + m * stride] : dd_of(0.0), dd_of(0.0)});
    }
    __syncthreads();
    dd_fft_lds<false>(x, W, P, logP, tw);
    if (act)
        for (int p = th.t; p <= N; p += th.n) out[b + p * stride] = x.re[th.w * P + p];
}

// Where a line lives: element t of line l is at base(l) + t * es, with
// base(l) = (l / nb) * sa + (l % nb) * sb (a two-level line index).
struct DDLines {
    long sa, sb, es;
    int nb;
    __device__ long base(long l) const { return (l / nb) * sa + (l % nb) * sb; }
};

enum DDMode { DD_FWD_REAL = 0, DD_FWD = 1, DD_CONV = 2, DD_INV = 3, DD_INV_REAL = 4 };

struct DDConv {  // octant lookup of T^ along axis-0 lines at (p1, p2)
    const dd* tensor;
    int N[3], P[3], D0, D1, d;
};

// W lines: load n_in inputs each (the rest zero), transform, store n_out
// outputs each.  The real modes run along the last axis and take the rows 2l and
// 2l + 1 of line l as one complex row a + i b (N_0 is even, so rows pair up);
// their spectra A and B hold the bins 0 .. P/2:
//   A[k] = (Z[k] + conj Z[P-k]) / 2,  B[k] = (Z[k] - conj Z[P-k]) / 2i.
template <int MODE>
__global__ __launch_bounds__(kDDThreads) void k_dd_pass(const void* __restrict__ in,
                                                        void* __restrict__ out, DDLines li,
                                                        DDLines lo, long lines, int W, int P,
                                                        int logP, int n_in, int n_out,
                                                        const cdd* __restrict__ tw, DDConv cv) {
    extern __shared__ dd lds[];
    const DDTile x{lds, lds + W * P};
    constexpr bool REAL = MODE == DD_FWD_REAL || MODE == DD_INV_REAL;
    const DDThread th(REAL, W, P);
    const int xw = th.w * P;
    const long line = (long)blockIdx.x * W + th.w;
    const bool act = line < lines;
    // bases of the line, or of its two rows
    const long l0 = act ? (REAL ? 2 * line : line) : 0, l1 = REAL && act ? l0 + 1 : l0;
    const long ia = li.base(l0), ib = li.base(l1), oa = lo.base(l0), ob = lo.base(l1);
    for (int t = th.t; t < P; t += th.n) {
        cdd v = cdd{dd_of(0.0), dd_of(0.0)};
        if (act) {
            if constexpr (MODE == DD_FWD_REAL) {
                if (t < n_in) {
                    v.re = ((const dd*)in)[ia + t];
                    v.im = ((const dd*)in)[ib + t];
                }
            } else if constexpr (MODE == DD_INV_REAL) {
                // Z[k] = A[k] + i B[k], Z[P-k] = conj A[k] + i conj B[k]
                const int k = t <= P / 2 ? t : P - t;
                cdd a = ((const cdd*)in)[ia + k];
                cdd b = ((const cdd*)in)[ib + k];
                if (t > P / 2) {
                    a = cconj(a);
                    b = cconj(b);
                }
                v = cdd{a.re - b.im, a.im + b.re};
            } else {
                if (t < n_in) v = ((const cdd*)in)[ia + t * li.es];
            }
        }
        x.put(xw + bitrev(t, logP), v);
    }
    __syncthreads();
    if constexpr (MODE == DD_CONV) {
        dd_fft_lds<false>(x, W, P, logP, tw);
        // neighbours of one line: T^ and the tile are contiguous along it
        const DDThread tr(true, W, P);
        const int rw = tr.w * P;
        const long l = (long)blockIdx.x * W + tr.w, ln = l < lines ? l : 0;
        // line at (p1, p2), p2 <= N_2, in 3D; p1 <= N_1 in 2D
        int a1 = (int)ln, a2 = 0;
        if (cv.d == 3) {
            const int p1 = (int)(ln / (cv.N[2] + 1));
            a2 = (int)(ln - (long)p1 * (cv.N[2] + 1));
            a1 = p1 <= cv.N[1] ? p1 : cv.P[1] - p1;
        }
        const dd* trow = cv.tensor + ((long)a2 * cv.D1 + a1) * cv.D0;
        // x (natural order) times T^, back into bit-reversed order for the
        // inverse: every product is formed before any is written back
        // (fixed trip counts keep the array in registers)
        constexpr int kKeep = kDDMaxP / kDDThreads;  // P / dd_line_threads(P) <= 8
        cdd keep[kKeep];
#pragma unroll
        for (int r = 0; r < kKeep; ++r) {
            const int t = tr.t + r * tr.n;
            if (t < P) {
                const int a0 = t <= cv.N[0] ? t : P - t;
                const dd s = trow[a0];
                cdd v = x.get(rw + t);
                v.re = v.re * s;
                v.im = v.im * s;
                keep[r] = v;
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kKeep; ++r) {
            const int t = tr.t + r * tr.n;
            if (t < P) x.put(rw + bitrev(t, logP), keep[r]);
        }
        __syncthreads();
    }
    if constexpr (MODE == DD_FWD || MODE == DD_FWD_REAL) dd_fft_lds<false>(x, W, P, logP, tw);
    else dd_fft_lds<true>(x, W, P, logP, tw);
    if (!act) return;
    for (int t = th.t; t < n_out; t += th.n) {
        const cdd z = x.get(xw + t);
        if constexpr (MODE == DD_FWD_REAL) {
            const cdd c = cconj(x.get(xw + (t == 0 ? 0 : P - t)));
            const cdd a = cadd(z, c), b = csub(z, c);
            ((cdd*)out)[oa + t] = cdd{a.re * 0.5, a.im * 0.5};
            ((cdd*)out)[ob + t] = cdd{b.im * 0.5, -(b.re * 0.5)};
        } else if constexpr (MODE == DD_INV_REAL) {
            ((dd*)out)[oa + t] = z.re;
            ((dd*)out)[ob + t] = z.im;
        } else {
            ((cdd*)out)[oa + t * lo.es] = z;
        }
    }
}

}  // namespace

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

size_t dd_twiddle_elems(const fsa_plan_s* pl) {
    size_t n = 0;
    for (int j = 0; j < pl->d; ++j) n += (size_t)pl->N[j];  // P_j / 2 each
    return n;
}

static const cdd* dd_tw(const fsa_plan_s* pl, int ax) {
    size_t off = 0;
    for (int j = 0; j < ax; ++j) off += (size_t)pl->N[j];
    return (const cdd*)pl->twiddles + off;
}

hipError_t build_tensor_dd(const fsa_plan_s* pl, hipStream_t st) {
    DDGeom g{};
    g.d = pl->d;
    g.eps = pl->kp.eps;
    g.kind = pl->kp.kind;
    for (int j = 0; j < 3; ++j) {
        g.N[j] = j < pl->d ? (int)pl->N[j] : 1;
        g.P[j] = 2 * g.N[j];
        g.L[j] = j < pl->d ? pl->L[j] : 1.0;
    }
    // twiddles of every axis
    size_t off = 0;
    for (int j = 0; j < pl->d; ++j) {
        const int half = (int)pl->N[j];
        hipLaunchKernelGGL(k_dd_twiddle, dim3((half + 255) / 256), dim3(256), 0, st,
                           (cdd*)pl->twiddles + off, 2 * half);
        off += half;
    }
    const long n = (long)pl->tensor_elems;
    dd *a = nullptr, *b = nullptr;
    hipError_t e = hipMallocAsync((void**)&a, sizeof(dd) * n, st);
    if (e == hipSuccess) e = hipMallocAsync((void**)&b, sizeof(dd) * n, st);
    if (e == hipSuccess) {
        const int grid = (int)((n + 255) / 256);
        hipLaunchKernelGGL(k_dd_sample, dim3(grid), dim3(256), 0, st, a, g);
        dd* src = a;
        dd* dst = b;
        for (int ax = 0; ax < pl->d; ++ax) {
            const int P = 2 * g.N[ax];
            const long lines = n / (g.N[ax] + 1);
            const int W = dd_lines(P, lines, device_cus());
            hipLaunchKernelGGL(k_dd_dct, dim3((unsigned)((lines + W - 1) / W)),
                               dim3(W * dd_line_threads(P)), sizeof(cdd) * (size_t)(W * P), st,
                               (const dd*)src, dst, g, ax, lines, W, dd_tw(pl, ax));
            dd* t = src;
            src = dst;
            dst = t;
        }
        hipLaunchKernelGGL(k_dd_finalize, dim3(grid), dim3(256), 0, st, (const dd*)src,
                           (dd*)pl->tensor, g);
        e = hipGetLastError();
    }
    if (a) (void)hipFreeAsync(a, st);
    if (b) (void)hipFreeAsync(b, st);
    return e;
}

// Step k of a double-double evaluation (2d - 1 launches).  X holds bins 0 .. N_last
// of the last axis, C order: (N_0, P_1, N_2 + 1) in 3D, (N_0, N_1 + 1) in 2D (the
// fused pass pads and crops axis 0 in LDS).
hipError_t launch_dd_step(const fsa_plan_s* pl, int k, const void* rho, void* phi, void* ws,
                          hipStream_t st) {
    const int d = pl->d;
    long N[3], P[3];
    int logP[3];
    for (int j = 0; j < d; ++j) {
        N[j] = pl->N[j];
        P[j] = 2 * N[j];
        int lg = 0;
        while ((1L << lg) < P[j]) ++lg;
        logP[j] = lg;
    }
    cdd* X = (cdd*)ws;
    DDConv cv{};
    cv.tensor = (const dd*)pl->tensor;
    cv.d = d;
    for (int j = 0; j < 3; ++j) {
        cv.N[j] = j < d ? (int)N[j] : 0;
        cv.P[j] = j < d ? (int)P[j] : 1;
    }
    const long H = N[d - 1] + 1;  // kept bins of the last axis
    cv.D0 = (int)N[0] + 1;
    cv.D1 = (int)N[1] + 1;
    // pass kinds in order: fwd last (real in), [fwd axis 1], conv axis 0,
    // [inv axis 1], inv last (real out)
    int ax, mode;
    if (d == 3) {
        static const int axes[5] = {2, 1, 0, 1, 2};
        static const int modes[5] = {DD_FWD_REAL, DD_FWD, DD_CONV, DD_INV, DD_INV_REAL};
        ax = axes[k];
        mode = modes[k];
    } else {
        static const int axes[3] = {1, 0, 1};
        static const int modes[3] = {DD_FWD_REAL, DD_CONV, DD_INV_REAL};
        ax = axes[k];
        mode = modes[k];
    }
    const int Pa = (int)P[ax], lg = logP[ax];
    DDLines li{}, lo{};
    long lines = 0;
    int n_in = 0, n_out = 0;
    if (d == 3) {
        switch (mode) {
        case DD_FWD_REAL:  // pairs of rows (i0 < N0, i1 < N1) of rho -> X[i0][i1][p2]
            lines = N[0] * N[1] / 2;
            li = DDLines{N[1] * N[2], N[2], 1, (int)N[1]};
            lo = DDLines{P[1] * H, H, 1, (int)N[1]};
            n_in = (int)N[2];
            n_out = (int)H;
            break;
        case DD_FWD:  // axis 1 at (i0 < N0, p2): X[i0][t][p2]
            lines = N[0] * H;
            li = lo = DDLines{P[1] * H, 1, H, (int)H};
            n_in = (int)N[1];
            n_out = (int)P[1];
            break;
        case DD_CONV:  // axis 0 at (p1, p2): X[t][p1][p2]
            lines = P[1] * H;
            li = lo = DDLines{H, 1, P[1] * H, (int)H};
            n_in = n_out = (int)N[0];
            break;
        case DD_INV:
            lines = N[0] * H;
            li = lo = DDLines{P[1] * H, 1, H, (int)H};
            n_in = (int)P[1];
            n_out = (int)N[1];
            break;
        default:  // DD_INV_REAL: X[i0][i1][t] -> pairs of phi rows
            lines = N[0] * N[1] / 2;
            li = DDLines{P[1] * H, H, 1, (int)N[1]};
            lo = DDLines{N[1] * N[2], N[2], 1, (int)N[1]};
            n_in = (int)H;
            n_out = (int)N[2];
            break;
        }
    } else {
        switch (mode) {
        case DD_FWD_REAL:  // pairs of rows i0 < N0 -> X[i0][p1]
            lines = N[0] / 2;
            li = DDLines{N[1], 0, 1, 1};
            lo = DDLines{H, 0, 1, 1};
            n_in = (int)N[1];
            n_out = (int)H;
            break;
        case DD_CONV:  // axis 0 at p1: X[t][p1]
            lines = H;
            li = lo = DDLines{1, 0, H, 1};
            n_in = n_out = (int)N[0];
            break;
        default:
            lines = N[0] / 2;
            li = DDLines{H, 0, 1, 1};
            lo = DDLines{N[1], 0, 1, 1};
            n_in = (int)H;
            n_out = (int)N[1];
            break;
        }
    }
    if (Pa > kDDMaxP || lines <= 0 || lines > 0x7fffffffL) return hipErrorInvalidValue;
    const int W = dd_lines(Pa, lines, device_cus());
    const dim3 grid((unsigned)((lines + W - 1) / W)), block(W * dd_line_threads(Pa));
    const size_t lds = sizeof(cdd) * (size_t)(W * Pa);
    const cdd* tw = dd_tw(pl, ax);
    const void* src = mode == DD_FWD_REAL ? rho : (const void*)X;
    void* dst = mode == DD_INV_REAL ? phi : (void*)X;
    switch (mode) {
    case DD_FWD_REAL:
        return launch_kernel(k_dd_pass<DD_FWD_REAL>, grid, block, lds, st, src, dst, li, lo, lines, W,
                             Pa, lg, n_in, n_out, tw, cv);
    case DD_FWD:
        return launch_kernel(k_dd_pass<DD_FWD>, grid, block, lds, st, src, dst, li, lo, lines, W,
                             Pa, lg, n_in, n_out, tw, cv);
    case DD_CONV:
        return launch_kernel(k_dd_pass<DD_CONV>, grid, block, lds, st, src, dst, li, lo, lines, W,
                             Pa, lg, n_in, n_out, tw, cv);
    case DD_INV:
        return launch_kernel(k_dd_pass<DD_INV>, grid, block, lds, st, src, dst, li, lo, lines, W,
                             Pa, lg, n_in, n_out, tw, cv);
    default:
        return launch_kernel(k_dd_pass<DD_INV_REAL>, grid, block, lds, st, src, dst, li, lo, lines, W,
                             Pa, lg, n_in, n_out, tw, cv);
    }
}

}  // namespace fsa
