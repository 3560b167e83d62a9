// fsa_spectral.hip -- the source terms of the dipole-dipole potentials.
//
// The 3D DDI is evaluated through the Coulomb kernel with the source
// d_nm rho = (n.grad)(m.grad) rho (Sec. 5.3):
//   Phi = -(m.n) rho - 3 Coulomb(d_nm rho).
// d_nm rho is the spectral derivative of rho on its own N-point grid,
// periodic on the box: a 3D DFT, the product with -(k.n)(k.m),
// k_j = pi q_j / L_j (q_j = i_j for i_j < N_j/2, else i_j - N_j), an inverse
// DFT and the real part.  Five launches on a complex N0 x N1 x (N2/2 + 1)
// array Z (the half spectrum, below) in the first workspace array, leaving
// -3 d_nm rho (real, plan precision) in the second one, where pass A of the
// Coulomb convolution reads it:
//   0  rows of rho (last axis, real) -> forward FFT -> Z
//   1  Z along axis 1, forward
//   2  Z along axis 0: forward, x 3 (k.n)(k.m) / (N0 N1 N2), inverse
//   3  Z along axis 1, inverse
//   4  Z rows, inverse, real part -> -3 d_nm rho
// (3 (k.n)(k.m) / prod N folds the -3, the sign of the derivative and the
// normalisation of the inverse DFT into one factor.)  The quasi-2D DDI
// (Sec. 5.3) convolves S = -(3/2)(d_{n_perp n_perp} - n_3^2 Lap) rho, whose
// transform is (3/2)((k.n_perp)^2 - n_3^2 |k|^2) rho^, in three launches:
// rows forward, axis 0 forward x factor x inverse, rows inverse.  Both
// factors are a scale times a quadratic form f(k) = k^T A k.
//
// rho is real, so Z keeps only the bins 0 <= i_last <= N_last/2 of the row
// transforms (a half spectrum: the other half is the conjugate), and the row
// inverse rebuilds each row from it.  Taking the real part of the full
// inverse DFT of f Z equals the inverse of g Z with g(k) = (f(k) + f(k~))/2,
// k~ the frequency of the bin that pairs with k under conjugation (-q_j,
// except that the Nyquist index N_j/2 pairs with itself); g is even under
// that pairing, so the half spectrum times g is consistent, and the axis-0
// launch multiplies by g.  Each team of a workgroup transforms one line with
// the team FFT.  The row launches read and write their contiguous rows
// directly (k_spec_row); the launches along the strided axes take WT lines
// adjacent in memory (k_spec_col).  Launches 1-3 work in place (each workgroup
// has read all its lines before it writes them back).
#include <hip/hip_runtime.h>

#include "fsa_internal.hpp"

namespace fsa {

namespace {

enum SpecKind { ROW_FWD_REAL = 0, COL_FWD = 1, COL_MUL = 2, COL_INV = 3, ROW_INV_REAL = 4 };

// Lines of a group: 128 bytes of neighbours along the strided axes.
constexpr int spec_lines_per_group(int T, int scr, int csize) {
    int wt = 128 / csize;
    while (wt > 1 && (wt * T > 1024 || wt * scr * csize > 160 * 1024)) wt /= 2;
    return wt;
}

template <typename R, int P>
struct Spec {
    using Ff = Fft<R, P, false>;
    using Fi = Fft<R, P, true>;
    static constexpr int T = Ff::T;
    static constexpr int WT = spec_lines_per_group(T, Ff::SCR, (int)sizeof(cpx<R>));
    static constexpr int THREADS = WT * T;
    static constexpr int LDS = WT * Ff::SCR;
    static_assert(Ff::last_radix() == Fi::first_radix(), "register hand-off");
};

// Lines of one launch.  Rows: row (u, v) starts at u * u_stride + v * v_stride
// (elements), and its other array's row (the launches read or write rows of
// another length) at u * ou_stride + v * ov_stride.  Strided axes: line u (next
// to line u + 1 in memory) of set v starts at u + v * v_stride, its element t
// at + t * es; n_h lines are a row of the half spectrum.  Groups take WT
// consecutive u.
struct SLines {
    int n_u, n_v;
    long u_stride, v_stride, es;
    long ou_stride, ov_stride;
    int n_h;
};

// The derivative factor scale * k^T A k of the axis-0 launch, k = (k0, k1,
// k2) with k0 along the launch's lines, (k1, k2) from the line index (a 2D plan maps its axis 1 to slot 2 and leaves slot 1 empty: c[1] = 0).
struct SMul {
    double c[3];  // pi / L_j
    double A[3][3];
    double scale;
    int N[3];
};

// Launches 0 and 4.  Rows are contiguous: each team reads and writes its own
// row straight from and to global memory (the team's accesses are
// consecutive); Z rows hold the half spectrum, H = P/2 + 1 bins.
template <typename R, int P, int KIND>
__global__ __launch_bounds__((Spec<R, P>::THREADS)) void k_spec_row(
    const void* in, void* out, SLines ln, const cpx<R>* __restrict__ tw) {
    using K = Spec<R, P>;
    using Ff = typename K::Ff;
    using Fi = typename K::Fi;
    using C = cpx<R>;
    constexpr int H = P / 2 + 1;
    __shared__ C lds[K::LDS];
    const int team = team_index<K::T>(), tid = threadIdx.x % K::T;
    const int ntu = (ln.n_u + K::WT - 1) / K::WT;
    const int tu = blockIdx.x % ntu, v = blockIdx.x / ntu;
    const long u = (long)tu * K::WT + team;
    const bool act = u < ln.n_u;
    const long rb = u * ln.u_stride + (long)v * ln.v_stride;
    const long ro = u * ln.ou_stride + (long)v * ln.ov_stride;
    C* sc = lds + team * Ff::SCR;
    C x[Ff::V];
    if constexpr (KIND == ROW_FWD_REAL) {
        Ff::load_first(x, tid, P, [&](int t) {
            return act ? mk(((const R*)in)[rb + t], R(0)) : mk(R(0), R(0));
        });
        Ff::template run_g<false, true>(x, sc, tid, Ff::staged(tw));
        if (act)
            Ff::store_last(x, tid, P, [&](int t, C c) {
                if (t < H) ((C*)out)[ro + t] = c;
            });
    } else {
        // Z[P - t] = conj Z[t] rebuilds the bins above P/2
        Fi::load_first(x, tid, P, [&](int t) {
            if (!act) return mk(R(0), R(0));
            return t < H ? ((const C*)in)[rb + t] : conj(((const C*)in)[rb + P - t]);
        });
        Fi::template run_g<false, true>(x, sc, tid, Fi::staged(tw));
        if (act) Fi::store_last(x, tid, P, [&](int t, C c) { ((R*)out)[ro + t] = c.x; });
    }
}

// Launches 1-3.  Thread tid * WT + w holds operands of line w, so that WT
// neighbours read the 128 bytes of one element of all lines straight into the
// registers of the first stage (and write the last stage's back): all of a
// thread's loads are in flight at once and the only trips through the LDS are
// the transform's own exchanges, where a thread's line is its column w (rows
// of 128 bytes: no bank is met twice).
// At 128^3 FP64 launches 1-3 take 10.3, 14.5 and 10.3 us (34 MB each: 3.3 TB/s);
// with the tile staged through the LDS before and after, its loads one after
// another, they took 17.6, 20.1 and 17.6.  A stage's twiddles are loaded ahead of
// its exchange (Fft::run_x; the five launches 152 -> 143 us at 256^3 FP32, 126 ->
// 121 at 192^3 FP64).
template <class C, int W>
struct Column {  // a team's scratch: entry i of column w of [i][W]
    C* p;
    __device__ __forceinline__ C& operator[](int i) const { return p[i * W]; }
};

template <typename R, int P, int KIND>
__global__ __launch_bounds__((Spec<R, P>::THREADS)) void k_spec_col(
    void* z, SLines ln, const cpx<R>* __restrict__ tw, SMul mul) {
    using K = Spec<R, P>;
    using Ff = typename K::Ff;
    using Fi = typename K::Fi;
    using C = cpx<R>;
    __shared__ C lds[K::LDS];
    const int w = threadIdx.x % K::WT, tid = threadIdx.x / K::WT;
    const Column<C, K::WT> sc{lds + w};
    const int ntu = (ln.n_u + K::WT - 1) / K::WT;
    int tu, v;
    if (ln.n_v > 1) {
        // the dispatcher deals workgroups to the 8 XCDs in turn: the groups of a
        // set go to one of them, whose L2 merges the lines that two groups share
        // (rows of n_h bins are not whole cache lines)
        const int s = blockIdx.x >> 3;
        tu = s % ntu;
        v = s / ntu * 8 + (int)(blockIdx.x & 7);
        if (v >= ln.n_v) return;
    } else {
        tu = blockIdx.x;
        v = 0;
    }
    const int u = tu * K::WT + w;
    const bool act = u < ln.n_u;
    C* const line = (C*)z + (long)v * ln.v_stride + u;
    auto sync = [] {
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0), as Fft::sync_lds
        if constexpr (K::THREADS <= 64) __builtin_amdgcn_wave_barrier();
        else __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    auto load = [&](int t) { return act ? line[t * ln.es] : mk(R(0), R(0)); };
    auto store = [&](int t, C c) {
        if (act) line[t * ln.es] = c;
    };
    C x[Ff::V];
    // the inverse runs the radices in reverse: its first stage has its own layout
    if constexpr (KIND == COL_INV) {
        Fi::load_first(x, tid, P, load);
    } else {
        Ff::load_first(x, tid, P, load);
        Ff::run_x(x, sc, tid, Ff::staged(tw), sync);
    }
    if constexpr (KIND == COL_FWD) {
        Ff::store_last(x, tid, P, store);
        return;
    }
    if constexpr (KIND == COL_MUL) {
        // line u = i1 n_h + i2 along axis 0; the register holds output i0.
        // g = (f(k) + f(k~)) / 2 with f = a k0^2 + b k0 + c along the line
        const int i1 = u / ln.n_h, i2 = u - i1 * ln.n_h;
        auto qv = [](int i, int n) { return i < n / 2 ? i : i - n; };
        auto qp = [&](int i, int n) { return qv(i == 0 ? 0 : n - i, n); };  // the paired bin
        const double k1 = mul.c[1] * qv(i1, mul.N[1]), k2 = mul.c[2] * qv(i2, mul.N[2]);
        const double p1 = mul.c[1] * qp(i1, mul.N[1]), p2 = mul.c[2] * qp(i2, mul.N[2]);
        const double ha = 0.5 * mul.scale * mul.A[0][0];
        const double hb = mul.scale * (mul.A[0][1] * k1 + mul.A[0][2] * k2);
        const double hbp = mul.scale * (mul.A[0][1] * p1 + mul.A[0][2] * p2);
        const double hc = 0.5 * mul.scale *
                          (mul.A[1][1] * (k1 * k1 + p1 * p1) +
                           2.0 * mul.A[1][2] * (k1 * k2 + p1 * p2) +
                           mul.A[2][2] * (k2 * k2 + p2 * p2));
        Ff::for_each_last(x, tid, [&](int i0, C& c) {
            const double k0 = mul.c[0] * qv(i0, mul.N[0]), p0 = mul.c[0] * qp(i0, mul.N[0]);
            c = scale(c, (R)(ha * (k0 * k0 + p0 * p0) + hb * k0 + hbp * p0 + hc));
        });
    }
    Fi::run_x(x, sc, tid, Fi::staged(tw), sync);
    Fi::store_last(x, tid, P, store);
}

template <typename R, int KIND>
hipError_t go(int P, const void* in, void* out, SLines ln, const void* tw, const SMul& mul,
              hipStream_t st) {
    switch (P) {
#define FSA_SPEC_CASE(p)                                                                        \
    case p: {                                                                                   \
        using K = Spec<R, p>;                                                                   \
        const int ntu = (ln.n_u + K::WT - 1) / K::WT;                                           \
        if constexpr (KIND == ROW_FWD_REAL || KIND == ROW_INV_REAL)                             \
            return launch_kernel(k_spec_row<R, p, KIND>, dim3(ntu * ln.n_v), dim3(K::THREADS),  \
                                 0, st, in, out, ln, (const cpx<R>*)tw);                        \
        else                                                                                    \
            return launch_kernel(k_spec_col<R, p, KIND>,                                        \
                                 dim3(ln.n_v > 1 ? ntu * ((ln.n_v + 7) / 8 * 8) : ntu),         \
                                 dim3(K::THREADS), 0, st, out, ln, (const cpx<R>*)tw, mul);     \
    }
        FSA_SPEC_CASE(8) FSA_SPEC_CASE(12) FSA_SPEC_CASE(16) FSA_SPEC_CASE(24) FSA_SPEC_CASE(32)
        FSA_SPEC_CASE(48) FSA_SPEC_CASE(64) FSA_SPEC_CASE(96) FSA_SPEC_CASE(128)
        FSA_SPEC_CASE(192) FSA_SPEC_CASE(256) FSA_SPEC_CASE(384) FSA_SPEC_CASE(512)
        FSA_SPEC_CASE(768) FSA_SPEC_CASE(1024) FSA_SPEC_CASE(1536) FSA_SPEC_CASE(2048)
#undef FSA_SPEC_CASE
    }
    return hipErrorInvalidValue;
}

constexpr double kPi = 3.14159265358979323846264338327950288;

// quasi-2D DDI: rows, axis 0 with the factor, rows inverse
template <typename R>
hipError_t step_2d(const fsa_plan_s* pl, int s, const void* rho, void* z, void* dst,
                   hipStream_t st) {
    const long N0 = pl->N[0], N1 = pl->N[1];
    const char* tw = (const char*)pl->twiddles;
    const void* tw0 = tw + pl->tw_off_n0 * pl->csize;
    const void* tw1 = tw + pl->tw_off_m * pl->csize;  // length N1
    SMul mul{};
    // 2D axes 0, 1 in slots 0, 2; (3/2)((k.n_perp)^2 - n_3^2 |k|^2) / (N0 N1)
    const double n0 = pl->dn[0], n1 = pl->dn[1], n3sq = pl->dn[2] * pl->dn[2];
    mul.c[0] = kPi / pl->L[0];
    mul.c[2] = kPi / pl->L[1];
    mul.N[0] = (int)N0;
    mul.N[1] = 1;
    mul.N[2] = (int)N1;
    mul.A[0][0] = n0 * n0 - n3sq;
    mul.A[2][2] = n1 * n1 - n3sq;
    mul.A[0][2] = mul.A[2][0] = n0 * n1;
    mul.scale = 1.5 / ((double)N0 * (double)N1);
    const long H1 = N1 / 2 + 1;  // half spectrum of the rows
    const SLines fwd{(int)N0, 1, N1, 0, 1, H1, 0, 0};  // rho rows -> Z rows
    const SLines inv{(int)N0, 1, H1, 0, 1, N1, 0, 0};  // Z rows -> source rows
    const SLines ax0{(int)H1, 1, 1, 0, H1, 0, 0, (int)H1};
    switch (s) {
    case 0: return go<R, ROW_FWD_REAL>((int)N1, rho, z, fwd, tw1, mul, st);
    case 1: return go<R, COL_MUL>((int)N0, z, z, ax0, tw0, mul, st);
    case 2: return go<R, ROW_INV_REAL>((int)N1, z, dst, inv, tw1, mul, st);
    }
    return hipErrorInvalidValue;
}

template <typename R>
hipError_t step_t(const fsa_plan_s* pl, int s, const void* rho, void* z, void* dst,
                  hipStream_t st) {
    if (pl->d == 2) return step_2d<R>(pl, s, rho, z, dst, st);
    const long N0 = pl->N[0], N1 = pl->N[1], N2 = pl->N[2];
    const char* tw = (const char*)pl->twiddles;
    const void* tw0 = tw + pl->tw_off_n0 * pl->csize;
    const void* tw1 = tw + pl->tw_off_n1 * pl->csize;
    const void* tw2 = tw + pl->tw_off_m * pl->csize;  // length N2
    SMul mul{};
    double prodN = 1.0;
    for (int j = 0; j < 3; ++j) {
        mul.c[j] = kPi / pl->L[j];
        mul.N[j] = (int)pl->N[j];
        prodN *= (double)pl->N[j];
    }
    // (k.n)(k.m) = k^T A k with A the symmetric part of n m^T
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b)
            mul.A[a][b] = 0.5 * (pl->dn[a] * pl->dm[b] + pl->dm[a] * pl->dn[b]);
    mul.scale = 3.0 / prodN;
    // Z is N0 x N1 x H2, the half spectrum of the rows
    const long H2 = N2 / 2 + 1;
    // rows: lines along axis 2, groups of consecutive rows
    const SLines fwd{(int)N1, (int)N0, N2, N1 * N2, 1, H2, N1 * H2, 0};  // rho -> Z
    const SLines inv{(int)N1, (int)N0, H2, N1 * H2, 1, N2, N1 * N2, 0};  // Z -> source
    // axis 1: lines at fixed (i0, i2), groups of consecutive i2
    const SLines ax1{(int)H2, (int)N0, 1, N1 * H2, H2, 0, 0, (int)H2};
    // axis 0: lines at fixed (i1, i2), all N1 H2 of them neighbours
    const SLines ax0{(int)(N1 * H2), 1, 1, 0, N1 * H2, 0, 0, (int)H2};
    switch (s) {
    case 0: return go<R, ROW_FWD_REAL>((int)N2, rho, z, fwd, tw2, mul, st);
    case 1: return go<R, COL_FWD>((int)N1, z, z, ax1, tw1, mul, st);
    case 2: return go<R, COL_MUL>((int)N0, z, z, ax0, tw0, mul, st);
    case 3: return go<R, COL_INV>((int)N1, z, z, ax1, tw1, mul, st);
    case 4: return go<R, ROW_INV_REAL>((int)N2, z, dst, inv, tw2, mul, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t spectral_step(const fsa_plan_s* pl, int s, const void* rho, void* z, void* dst,
                         hipStream_t st) {
    return pl->prec == FSA_F32 ? step_t<float>(pl, s, rho, z, dst, st)
                               : step_t<double>(pl, s, rho, z, dst, st);
}

}  // namespace fsa
