// fsa_plane.hpp -- passes B, C and D of a 3D evaluation on small planes, in one
// launch (gfx950).
//
// Passes B, C and D exchange, for each bin p2, the padded plane Y[p1][i0] of
// P1 x N0 complex values.  A small plane (up to 4096 values) fits a workgroup's
// LDS, and one workgroup takes it through all three passes: the plane is read
// from X1 and written back to X1 once, and one launch takes the place of three,
// each of which is one item's latency on grids this small (3.4-4.2 us at 32^3).
//
// The values live in registers while the teams transform (their exchange scratch
// then owns the LDS), and go through the LDS as one tile between the passes.
// Each transform is the same team FFT, on the same radices, as the pass of its
// own launch computes, so the results are bitwise the same.
//
// The line at N0 N1 <= 2048 (axes of at most 128, the lengths it is compiled for): a
// plane is one workgroup's work, whose arithmetic grows with the plane and cannot
// spread over the device when the planes are fewer than the CUs.  Evaluations in us,
// separate / in one launch: 32^3 FP64 20.4 / 14.7, 32 x 64 x 64 20.1 / 16.3 FP32 and
// 22.1 / 18.8 FP64, 64 x 32 x 256 32.8 / 24.2 and 35.9 / 32.9; past the line 48 x 48 x 256
// FP32 37.2 / 38.1, 64 x 64 x 256 FP64 56.3 / 62.1, 32 x 128 x 64 FP64 31.1 / 39.3.  Longer
// last axes only add planes: 32 x 64 x 2048 113 / 87 (FP32) and 205 / 158 (FP64).
// Exceptions: FEW_SLOW.
#pragma once

#include "fsa_fft.hpp"
#include "fsa_jobs.hpp"
#include "fsa_passes.hpp"

namespace fsa {

constexpr int kPlaneValues = 2 * 2048;  // N0 P1

template <typename R, int P1, int P0>
struct Plane {
    using C = cpx<R>;
    using F1 = Fft<R, P1, false>;  // pass B
    using I1 = Fft<R, P1, true>;   // pass D
    using F0 = Fft<R, P0, false>;  // pass C
    using I0 = Fft<R, P0, true>;
    static constexpr int N1 = P1 / 2, N0 = P0 / 2;
    static constexpr int T1 = F1::T, T0 = F0::T;
    // threads: a power of two from 64, at least 8 values of the plane each beyond 64
    // (with 16 values each 32^3 FP32 takes 15.2 us instead of 13.5, with 4 14.0)
    static constexpr int VPT = 8;
    static constexpr int threads() {
        int t = 64;
        while (t < 1024 && 2 * t * VPT <= N0 * P1) t *= 2;
        return t;
    }
    static constexpr int THREADS = threads();
    static constexpr bool WHOLE = THREADS % T1 == 0 && THREADS % T0 == 0;  // teams fill it
    static constexpr int G1 = THREADS / T1, G0 = THREADS / T0;  // teams
    static constexpr int RB = cdiv(N0, G1), RC = cdiv(P1, G0);  // lines per team
    // row pitch of the tile: lanes along p1 (a team's in passes B and D) and the
    // teams beside it fall on different banks
    static constexpr int TS = N0 + cmax(1, (sizeof(R) == 4 ? 32 : 16) / T1);
    static constexpr int LDS = cmax(P1 * TS, cmax(G1 * F1::SCR, G0 * F0::SCR));
    static constexpr bool FITS =
        N0 * P1 <= kPlaneValues && LDS * (int)sizeof(C) <= kMaxLds && WHOLE;
    // FP32 keeps the twiddles of both axes in registers
    static constexpr bool REG = sizeof(R) == 4;
    static_assert(F0::last_radix() == I0::first_radix(), "register hand-off");
    // operands a thread takes through the stages of pass B and of pass C one after
    // another (pass D and the inverse of C repeat them)
    static constexpr int CHAIN = RB * F1::V * F1::S + RC * F0::V * F0::S;
    // Planes whose workgroup is slower than the three launches while few of them run
    // side by side: in FP64, long chains along long axes.  One launch / apart, us: 12 x
    // 96 at N_2 = 8, 32, 64, 96 22.5 / 20.3, 23.9 / 21.0, 24.2 / 22.6, 29.8 / 30.6; 96 x 16
    // 20.3 / 20.0, 21.6 / 20.0, 22.0 / 21.9, 27.7 / 31; but 24 x 64, as long a chain, at 8,
    // 16, 32, 64 20.1 / 20.0, 21.3 / 20.5, 21.5 / 21.1, 21.9 / 23.1.  The others gain in a
    // stream at every N_2 (64 x 32 at N_2 = 8: 18.2 / 19.6), where five launches take 20
    // us at least; replayed from a graph, where that is 16, some lose up to N_2 = 32
    // (64 x 32, 128 x 16, 96 x 8 FP64 at 8: 17.8 / 16.0, 18.4 / 16.2, 17.5 / 15.9): a
    // grid's schedule in the tuning table says so ("one_launch": 0).
    static constexpr bool FEW_SLOW =
        sizeof(R) == 8 && N0 * N1 > 1024 && CHAIN >= 120 && cmax(P0, P1) >= 192;
    static constexpr int FEW = 96;
};

template <typename R, int P1, int P0>
__global__ __launch_bounds__((Plane<R, P1, P0>::THREADS)) void k_plane(
    JobPlane jb, const cpx<R>* __restrict__ tw1, const cpx<R>* __restrict__ tw0) {
    using K = Plane<R, P1, P0>;
    using F1 = typename K::F1;
    using I1 = typename K::I1;
    using F0 = typename K::F0;
    using I0 = typename K::I0;
    using C = cpx<R>;
    constexpr int N1 = K::N1, N0 = K::N0;
    __shared__ C lds[K::LDS];
    const int p2 = blockIdx.x;
    C* const x1 = (C*)jb.x1 + (size_t)p2 * N1;  // row i0 at i0 * H * N1
    const size_t pitch = (size_t)jb.H * N1;
    // every phase takes a fresh copy of the thread index (fresh_lane): kept for all
    // of them, the addresses of three transforms cost half the registers

    // pass B: line i0 = team1 + r G1
    {
        const int th = opaque(threadIdx.x), team1 = team_of<K::T1>(th), tid1 = th % K::T1;
        C* const scr1 = lds + team1 * F1::SCR;
        C v[K::RB][F1::V];
#pragma unroll
        for (int r = 0; r < K::RB; ++r) {
            const int i0 = team1 + r * K::G1;
            F1::load_first(v[r], tid1, N1, [&](int i) {
                return i0 < N0 ? x1[i0 * pitch + i] : mk(R(0), R(0));
            });
        }
        C w[K::REG ? F1::NTW : 1];
        if constexpr (K::REG) F1::load_tw_st(w, tid1, F1::staged(tw1));
#pragma unroll
        for (int r = 0; r < K::RB; ++r) {
            if constexpr (K::REG) F1::template run_r<true>(v[r], scr1, tid1, w);
            else F1::template run_g<true>(v[r], scr1, tid1, F1::staged(tw1));
        }
        sync_wg_lds();
#pragma unroll
        for (int r = 0; r < K::RB; ++r) {
            const int i0 = team1 + r * K::G1;
            if (i0 < N0)
                F1::store_last(v[r], tid1, P1, [&](int p1, C c) { lds[p1 * K::TS + i0] = c; });
        }
    }
    sync_wg_lds();

    // pass C: pencil p1 = team0 + r G0; u keeps its non-zero half
    {
        const int th = opaque(threadIdx.x), team0 = team_of<K::T0>(th), tid_ = th % K::T0;
        C* const scr0 = lds + team0 * F0::SCR;
        constexpr int NH = F0::first_nbt() * (F0::first_radix() / 2);
        constexpr int NK = I0::nbt(I0::S - 1) * (I0::last_radix() / 2);
        C u[K::RC][cmax(NH, NK)];
#pragma unroll
        for (int r = 0; r < K::RC; ++r) {
            const int p1 = team0 + r * K::G0;
#pragma unroll
            for (int b = 0; b < F0::first_nbt(); ++b)
#pragma unroll
                for (int q = 0; q < F0::first_radix() / 2; ++q) {
                    const int i = F0::first_index(tid_, b, q);
                    u[r][b * (F0::first_radix() / 2) + q] =
                        (i >= 0 && p1 < P1) ? lds[p1 * K::TS + i] : mk(R(0), R(0));
                }
        }
        C wf[K::REG ? F0::NTW : 1], wi[K::REG && !F0::palindromic() ? I0::NTW : 1];
        if constexpr (K::REG) F0::load_tw_st(wf, tid_, F0::staged(tw0));
        if constexpr (K::REG && !F0::palindromic()) I0::load_tw_st(wi, tid_, I0::staged(tw0));
        sync_wg_lds();
#pragma unroll
        for (int r = 0; r < K::RC; ++r) {
            const int tid0 = opaque(tid_);
            const int p1 = team0 + r * K::G0 < P1 ? team0 + r * K::G0 : 0;
            const int a1 = p1 <= N1 ? p1 : P1 - p1;
            const R* trow = (const R*)jb.tensor + ((size_t)p2 * (N1 + 1) + a1) * (N0 + 1);
            C v[F0::V];
#pragma unroll
            for (int b = 0; b < F0::first_nbt(); ++b)
#pragma unroll
                for (int q = 0; q < F0::first_radix(); ++q)
                    v[b * F0::first_radix() + q] =
                        q < F0::first_radix() / 2 ? u[r][b * (F0::first_radix() / 2) + q]
                                                  : mk(R(0), R(0));
            R tv[F0::V];
            {
                int i = 0;
                F0::for_each_last(v, tid0, [&](int p0, C&) { tv[i++] = trow[p0 <= N0 ? p0 : P0 - p0]; });
            }
            if constexpr (K::REG) F0::template run_r<true>(v, scr0, tid0, wf);
            else F0::template run_g<true>(v, scr0, tid0, F0::staged(tw0));
            {
                int i = 0;
                F0::for_each_last(v, tid0, [&](int, C& c) { c = scale(c, tv[i++]); });
            }
            if constexpr (K::REG && F0::palindromic()) I0::run_r(v, scr0, tid0, wf);
            else if constexpr (K::REG) I0::run_r(v, scr0, tid0, wi);
            else if constexpr (F0::palindromic()) I0::run_g(v, scr0, tid0, F0::staged(tw0));
            else I0::run_g(v, scr0, tid0, I0::staged(tw0));
            {
                int i = 0;
                I0::store_last_slots(v, tid0, [&](C c) { u[r][i++] = c; });
            }
        }
        sync_wg_lds();
#pragma unroll
        for (int r = 0; r < K::RC; ++r) {
            const int p1 = team0 + r * K::G0;
            if (p1 < P1) {
                int i = 0;
                I0::last_slots(tid_, [&](int i0, bool ok) {
                    if (ok) lds[p1 * K::TS + i0] = u[r][i];
                    ++i;
                });
            }
        }
    }
    sync_wg_lds();

    // pass D
    {
        const int th = opaque(threadIdx.x), team1 = team_of<K::T1>(th), tid1 = th % K::T1;
        C* const scr1 = lds + team1 * F1::SCR;
        C v[K::RB][I1::V];
#pragma unroll
        for (int r = 0; r < K::RB; ++r) {
            const int i0 = team1 + r * K::G1;
            I1::load_first(v[r], tid1, P1, [&](int p1) {
                return i0 < N0 ? lds[p1 * K::TS + i0] : mk(R(0), R(0));
            });
        }
        C w[K::REG && !F1::palindromic() ? I1::NTW : K::REG ? F1::NTW : 1];
        if constexpr (K::REG) {
            if constexpr (F1::palindromic()) F1::load_tw_st(w, tid1, F1::staged(tw1));
            else I1::load_tw_st(w, tid1, I1::staged(tw1));
        }
        sync_wg_lds();
#pragma unroll
        for (int r = 0; r < K::RB; ++r) {
            if constexpr (K::REG) I1::run_r(v[r], scr1, tid1, w);
            else if constexpr (F1::palindromic()) I1::run_g(v[r], scr1, tid1, F1::staged(tw1));
            else I1::run_g(v[r], scr1, tid1, I1::staged(tw1));
            const int i0 = team1 + r * K::G1;
            if (i0 < N0)
                I1::store_last(v[r], tid1, N1, [&](int i1, C c) { x1[i0 * pitch + i1] = c; });
        }
    }
}

}  // namespace fsa
