// The transform as the kernels run it where twiddles are loaded ahead of an exchange:
// each stage's twiddles from the staged table into an array of their own
// (load_tw_stage), the exchange through the padded scratch, the butterflies from that
// array (compute_w); thread by thread, every supported length, both radix families
// and directions.  Against a direct sum, relative to the largest output; prints "ok".
#include <cmath>
#include <cstdio>
#include <vector>

#include "../../paper_2504_19410_amd/csrc/fsa_fft.hpp"

using namespace fsa;

static int g_bad = 0;
constexpr double kPi = 3.14159265358979323846264338327950288;

// thread t's registers
template <class F>
static typename F::C (&regs(std::vector<typename F::C>& v, int t))[F::V] {
    return *reinterpret_cast<typename F::C(*)[F::V]>(&v[(size_t)t * F::V]);
}

template <class F, int s>
static void stages(std::vector<typename F::C>& v, std::vector<typename F::C>& scr,
                   const typename F::C* st) {
    using C = typename F::C;
    if constexpr (s < F::S) {
        for (int t = 0; t < F::T; ++t)
            F::template store<s - 1>(regs<F>(v, t), scr.data(), t);
        for (int t = 0; t < F::T; ++t) {
            C w[F::tw_count(s)];
            F::template load_tw_stage<s, 0>(w, t, st);
            F::template load<s>(regs<F>(v, t), scr.data(), t);
            F::template compute_w<s, 0>(regs<F>(v, t), t, w);
        }
        stages<F, s + 1>(v, scr, st);
    }
}

template <int P, bool INV, int ALT>
static void check_one() {
    using F = Fft<double, P, INV, ALT>;
    using C = cpx<double>;
    const double nan = std::nan("");
    std::vector<C> tw((size_t)kTwTables * P, mk(nan, nan)), root(P), in(P), out(P, mk(nan, nan));
    for (int m = 0; m < P; ++m) root[m] = mk(std::cos(2 * kPi * m / P), -std::sin(2 * kPi * m / P));
    const FftPlan p = make_fft_plan(P, ALT);
    int r[8] = {};
    for (int s = 0; s < p.n; ++s) r[s] = p.r[INV ? p.n - 1 - s : s];
    for (int e = 0; e < P; ++e) {
        const int m = staged_index(r, p.n, P, e);
        if (m >= 0) tw[(size_t)staged_table(ALT, INV) * P + e] = root[m];
    }
    for (int i = 0; i < P; ++i) in[i] = mk(std::sin(1.0 + 3.0 * i), std::cos(2.0 + 0.7 * i * i));
    std::vector<C> v((size_t)F::T * F::V, mk(0.0, 0.0)), scr(F::SCR, mk(nan, nan));
    const C* st = F::staged(tw.data());
    for (int t = 0; t < F::T; ++t) {
        F::load_first(regs<F>(v, t), t, P, [&](int i) { return in[i]; });
        F::template compute_st<0>(regs<F>(v, t), t, st);
    }
    stages<F, 1>(v, scr, st);
    for (int t = 0; t < F::T; ++t)
        F::store_last(regs<F>(v, t), t, P, [&](int i, C c) { out[i] = c; });
    double err = 0.0, top = 0.0;
    for (int k = 0; k < P; ++k) {
        double x = 0.0, y = 0.0;
        for (int i = 0; i < P; ++i) {
            const C w = root[(long)i * k % P];
            const double c = w.x, s = INV ? -w.y : w.y;
            x += in[i].x * c - in[i].y * s;
            y += in[i].x * s + in[i].y * c;
        }
        const double e = std::hypot(out[k].x - x, out[k].y - y), a = std::hypot(x, y);
        if (!(e <= err)) err = e;  // keeps a NaN
        if (a > top) top = a;
    }
    // the direct sum's own rounding, P terms of size one, dominates
    if (!(err <= 2.3e-16 * P * top)) {
        ++g_bad;
        std::printf("P %d inv %d family %d: %g of %g\n", P, INV, ALT, err, top);
    }
}

template <int P>
static void check_length() {
    check_one<P, false, 0>();
    check_one<P, true, 0>();
    check_one<P, false, 1>();
    check_one<P, true, 1>();
}

int main() {
#define L(p) check_length<p>();
    L(8) L(12) L(16) L(24) L(32) L(48) L(64) L(96) L(128) L(192) L(256) L(384) L(512) L(768)
    L(1024) L(1536) L(2048) L(3072) L(4096)
    std::printf(g_bad ? "%d wrong\n" : "ok\n", g_bad);
    return g_bad != 0;
}
