// The staged twiddle tables against the plain one: every supported length, both
// radix families and directions.  Prints "ok" if every stage reads the same
// values, bit for bit, through both.
#include <cmath>
#include <cstdio>
#include <cstring>
#include <vector>

#include "../../paper_2504_19410_amd/csrc/fsa_fft.hpp"

using namespace fsa;

static int g_bad = 0;

// stage s and the ones after it on two copies of the operands
template <class F, int s>
static void stage(typename F::C (&v)[F::V], typename F::C (&w)[F::V], int t,
                  const typename F::C* tw) {
    if constexpr (s < F::S) {
        F::template compute<s>(v, t, tw);
        F::template compute_st<s>(w, t, F::staged(tw));
        stage<F, s + 1>(v, w, t, tw);
    }
}

template <typename R, int P, bool INV, int ALT>
static void check_one() {
    using F = Fft<R, P, INV, ALT>;
    using C = cpx<R>;
    constexpr double kPi = 3.14159265358979323846264338327950288;
    std::vector<C> tw((size_t)kTwTables * P, mk(R(NAN), R(NAN)));
    for (int m = 0; m < P; ++m)
        tw[m] = mk((R)std::cos(2.0 * kPi * m / P), (R)-std::sin(2.0 * kPi * m / P));
    for (int alt = 0; alt < 2; ++alt)
        for (int inv = 0; inv < 2; ++inv) {
            const FftPlan p = make_fft_plan(P, alt);
            int r[8] = {};
            for (int s = 0; s < p.n; ++s) r[s] = p.r[inv ? p.n - 1 - s : s];
            for (int e = 0; e < P; ++e) {
                const int m = staged_index(r, p.n, P, e);
                if (m >= P) ++g_bad;
                else if (m >= 0) tw[(size_t)staged_table(alt, inv != 0) * P + e] = tw[m];
            }
        }
    for (int t = 0; t < F::T; ++t) {
        C a[F::NTW], b[F::NTW];
        std::memset((void*)a, 0, sizeof a);
        std::memset((void*)b, 0, sizeof b);
        F::load_tw(a, t, tw.data());
        F::load_tw_st(b, t, F::staged(tw.data()));
        // butterfly slots beyond NB hold entry k = 0 in both
        if (std::memcmp((const void*)a, (const void*)b, sizeof a) != 0) ++g_bad;
        C v[F::V], w[F::V];
        for (int i = 0; i < F::V; ++i) v[i] = w[i] = mk(R(0.25 + i), R(1.5 - i));
        stage<F, 1>(v, w, t, tw.data());
        if (std::memcmp((const void*)v, (const void*)w, sizeof v) != 0) ++g_bad;
    }
}

template <typename R, int P>
static void check_length() {
    check_one<R, P, false, 0>();
    check_one<R, P, true, 0>();
    check_one<R, P, false, 1>();
    check_one<R, P, true, 1>();
}

int main() {
#define L(p) check_length<float, p>(), check_length<double, p>();
    L(8) L(12) L(16) L(24) L(32) L(48) L(64) L(96) L(128) L(192) L(256) L(384) L(512) L(768)
    L(1024) L(1536) L(2048) L(3072) L(4096)
    if (g_bad) std::printf("%d differences\n", g_bad);
    else std::printf("ok\n");
    return g_bad != 0;
}
