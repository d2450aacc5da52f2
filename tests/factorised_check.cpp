// Host build of the generated contraction programs (device qualifiers and the
// scheduling barrier defined away): the factorised program of a level, in four
// and in eight clusters, against the expanded program of the same level, on
// random moments and xi.  Built and run by tests/test_factorised_program.py.
#include <cmath>
#include <cstdio>
#include <random>
#define __device__
#define __forceinline__ inline
#define MTP_FACT_SCHED()
using std::fma;
inline double cmul(double a, double b) { return a * b; }
inline double cfma(double a, double b, double c) { return fma(a, b, c); }
namespace A {
template <int L> struct Level;
#include LEVEL_A
}
namespace B {
template <int L> struct Level;
#include LEVEL_B
}
using LA = A::Level<LV>;
using LB = B::Level<LV>;
constexpr int NC = LA::NC, NL = LA::NLIN, NP = LB::NPROD;
template <int NW, int P> void clusters(const double *M, const double *p, const double *xi, double *B, double *sum) {
    if constexpr (P < NW) {
        double d[NW == 4 ? LB::FMAX4 : LB::FMAX8];
        if constexpr (NW == 4) LB::template fact4<P, true>(M, p, xi, B, d);
        else LB::template fact8<P, true>(M, p, xi, B, d);
        const int n = NW == 4 ? LB::fncomp4[P] : LB::fncomp8[P];
        for (int k = 0; k < n; ++k) sum[NW == 4 ? LB::fcomp4[P][k] : LB::fcomp8[P][k]] += d[k];
        clusters<NW, P + 1>(M, p, xi, B, sum);
    }
}
template <int NW> double check(std::mt19937_64 &rng) {
    std::normal_distribution<double> nd(0.0, 1.0);
    double worst = 0;
    for (int trial = 0; trial < 20; ++trial) {
        double M[NC], xi[NL], Ba[NL], dMa[NC], Va;
        for (auto &v : M) v = nd(rng);
        for (auto &v : xi) v = nd(rng);
        LA::template contract<double, true>(M, (const double *)xi, (double *)Ba, dMa, Va);
        double gl[LB::NLOW + 1], p[NP], dz[LB::NLOW + 1], d[LB::NLOWC + 1], sum[NC + NP] = {}, Bb[NL], Vb;
        for (auto &v : Bb) v = NAN;   // every B_alpha must be written
        p[0] = 1.0;
        LB::low_values((const double *)M, gl, p);
        LB::template low_functions<true>(gl, (const double *)xi, (double *)Bb, dz, Vb);
        clusters<NW, 0>(M, p, xi, Bb, sum);
        LB::low_coupling(gl, p, (const double *)(sum + NC), dz, Vb);
        LB::low_reverse((const double *)M, (const double *)dz, d);
        for (int k = 0; k < LB::NLOWC; ++k) sum[LB::low_comp[k]] += d[k];
        double sc = std::fabs(Va), e = std::fabs(Va - Vb), sd = 0, ed = 0;
        for (int k = 0; k < NL; ++k) {
            sc = std::fmax(sc, std::fabs(Ba[k]));
            e = std::isnan(Bb[k]) ? INFINITY : std::fmax(e, std::fabs(Ba[k] - Bb[k]));
        }
        for (int k = 0; k < NC; ++k) {
            sd = std::fmax(sd, std::fabs(dMa[k]));
            ed = std::fmax(ed, std::fabs(dMa[k] - sum[k]));
        }
        worst = std::fmax(worst, std::fmax(e / sc, ed / sd));
    }
    return worst;
}
int main() {
    std::mt19937_64 rng(5);
    const double w4 = check<4>(rng), w8 = check<8>(rng);
    std::printf("level %d: worst relative difference %.3g (four clusters), %.3g (eight)\n", LV, w4, w8);
    return w4 < 1e-12 && w8 < 1e-12 ? 0 : 1;
}
