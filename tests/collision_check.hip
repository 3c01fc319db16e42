// Host run of the kernels' own ES-BGK solve (built and run by
// tests/test_collision_check.py; no GPU is involved): the device functions of
// quasi_eq.hpp are compiled for the host as they stand, a wave being one lane.
//
// Usage: collision_check qe D f32|f32s|f64 Pr tau cells seed spread
// Random strictly positive cells g_i = w_i exp(spread n_i), n_i normal; for each
// the quasi-equilibrium as the step forms it, and the factored Newton solve
// (qe_newton) in the step's type and in double.  Prints, on one line:
//   cells accepted, accepted with a non-finite d, refused though the Newton
//   solve in the same type accepts them, and the largest error of d, relative
//   to the cell's density, of the step and of that Newton solve.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>

// what the device functions use, for the host
#undef __device__
#define __device__ __attribute__((host)) __attribute__((device))
#define __ballot(p) ((p) ? 1ull : 0ull)
#define __builtin_amdgcn_rcpf(v) (1.0f / (v))
#define __builtin_amdgcn_rcp(v) (1.0 / (v))
#define __builtin_amdgcn_sqrtf(v) sqrtf(v)
#define __builtin_amdgcn_sched_barrier(m) ((void)0)
#define __builtin_amdgcn_readfirstlane(v) (v)
#define asm(...)
#include "../paper_2203_12946_amd/csrc/lattice.hpp"
#include "../paper_2203_12946_amd/csrc/quasi_eq.hpp"

using namespace eselbm;

// one cell as the step sees it: stored values p, d = feq - g, rho, u
template <int D, typename T, typename E, bool SH>
struct Cell {
    T p[Lat<D>::Q], d[Lat<D>::Q];
    E rho, u[3];
    explicit Cell(const double (&g)[Lat<D>::Q])
    {
        E r = E(0), j[3] = {E(0), E(0), E(0)};
        for (int i = 0; i < Lat<D>::Q; ++i) {
            p[i] = SH ? T(g[i] - Lat<D>::w(i)) : T(g[i]);
            const E dev = SH ? E(p[i]) : E(p[i]) - E(Lat<D>::w(i));
            r += dev;
            for (int a = 0; a < D; ++a) j[a] += E(Lat<D>::c(i, a)) * dev;
        }
        rho = E(1) + r;
        for (int a = 0; a < 3; ++a) u[a] = j[a] / rho;
        const Equilibrium<D, E> eq(r, u);
        for (int i = 0; i < Lat<D>::Q; ++i) d[i] = T(eq.dev(i) - (SH ? E(p[i]) : E(p[i]) - E(Lat<D>::w(i))));
        conserve_moments<D, T>(d);
    }
};

// f^QE - g of a cell by the factored Newton solve alone
template <int D, typename T, typename E, bool SH>
static bool newton(const Cell<D, T, E, SH> &c, E cpr, double (&d)[Lat<D>::Q])
{
    constexpr int Q = Lat<D>::Q, K = QEBasis<D>::K;
    auto fe = [&](int i) { return E(gval<D, T, SH>(i, c.p)) + E(c.d[i]); };
    E md[Q], tgt[K], delta[K];
    for (int i = 0; i < Q; ++i) md[i] = E(c.d[i]);
    contract_rows<D, E>(md);
    for (int k = 0; k < K; ++k) tgt[k] = k <= D ? E(0) : -cpr * md[QEBasis<D>::m1(k)];
    int it = 0;
    if (!qe_newton<D, E>(fe, tgt, delta, it)) return false;
    T dn[Q];
    for (int i = 0; i < Q; ++i) dn[i] = c.d[i];
    qe_excess<D, E>(delta, fe, [&](int i, E r) { dn[i] = T(E(dn[i]) + r); });
    conserve_moments<D, T>(dn);
    for (int i = 0; i < Q; ++i) d[i] = dn[i];
    return true;
}

template <int D, typename T, typename E, bool SH>
static int run_qe(double pr, double tau, int cells, unsigned seed, double spread)
{
    constexpr int Q = Lat<D>::Q;
    const double cpr = (1.0 - 1.0 / pr) / (1.0 + 1.0 / (2.0 * tau * pr));
    std::mt19937_64 rng(seed);
    std::normal_distribution<double> normal;
    int accepted = 0, nonfinite = 0, refused = 0;
    double err = 0.0, err_newton = 0.0;
    for (int n = 0; n < cells; ++n) {
        double g[Q], ref[Q], own[Q];
        for (int i = 0; i < Q; ++i) g[i] = Lat<D>::w(i) * std::exp(spread * normal(rng));
        Cell<D, T, E, SH> c(g);
        // the cell as stored, in double
        for (int i = 0; i < Q; ++i) g[i] = (SH ? Lat<D>::w(i) : 0.0) + (double)c.p[i];
        const bool ok64 = newton(Cell<D, double, double, false>(g), cpr, ref);
        const bool ok_own = newton(c, E(cpr), own);
        int it = 0;
        const bool ok = quasi_equilibrium<D, T, E, SH>(c.p, c.d, c.rho, c.u, E(cpr), it);
        refused += ok_own && !ok;
        if (!ok) continue;
        ++accepted;
        bool fin = true;
        for (int i = 0; i < Q; ++i) fin = fin && std::isfinite((double)c.d[i]);
        nonfinite += !fin;
        if (!ok64) continue;
        for (int i = 0; i < Q; ++i) {
            err = std::fmax(err, std::fabs((double)c.d[i] - ref[i]) / (double)c.rho);
            if (ok_own) err_newton = std::fmax(err_newton, std::fabs(own[i] - ref[i]) / (double)c.rho);
        }
    }
    std::printf("%d %d %d %.3e %.3e\n", accepted, nonfinite, refused, err, err_newton);
    return 0;
}

int main(int argc, char **argv)
{
    if (argc != 9 || std::strcmp(argv[1], "qe")) return 2;
    const int D = std::atoi(argv[2]), cells = std::atoi(argv[6]);
    const double pr = std::atof(argv[4]), tau = std::atof(argv[5]), spread = std::atof(argv[8]);
    const unsigned seed = (unsigned)std::atoi(argv[7]);
    const char *t = argv[3];
    if (!std::strcmp(t, "f64"))
        return D == 2 ? run_qe<2, double, double, false>(pr, tau, cells, seed, spread)
                      : run_qe<3, double, double, false>(pr, tau, cells, seed, spread);
    if (!std::strcmp(t, "f32s"))
        return D == 2 ? run_qe<2, float, double, true>(pr, tau, cells, seed, spread)
                      : run_qe<3, float, double, true>(pr, tau, cells, seed, spread);
    return D == 2 ? run_qe<2, float, float, false>(pr, tau, cells, seed, spread)
                  : run_qe<3, float, float, false>(pr, tau, cells, seed, spread);
}
