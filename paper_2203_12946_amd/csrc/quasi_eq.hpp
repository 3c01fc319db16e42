// Quasi-equilibrium of the entropic lattice ES-BGK collision (the section on
// the exact path length of the entropic lattice ES-BGK model).
//
// f^QE minimises H over the states with the cell's mass and momentum and the
// pressure tensor P(f^eq) + c_Pr sigma, sigma = P(g) - P(f^eq), P(f) =
// sum_i f_i c_i c_i, c_Pr = (1 - 1/Pr) / (1 + 1/(2 tau1 Pr)).  The paper
// writes the Maxwellian pressure where P(f^eq) stands: the lattice's own
// equilibrium pressure takes its place, so that f^QE = f^eq at Pr = 1 or
// sigma = 0.  The minimiser is f^QE_i = f^eq_i exp(delta . phi_i) over the
// basis phi = (1, c_a, c_a c_b for a <= b) (f^eq is the minimiser without
// the pressure constraint); delta solves the moment equations
//   F_k(delta) = sum_i f^eq_i expm1(delta . phi_i) phi_ik - T_k = 0,
// T = (0, 0, c_Pr sigma), and is found numerically, as the paper does, by
// Newton's method from delta = 0.
//
// Structure for a lane:
//  - On the tensor-product lattice every product phi_k phi_l reduces to a
//    monomial c_x^ex c_y^ey c_z^ez with exponents in {0, 1, 2} (c^3 = c,
//    c^4 = c^2).  All Q such moments of a per-population value are taken by
//    contracting one axis at a time (three adds per row of three), so the
//    residual and the Jacobian sum_i f^QE_i phi_i phi_i^T come from two
//    contractions per iteration instead of K^2 sums.
//  - The Jacobian is factored in single precision whatever the arithmetic
//    type: Newton then converges at least linearly at the rate of that
//    rounding (about 1e-7 times its condition), a handful of iterations
//    to double precision, while the residual, the step and delta are in E.
#pragma once

#include "lattice.hpp"

namespace eselbm {

__device__ inline float expm1_(float v) { return expm1f(v); }
__device__ inline double expm1_(double v) { return expm1(v); }

// expm1 for |v| <= 1/32 by its Taylor polynomial: truncated after v^N its
// relative error is below |v|^N / (N+1)! <= 4e-11 (float, N = 5) and 8e-21
// (double, N = 9), under the rounding of the type.  Near equilibrium every
// exponent delta . phi_i of a cell lies in that range (|delta . phi_i| <=
// sum_k |delta_k|, since phi_ik is 0 or +-1).
template <typename E>
struct SmallExpm1;
template <>
struct SmallExpm1<float> {
    static constexpr int N = 5;
};
template <>
struct SmallExpm1<double> {
    static constexpr int N = 9;
};
template <typename E>
__device__ inline E expm1_small(E v)
{
    constexpr int N = SmallExpm1<E>::N;
    // 1/k! for k = 1..N
    double inv_fact[N + 1];
    inv_fact[0] = 1.0;
#pragma unroll
    for (int k = 1; k <= N; ++k) inv_fact[k] = inv_fact[k - 1] / k;
    E p = E(inv_fact[N]);
#pragma unroll
    for (int k = N - 1; k >= 1; --k) p = fma_(p, v, E(inv_fact[k]));
    return p * v;
}
constexpr double kSmallExpArg = 1.0 / 32.0;

template <int D>
struct QEBasis {
    static constexpr int K = D == 2 ? 6 : 10;
    // exponent of basis function k along axis a: 1, c_x, c_y[, c_z], then
    // c_a c_b for a <= b in the order xx, xy[, xz], yy[, yz, zz]
    __host__ __device__ static constexpr int e(int k, int a)
    {
        if (k == 0) return 0;
        if (k <= D) return a == k - 1 ? 1 : 0;
        int q = k - 1 - D;
        for (int p = 0; p < D; ++p)
            for (int r = p; r < D; ++r) {
                if (q == 0) return (a == p) + (a == r);
                --q;
            }
        return 0;
    }
    // reduced exponent of a product: c^3 = c, c^4 = c^2
    __host__ __device__ static constexpr int red(int n) { return n == 0 ? 0 : (n % 2 == 1 ? 1 : 2); }
    // moment index (ex + 3 ey + 9 ez) of basis function k, and of phi_k phi_l
    __host__ __device__ static constexpr int m1(int k) { return e(k, 0) + 3 * e(k, 1) + 9 * e(k, 2); }
    __host__ __device__ static constexpr int m2(int k, int l)
    {
        return red(e(k, 0) + e(l, 0)) + 3 * red(e(k, 1) + e(l, 1)) + 9 * red(e(k, 2) + e(l, 2));
    }
    // phi_k at population i
    __host__ __device__ static constexpr int phi(int k, int i)
    {
        int v = 1;
        for (int a = 0; a < D; ++a) {
            const int c = Lat<D>::c(i, a);
            v *= e(k, a) == 0 ? 1 : (e(k, a) == 1 ? c : c * c);
        }
        return v;
    }
};

// Moments m[ex + 3 ey + 9 ez] = sum_i v_i c_x^ex c_y^ey c_z^ez, exponents in
// {0, 1, 2}: per axis, a row (v_-, v_0, v_+) becomes (sum, v_+ - v_-, v_+ + v_-).
template <int D, typename V>
__device__ inline void contract_rows(V (&m)[Lat<D>::Q])
{
    constexpr int Q = Lat<D>::Q;
#pragma unroll
    for (int stride = 1; stride < Q; stride *= 3) {
#pragma unroll
        for (int base = 0; base < Q; ++base) {
            if ((base / stride) % 3 != 0) continue;
            const V a = m[base], b = m[base + stride], c = m[base + 2 * stride];
            m[base] = (a + b) + c;
            m[base + stride] = c - a;
            m[base + 2 * stride] = c + a;
        }
    }
}

// The exponents delta . phi_i of a cell, grouped by axis.  With the basis
// ordered (1, c_x, c_y[, c_z], c_x^2, c_x c_y[, c_x c_z], c_y^2[, c_y c_z,
// c_z^2]) (QEBasis),
//   delta . phi_i = X(c_x) + R(c_y, c_z) + c_x G(c_y, c_z),
// X holding the terms in c_x alone (and the constant), R those in c_y and
// c_z alone, G the coefficients of the mixed products with c_x: 3 + 2 x 3^(D-1)
// values formed once, then one or two additions per population instead of a
// sum over the K basis functions.
template <int D, typename E>
struct QEArgs {
    E X[3], R[D == 3 ? 9 : 3], G[D == 3 ? 9 : 3];
    __device__ explicit QEArgs(const E (&dl)[QEBasis<D>::K])
    {
        // basis indices: D = 3: 0 1, 1 x, 2 y, 3 z, 4 xx, 5 xy, 6 xz, 7 yy,
        // 8 yz, 9 zz; D = 2: 0 1, 1 x, 2 y, 3 xx, 4 xy, 5 yy
        constexpr int XX = D == 3 ? 4 : 3, XY = D == 3 ? 5 : 4, YY = D == 3 ? 7 : 5;
        X[0] = (dl[0] - dl[1]) + dl[XX];
        X[1] = dl[0];
        X[2] = (dl[0] + dl[1]) + dl[XX];
        const E Y[3] = {dl[YY] - dl[2], E(0), dl[YY] + dl[2]};
        if constexpr (D == 3) {
            const E Z[3] = {dl[9] - dl[3], E(0), dl[9] + dl[3]};
#pragma unroll
            for (int cz = -1; cz <= 1; ++cz)
#pragma unroll
                for (int cy = -1; cy <= 1; ++cy) {
                    const int r = (cy + 1) + 3 * (cz + 1);
                    E rv = Y[cy + 1] + Z[cz + 1];
                    if (cy * cz > 0) rv += dl[8];
                    if (cy * cz < 0) rv -= dl[8];
                    R[r] = rv;
                    E g = E(0);
                    if (cy > 0) g += dl[XY];
                    if (cy < 0) g -= dl[XY];
                    if (cz > 0) g += dl[6];
                    if (cz < 0) g -= dl[6];
                    G[r] = g;
                }
        } else {
#pragma unroll
            for (int cy = -1; cy <= 1; ++cy) {
                R[cy + 1] = Y[cy + 1];
                G[cy + 1] = cy > 0 ? dl[XY] : (cy < 0 ? -dl[XY] : E(0));
            }
        }
    }
    // delta . phi_i (i compile-time after unrolling)
    __device__ E operator()(int i) const
    {
        const int cx = Lat<D>::c(i, 0), r = (Lat<D>::c(i, 1) + 1) + 3 * (D == 3 ? Lat<D>::c(i, 2) + 1 : 0);
        if (cx == 0) return X[1] + R[r];
        return cx > 0 ? (X[2] + R[r]) + G[r] : (X[0] + R[r]) - G[r];
    }
};

template <typename E>
struct QECfg;
// Converged when no component of the Newton step exceeds tol; given up
// after maxit steps or on a step of 1e3 or more (a target pressure that no
// positive state carries sends the multipliers off to infinity).  Near
// equilibrium three to five steps suffice; cells far from it can need
// tens, and a wave runs until its slowest lane stops.
template <>
struct QECfg<float> {
    static constexpr float tol = 1e-6f;
    static constexpr int maxit = 50;
};
template <>
struct QECfg<double> {
    static constexpr double tol = 1e-13;
    static constexpr int maxit = 50;
};

// true in every lane when every lane's exponents delta . phi_i are within the
// range of expm1_small (a wave-uniform choice, so that the wave takes one of
// the two forms)
template <int K, typename E>
__device__ inline bool small_exponents(const E (&dl)[K])
{
    E bound = E(0);
#pragma unroll
    for (int k = 0; k < K; ++k) bound += abs_(dl[k]);
    return __ballot(!(bound <= E(kSmallExpArg))) == 0ull;
}

// out(i, r_i) of r_i = feq_i expm1(delta . phi_i)
template <int D, typename E, typename FE, typename OUT>
__device__ inline void qe_excess(const E (&delta)[QEBasis<D>::K], FE fe, OUT out)
{
    const QEArgs<D, E> qa(delta);
    if (small_exponents(delta)) {
#pragma unroll
        for (int i = 0; i < Lat<D>::Q; ++i) out(i, fe(i) * expm1_small(qa(i)));
    } else {
#pragma unroll
        for (int i = 0; i < Lat<D>::Q; ++i) out(i, fe(i) * expm1_(qa(i)));
    }
}

// The inverse of the Jacobian at delta = 0, J0 = sum_i feq_i phi_i phi_i^T, in
// closed form.  The equilibrium is a product over the axes, so under it the
// c_a are independent, and in the basis
//   1, v_a = c_a - u_a, v_a v_b, q_a = c_a^2 - s_a - k_a v_a,
//   s_a = <c_a^2>, V_a = s_a - u_a^2, k_a = u_a (1 - s_a) / V_a,
// orthogonal under it, J0 is rho diag(1, V_a, V_a V_b, W_a),
// W_a = s_a (1 - s_a) - k_a^2 V_a.  With M the change to that basis
// J0^-1 = M^T diag^-1 M: some 60 operations, no factorisation.
template <int D, typename E>
struct QEInverse {
    E u[3], k[3], sk[3], ir, iV[3], iW[3];  // sk = s - k u
    __device__ QEInverse(E rho, const E (&u_)[3])
    {
        ir = rcp_(rho);
#pragma unroll
        for (int a = 0; a < D; ++a) {
            u[a] = u_[a];
            const E u2 = u[a] * u[a], sq = sqrt_(fma_(E(3), u2, E(1)));
            const E s = E(1.0 / 3.0) + E(2) * u2 * rcp_(E(1) + sq), V = s - u2;
            iV[a] = rcp_(V);
            k[a] = u[a] * (E(1) - s) * iV[a];
            iW[a] = rcp_(s * (E(1) - s) - k[a] * k[a] * V);
            sk[a] = fma_(-k[a], u[a], s);
        }
    }
    // out = J0^-1 r (r and out in the basis QEBasis)
    template <typename R>
    __device__ void operator()(R r, E (&out)[QEBasis<D>::K]) const
    {
        constexpr int SEC = 1 + D;  // second moments, a <= b
        const E m0 = r(0);
        E c0 = m0, c1[3] = {E(0), E(0), E(0)};
#pragma unroll
        for (int a = 0; a < D; ++a) {
            const E e = fma_(-u[a], m0, r(1 + a)) * iV[a];
            c0 = fma_(-u[a], e, c0);
            c1[a] = e;
        }
        int q = SEC;
#pragma unroll
        for (int a = 0; a < D; ++a)
#pragma unroll
            for (int b = a; b < D; ++b, ++q) {
                if (a == b) {
                    // q_a = c_a^2 - k_a c_a - (s_a - k_a u_a)
                    const E e = (r(q) - fma_(k[a], r(1 + a), sk[a] * m0)) * iW[a];
                    out[q] = e * ir;
                    c1[a] = fma_(-k[a], e, c1[a]);
                    c0 = fma_(-sk[a], e, c0);
                } else {
                    const E e = (r(q) - fma_(u[a], r(1 + b), u[b] * fma_(-u[a], m0, r(1 + a)))) * (iV[a] * iV[b]);
                    out[q] = e * ir;
                    c1[a] = fma_(-u[b], e, c1[a]);
                    c1[b] = fma_(-u[a], e, c1[b]);
                    c0 = fma_(u[a] * u[b], e, c0);
                }
            }
        out[0] = c0 * ir;
#pragma unroll
        for (int a = 0; a < D; ++a) out[1 + a] = c1[a] * ir;
    }
};

// The solve near equilibrium.  delta starts from the exact first Newton step,
// J0^-1 T; each further step is Newton's with the inverse of J = J0 + dJ, dJ_kl
// = sum_i r_i phi_ik phi_il, as its Neumann series from J0^-1 to NT terms:
//   s = sum_m (-J0^-1 dJ)^m (-J0^-1 F),
// whose matrix entries are the moments the residual needs anyway.  With g the
// measured ratio of successive terms a step leaves an error of about
// (g^NT + |s|) |s|; converged when that is below tol.  Returns false where the
// terms do not shrink (g above 0.3) or maxit steps do not do: the caller then
// takes Newton's method with a factored Jacobian.
template <typename E>
struct QEFastCfg;
template <>
struct QEFastCfg<float> {
    static constexpr int NT = 2, maxit = 6;
    static constexpr float tol = 1e-9f;
};
template <>
struct QEFastCfg<double> {
    static constexpr int NT = 4, maxit = 6;
    static constexpr double tol = 1e-17;
};
template <int D, typename E, typename FE>
__device__ inline bool qe_fast(FE fe, const QEInverse<D, E> &inv, const E (&tgt)[QEBasis<D>::K],
                               E (&delta)[QEBasis<D>::K], int &iters)
{
    using B = QEBasis<D>;
    using C = QEFastCfg<E>;
    constexpr int Q = Lat<D>::Q, K = B::K;
    inv([&](int k) { return k <= D ? E(0) : tgt[k]; }, delta);
    bool conv = false, ok = true;
    int it = 1;
    for (; it <= C::maxit && ok && !conv; ++it) {
        E mr[Q];
        qe_excess<D, E>(delta, fe, [&](int i, E r) { mr[i] = r; });
        contract_rows<D, E>(mr);
        E t[K], s[K];
        inv([&](int k) { return tgt[k] - mr[B::m1(k)]; }, t);
        E m0 = E(0), m1 = E(0), g = E(0);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            s[k] = t[k];
            m0 = fmax_(m0, abs_(t[k]));
        }
#pragma unroll
        for (int m = 1; m < C::NT; ++m) {
            E y[K];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                E v = E(0);
#pragma unroll
                for (int l = 0; l < K; ++l) v = fma_(mr[B::m2(k, l)], t[l], v);
                y[k] = -v;
            }
            inv([&](int k) { return y[k]; }, t);
            m1 = E(0);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                s[k] += t[k];
                m1 = fmax_(m1, abs_(t[k]));
            }
            if (m == 1) g = m1;
        }
        E mx = E(0);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            delta[k] += s[k];
            mx = fmax_(mx, abs_(s[k]));
        }
        ok = g <= E(0.3) * m0 && mx < E(0.25);
        E gn = g * rcp_(fmax_(m0, E(1e-30)));
        gn = C::NT == 2 ? gn * gn : (gn * gn) * (gn * gn);
        conv = ok && (gn + mx) * mx <= C::tol;
    }
    // The maxima drop a NaN: where the moments of overflowing exponentials
    // left one in the step, it shows in the sum of the multipliers, which the
    // caller's choice of the exponential's form takes anyway.  The bound on a
    // multiplier is that of qe_newton's steps.
    E sum = E(0);
#pragma unroll
    for (int k = 0; k < K; ++k) sum += abs_(delta[k]);
    iters = it - 1;
    return conv && sum < E(1e3);
}

// The solve by Newton's method from delta = 0 with the Jacobian factored, for
// the cells qe_fast leaves (far from equilibrium).
template <int D, typename E, typename FE>
__device__ inline bool qe_newton(FE fe, const E (&tgt)[QEBasis<D>::K], E (&delta)[QEBasis<D>::K], int &iters)
{
    using B = QEBasis<D>;
    constexpr int Q = Lat<D>::Q, K = B::K;
    // moments of f^eq (single precision: they serve the Jacobian only)
    float mfe[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) mfe[i] = float(fe(i));
    contract_rows<D, float>(mfe);

#pragma unroll
    for (int k = 0; k < K; ++k) delta[k] = E(0);
    bool conv = false;
    int it = 0;
    for (; it < QECfg<E>::maxit && !conv; ++it) {
        // r_i = feq_i expm1(delta . phi_i): its moments give the residual,
        // and with those of feq the Jacobian's (f^QE = feq + r).  The first
        // step starts from delta = 0, where r = 0: its moments are zero
        // without evaluating the Q exponentials.
        E mr[Q];
        if (it == 0) {
#pragma unroll
            for (int i = 0; i < Q; ++i) mr[i] = E(0);
        } else {
            qe_excess<D, E>(delta, fe, [&](int i, E r) { mr[i] = r; });
            contract_rows<D, E>(mr);
        }
        // Cholesky of J_kl = sum f^QE phi_k phi_l, packed lower triangle
        float L[K * (K + 1) / 2];
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int l = 0; l <= k; ++l) L[k * (k + 1) / 2 + l] = mfe[B::m2(k, l)] + float(mr[B::m2(k, l)]);
        bool spd = true;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            float dj = L[j * (j + 1) / 2 + j];
#pragma unroll
            for (int q = 0; q < j; ++q) dj -= L[j * (j + 1) / 2 + q] * L[j * (j + 1) / 2 + q];
            spd = spd && dj > 0.0f;
            const float ljj = sqrt_(fmax_(dj, 1e-30f)), ij = rcp_(ljj);
            L[j * (j + 1) / 2 + j] = ljj;
#pragma unroll
            for (int r = j + 1; r < K; ++r) {
                float v = L[r * (r + 1) / 2 + j];
#pragma unroll
                for (int q = 0; q < j; ++q) v -= L[r * (r + 1) / 2 + q] * L[j * (j + 1) / 2 + q];
                L[r * (r + 1) / 2 + j] = v * ij;
            }
        }
        // step s = -J^-1 F in E
        E y[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            E v = tgt[k] - mr[B::m1(k)];
#pragma unroll
            for (int q = 0; q < k; ++q) v -= E(L[k * (k + 1) / 2 + q]) * y[q];
            y[k] = v * E(rcp_(L[k * (k + 1) / 2 + k]));
        }
        E mx = E(0);
#pragma unroll
        for (int k = K - 1; k >= 0; --k) {
            E v = y[k];
#pragma unroll
            for (int q = k + 1; q < K; ++q) v -= E(L[q * (q + 1) / 2 + k]) * y[q];
            y[k] = v * E(rcp_(L[k * (k + 1) / 2 + k]));
            delta[k] += y[k];
            mx = fmax_(mx, abs_(y[k]));
        }
        // a NaN step fails both comparisons and ends the loop unconverged
        if (!spd || !(mx < E(1e3))) break;
        conv = mx <= E(QECfg<E>::tol);
    }
    iters = it;
    return conv;
}

// Replaces d = feq - g by f^QE - g.  p holds the stored values (g, or g - w
// when SH), d the deviation of the equilibrium, rho and u its density and
// velocity; E is the arithmetic type of the solve.  Returns false when Newton
// does not converge (the target pressure lies beyond what positive
// populations carry): d is then left as the equilibrium's.  iters receives
// the Newton iterations.
template <int D, typename T, typename E, bool SH>
__device__ inline bool quasi_equilibrium(const T (&p)[Lat<D>::Q], T (&d)[Lat<D>::Q], E rho, const E (&u)[3], E cpr,
                                         int &iters)
{
    using B = QEBasis<D>;
    constexpr int Q = Lat<D>::Q, K = B::K;
    auto fe = [&](int i) { return E(gval<D, T, SH>(i, p)) + E(d[i]); };
    // target T_k = c_Pr sigma_k = -c_Pr sum_i d_i phi_ik (second moments)
    E tgt[K], delta[K];
    {
        E md[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) md[i] = E(d[i]);
        contract_rows<D, E>(md);
#pragma unroll
        for (int k = 0; k < K; ++k) tgt[k] = k <= D ? E(0) : -cpr * md[B::m1(k)];
    }
    bool conv = qe_fast<D, E>(fe, QEInverse<D, E>(rho, u), tgt, delta, iters);
    if (!conv) conv = qe_newton<D, E>(fe, tgt, delta, iters);
    if (!conv) return false;
    qe_excess<D, E>(delta, fe, [&](int i, E r) { d[i] = T(E(d[i]) + r); });
    conserve_moments<D, T>(d);
    return true;
}

}  // namespace eselbm
