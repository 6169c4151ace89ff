// Host side of the periodic splitting in FP64: the window that cuts 1/r into a
// short-range part, zero beyond r_c = L / 2, and a smooth part whose Fourier
// series ends at |n| = kWindowN.
//
// Any even window phi on [-r_c, r_c] splits 1/r = S(r) + Phi(r) / r with
// Phi(r) = int_0^r phi / int_0^{r_c} phi (Phi = 1 beyond r_c), and Phi(r) / r has
// the transform (4 pi / k^2) phihat(k) / phihat(0), phihat(k) = int phi(s) cos(k s) ds.
// Ewald's Gaussian is one choice (Phi = erf).  The window best concentrated on
// both sides at once is the prolate spheroidal function psi of order zero and
// bandwidth c (Slepian and Pollak, Bell Syst. Tech. J. 40, 43 (1961)): its
// transform is psi itself, phihat(k) / phihat(0) = psi(k r_c / c) / psi(0) for
// k <= c / r_c, and its tails are of the size psi(1) / psi(0).  With
// c = pi kWindowN the last reciprocal vector |n| = kWindowN lies at the band's
// edge; kWindowN = 13 leaves psi(1) / psi(0) = 4e-17 and a jump of the force
// kernel at r_c of 2e-16, where the Gaussian needs |n| <= 23 for 1e-15: 4 601
// vectors in half of k-space instead of 25 441.
//
// psi is expanded in normalised Legendre polynomials P_0, P_2, ...; its
// coefficients are the eigenvector of the lowest eigenvalue of a symmetric
// tridiagonal matrix (the spheroidal equation in that basis), found by inverse
// iteration.  The real-space loop needs the smooth part as polynomials in
// t = 1 - 2 (r / r_c)^2:
//   potential  Phi / r             = r_c^{-1} sum_i pot[i] t^i
//   force      (Phi - r phi) / r^3 = r_c^{-3} sum_i force[i] t^i
// the potential's interpolated at Chebyshev nodes (degree 29), the force's its
// derivative, 4 d/dt (degree 28); both within 1e-16 of the value at r_c.  All in
// long double, once per process (1 ms).
#pragma once

#include <cmath>

namespace colatus {

constexpr int kWindowN = 13;       // |n| <= kWindowN in reciprocal space
constexpr int kWindowDegree = 28;  // of the force polynomial (the potential's: one more)

struct EwaldWindow {
    static constexpr int kTerms = 48;  // Legendre terms P_0 .. P_94
    long double b[kTerms];             // psi(x) = sum_i b[i] P_{2i}(x)
    long double integral;              // int_0^1 psi
    double force[kWindowDegree + 1], pot[kWindowDegree + 2];
    double self;       // lim_{r->0} r_c Phi / r = psi(0) / integral
    double mean_s2;    // int_0^1 s^2 psi / integral
    // weight of reciprocal vector n by |n|^2 (a plan of a new box side needs them
    // all: 0.3 of its 0.5 ms when they are evaluated anew)
    double weight[kWindowN * kWindowN + 1];

    // P_0 .. P_{2 kTerms} at x
    static void legendre(long double x, long double *P)
    {
        P[0] = 1.0L;
        P[1] = x;
        for (int n = 1; n < 2 * kTerms; ++n)
            P[n + 1] = ((2 * n + 1) * x * P[n] - n * P[n - 1]) / (n + 1);
    }
    long double psi(long double x) const
    {
        long double P[2 * kTerms + 1], s = 0.0L;
        legendre(x, P);
        for (int i = kTerms - 1; i >= 0; --i)
            s += b[i] * P[2 * i];
        return s;
    }
    // int_0^x psi, from int P_n = (P_{n+1} - P_{n-1}) / (2n + 1)
    long double primitive(long double x) const
    {
        long double P[2 * kTerms + 1], s = 0.0L;
        legendre(x, P);
        for (int i = kTerms - 1; i > 0; --i)
            s += b[i] * (P[2 * i + 1] - P[2 * i - 1]) / (4 * i + 1);
        return s + b[0] * x;
    }
    EwaldWindow()
    {
        const long double pi = acosl(-1.0L), c = pi * kWindowN;
        // the matrix: diagonal dg, off-diagonal od
        long double dg[kTerms], od[kTerms], v[kTerms];
        for (int i = 0; i < kTerms; ++i) {
            const long double k = 2 * i;
            dg[i] = k * (k + 1) + (2 * k * (k + 1) - 1) / ((2 * k + 3) * (2 * k - 1)) * c * c;
            od[i] = (k + 2) * (k + 1) / ((2 * k + 3) * sqrtl((2 * k + 1) * (2 * k + 5))) * c * c;
            v[i] = 1.0L;
        }
        // positive definite: inverse iteration converges like (chi_0 / chi_2)^k
        for (int it = 0; it < 80; ++it) {
            long double d[kTerms];
            d[0] = dg[0];
            for (int i = 1; i < kTerms; ++i) {
                const long double f = od[i - 1] / d[i - 1];
                d[i] = dg[i] - f * od[i - 1];
                v[i] -= f * v[i - 1];
            }
            v[kTerms - 1] /= d[kTerms - 1];
            for (int i = kTerms - 2; i >= 0; --i)
                v[i] = (v[i] - od[i] * v[i + 1]) / d[i];
            long double s = 0.0L;
            for (int i = 0; i < kTerms; ++i)
                s += v[i] * v[i];
            s = 1.0L / sqrtl(s);
            for (int i = 0; i < kTerms; ++i)
                v[i] *= s;
        }
        for (int i = 0; i < kTerms; ++i)
            b[i] = v[i] * sqrtl((4 * i + 1) / 2.0L);
        integral = primitive(1.0L);
        const long double psi0 = psi(0.0L);
        for (int n2 = 0; n2 <= kWindowN * kWindowN; ++n2)
            weight[n2] = (double)(psi(sqrtl((long double)n2) / kWindowN) / psi0);
        self = (double)(psi0 / integral);
        // x^2 = (2 P_2 + P_0) / 3 and int_0^1 P_n^2 = 1 / (2n + 1)
        mean_s2 = (double)((b[0] / 3.0L + 2.0L / 15.0L * b[1]) / integral);
        constexpr int n = kWindowDegree + 2;
        long double val[n], mono[n];
        for (int k = 0; k < n; ++k) {
            const long double x = sqrtl(0.5L * (1.0L - cosl(pi * (k + 0.5L) / n)));
            val[k] = primitive(x) / integral / x;
            mono[k] = 0.0L;
        }
        // Chebyshev coefficients, to powers by T_{j+1} = 2 t T_j - T_{j-1}
        long double T0[n] = {1.0L}, T1[n] = {0.0L, 1.0L};
        for (int j = 0; j < n; ++j) {
            long double cheb = 0.0L;
            for (int k = 0; k < n; ++k)
                cheb += val[k] * cosl(pi * j * (k + 0.5L) / n);
            cheb *= (j == 0 ? 1.0L : 2.0L) / n;
            long double T2[n];
            for (int i = 0; i < n; ++i) {
                mono[i] += cheb * T0[i];
                T2[i] = (i > 0 ? 2.0L * T1[i - 1] : 0.0L) - T0[i];
            }
            for (int i = 0; i < n; ++i) {
                T0[i] = T1[i];
                T1[i] = T2[i];
            }
        }
        for (int i = 0; i < n; ++i)
            pot[i] = (double)mono[i];
        for (int i = 1; i < n; ++i)
            force[i - 1] = (double)(4.0L * i * mono[i]);
    }
};

inline const EwaldWindow &ewald_window()
{
    static const EwaldWindow w;
    return w;
}

}  // namespace colatus
