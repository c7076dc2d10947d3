// noise_node.hpp -- the 2D noise covariance of one table node, shared by the phi-node and
// time-node table kernels.
//
// Eq. (covariance_matrix_direct) from the full Bunch-Davies mode of eq. (delta_phi_bessel) at
// -k eta = sigma: with y = -k eta, delta phi_k = H k^(-3/2) F(y), F = y^(3/2) (A J_nu + B Y_nu),
// delta pi_k = H k^(-3/2) (-y F'(y)), so Xi = H^2/(2 pi^2) [[|F|^2, Re(F conj G)], [., |G|^2]]
// with G = -y F'.  Y_nu = (J_nu cos nu pi - J_-nu)/sin nu pi turns F into alpha_+ y^(3/2) J_nu +
// alpha_- y^(3/2) J_-nu, each J_mu summed as its power series (at most 30 terms: below 1e-40 of the
// leading term for sigma <= 2), each term from the one before.  nu^2 = 9/4 - 3 (V''/V - (V'/V)^2) and
// H^2 = V/3 as for the 1D table.
#pragma once

#include "potential.hpp"

#include <hip/hip_runtime.h>

#include <cmath>

namespace fpt {

struct Cplx {
    double re, im;
};
__device__ __forceinline__ Cplx cscale(Cplx a, double s) { return {a.re * s, a.im * s}; }
__device__ __forceinline__ Cplx cadd(Cplx a, Cplx b) { return {a.re + b.re, a.im + b.im}; }

// A value h with a correction l, and sums, products and quotients that keep it (two_sum: Knuth's).
struct Sum2 {
    double h, l;
};
__device__ __forceinline__ Sum2 two_sum(double a, double b)
{
    const double s = a + b, v = s - a;
    return {s, (a - (s - v)) + (b - v)};
}
__device__ __forceinline__ Sum2 add2(Sum2 a, Sum2 b)
{
    const Sum2 s = two_sum(a.h, b.h);
    return {s.h, s.l + (a.l + b.l)};
}
__device__ __forceinline__ Sum2 mul2(Sum2 a, double b)
{
    const double p = a.h * b;
    return {p, fma(a.h, b, -p) + a.l * b};
}
__device__ __forceinline__ Sum2 div2(Sum2 a, Sum2 b)
{
    const double q = a.h / b.h;
    return {q, (fma(-q, b.h, a.h) + (a.l - q * b.l)) / b.h};
}

// Xi at phi; false (and zeros) where V <= 0, nu^2 <= 0 or nu is within 1e-3 of an integer (the
// Y_nu form above needs sin nu pi away from 0).
__device__ inline bool bessel2d_node(const PotParams &pp, double sigma, double phi, double &Xpp, double &Xpq,
                                     double &Xqq)
{
    double V, dV, d2V;
    pot_eval(pp, phi, false, V, dV, d2V);
    const double r1 = dV / V, r2 = d2V / V;
    const double nu2 = 2.25 - 3.0 * (r2 - r1 * r1);
    const double nu = nu2 > 0.0 ? sqrt(nu2) : 0.0;
    double sn, cs;
    sincospi(nu, &sn, &cs);
    if (!(V > 0.0) || !(nu2 > 0.0) || fabs(sn) < 1e-3) {
        Xpp = Xpq = Xqq = 0.0;
        return false;
    }
    // A_k, B_k of eq. (A_k_and_B_k): sqrt(pi)/2 exp(i (nu + 1/2) pi/2), sqrt(pi)/2 exp(i (nu + 3/2) pi/2)
    const double hs = 0.5 * sqrt(M_PI);
    double sa, ca, sb, cb;
    sincospi(0.5 * (nu + 0.5), &sa, &ca);
    sincospi(0.5 * (nu + 1.5), &sb, &cb);
    const Cplx Ak = {hs * ca, hs * sa}, Bk = {hs * cb, hs * sb};
    const Cplx alpha[2] = {cadd(Ak, cscale(Bk, cs / sn)), cscale(Bk, -1.0 / sn)};
    const double mus[2] = {nu, -nu};
    Cplx F = {0.0, 0.0}, G = {0.0, 0.0};
    // term_m = (-1)^m sigma^p / (m! Gamma(m + mu + 1) 2^(2m + mu)), p = 2m + mu + 3/2.  With powers and
    // gamma functions taken anew for every term, a node cost 240 library calls and 2048 nodes 103 us on
    // their 32 waves; the ratio of neighbouring terms leaves two of each.  Terms and sums carry
    // their rounding errors: without them the recurrence was off by up to 11 % more than separate terms (rms of
    // Xpp over 281 nodes at sigma = 0.05, 1, 1.5: 8.3e-16, 4.7e-16, 5.2e-16 against 8.1e-16, 4.2e-16, 4.9e-16), with
    // them by less (7.8e-16, 3.6e-16, 3.4e-16).
    const double rt = sqrt(sigma), p = sigma * rt;
    const double dp = fma(sigma, rt, -p) + sigma * (fma(-rt, rt, sigma) / (2.0 * rt));      // sigma^(3/2) = p + dp
    const double q = -0.25 * sigma * sigma, dq = -0.25 * fma(sigma, sigma, 4.0 * q);        // -(sigma/2)^2 = q + dq
    for (int k = 0; k < 2; ++k) {
        const double mu = mus[k];
        const double w = pow(0.5 * sigma, mu), gam = tgamma(mu + 1.0);
        Sum2 t = div2(mul2(Sum2{p, dp}, w), Sum2{gam, 0.0});
        Sum2 f = t, g = mul2(t, mu + 1.5);
        for (int m = 1; m < 30; ++m) {
            const Sum2 md = two_sum((double)m, mu);
            const Sum2 n = {t.h * q, fma(t.h, q, -t.h * q) + fma(t.l, q, t.h * dq)};
            t = div2(n, mul2(md, (double)m));
            f = add2(f, t);
            const Sum2 c = two_sum(2.0 * m + 1.5, mu);
            g = add2(g, Sum2{t.h * c.h, fma(t.h, c.h, -t.h * c.h) + fma(t.l, c.h, t.h * c.l)});
            if (fabs(t.h) * 1e3 < 1e-18 * fmin(fabs(f.h), fabs(g.h)) && (double)m > nu) break;
        }
        F = cadd(F, cscale(alpha[k], f.h + f.l));
        G = cadd(G, cscale(alpha[k], -(g.h + g.l)));
    }
    const double c = (V / 3.0) / (2.0 * M_PI * M_PI);
    Xpp = c * (F.re * F.re + F.im * F.im);
    Xpq = c * (F.re * G.re + F.im * G.im);      // Re(F conj(G))
    Xqq = c * (G.re * G.re + G.im * G.im);
    return true;
}

}  // namespace fpt
