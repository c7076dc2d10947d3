// fpt_table.hip -- the Bessel-matched noise table of eq. (covariance_constant_nu_bessel_matched)
// (Sec. 3.4): the classical trajectory, one Fourier mode per table node solved through
// eq. (full_delta_phi) from its Bunch-Davies state to the coarse-graining time, and the
// Bessel coefficient B_k of eq. (bessel_matching) that rescales the node's noise.
//
// The classical trajectory is a sequential ODE whose samples, kBgStep e-folds apart, the nodes
// read.  bg_macro_kernel strides over up to kMacroMax samples per step with an order-16 extrapolated
// step whose columns run on the lanes of one wave, and bg_fill_kernel fills the samples in between,
// each chunk of samples on a thread of its own.  A mode is linear in its own state, so its solve
// splits in time: mode_segment_kernel integrates the 2 x 2 propagator of one segment of one node per
// thread, and the node's thread multiplies the segments.  All in FP64.
#include "internal.hpp"
#include "noise_node.hpp"

#include <hip/hip_runtime.h>

#include <climits>
#include <cmath>

namespace fpt {

namespace {

constexpr double kBgStep = 1e-4;         // e-folds between trajectory samples
constexpr int kBgLast = 2000000;         // the trajectory's last sample at most: 200 e-folds
constexpr double kModeMaxStep = 2.5e-4;  // largest RK4 step of a mode, in e-folds
constexpr double kStepsPerPeriod = 800.0;
constexpr double kStartRatio = 100.0;    // a mode starts at k = 100 aH
constexpr int kMacroMax = 2048;          // samples spanned by one extrapolated step of the trajectory, at most
constexpr int kFillChunk = 16;           // trajectory samples filled by one thread
constexpr int kCols = 8;                 // columns of the extrapolation (2, 4, .., 16 midpoint steps)

using Pot = PotParams;

// The RK4 step that ends on the kink of the piecewise-linear potential is evaluated on the
// upper branch (pot_eval's `upper`).

__device__ inline double hubble2(const Pot &p, double phi, double pi_)
{
    double V, dV, d2V;
    pot_eval(p, phi, false, V, dV, d2V);
    return V / (3.0 - 0.5 * pi_ * pi_);
}

// nu^2 of eq. (nu_squared_approximation).
__device__ inline double nu2_of(const Pot &p, double phi)
{
    double V, dV, d2V;
    pot_eval(p, phi, false, V, dV, d2V);
    const double r1 = dV / V;
    return 2.25 - 3.0 * (d2V / V - r1 * r1);
}

// The background.
struct Bg {
    double phi, pi_;
};

// Its time derivative in N: eq. (klein_gordon) in e-folds with H^2 = V/(3 - eps1) from eq. (Friedmann).
__device__ inline Bg deriv(const Pot &p, const Bg &s, bool upper)
{
    double V, dV, d2V;
    pot_eval(p, s.phi, upper, V, dV, d2V);
    const double q = 3.0 - 0.5 * s.pi_ * s.pi_;
    return Bg{s.pi_, -q * (s.pi_ + dV / V)};
}

__device__ inline Bg axpy(const Bg &s, const Bg &k, double c) { return Bg{s.phi + c * k.phi, s.pi_ + c * k.pi_}; }

__device__ inline Bg rk4(const Pot &p, double h, const Bg &s, bool upper)
{
    const Bg k1 = deriv(p, s, upper);
    const Bg k2 = deriv(p, axpy(s, k1, 0.5 * h), upper);
    const Bg k3 = deriv(p, axpy(s, k2, 0.5 * h), upper);
    const Bg k4 = deriv(p, axpy(s, k3, h), upper);
    const double c = h / 6.0;
    return Bg{s.phi + c * (k1.phi + 2.0 * (k2.phi + k3.phi) + k4.phi),
              s.pi_ + c * (k1.pi_ + 2.0 * (k2.pi_ + k3.pi_) + k4.pi_)};
}

// Integrate from *N to N_stop in steps of at most h_max.  On the piecewise-linear potential, the step that
// would take phi from above phi_T to at or below it is cut, by bisection of its length, to end on phi_T, and
// phi continues one ulp below phi_T.
__device__ void advance(const Pot &p, double &N, double N_stop, Bg &s, double h_max)
{
    const bool has_kink = p.kind == kPotPiecewiseLinear;
    while (N < N_stop) {
        const double h = fmin(h_max, N_stop - N);
        const Bg t = rk4(p, h, s, false);
        if (!(has_kink && s.phi > p.phi_T && t.phi <= p.phi_T)) {
            s = t;
            N += h;
            continue;
        }
        double lo = 0.0, hi = h;
        for (int it = 0; it < 64; ++it) {
            const double mid = 0.5 * (lo + hi);
            if (rk4(p, mid, s, true).phi > p.phi_T) lo = mid;
            else hi = mid;
        }
        s = rk4(p, hi, s, true);
        N += hi;
        s.phi = nextafter(p.phi_T, -INFINITY);
    }
}

// J_mu(y) and y J_mu'(y) by the power series, each term from the previous one:
// t_m = t_{m-1} (-(y/2)^2) / (m (m + mu)),  t_0 = (y/2)^mu / Gamma(mu + 1).
__device__ inline void bessel_j(double mu, double y, double &J, double &yJp)
{
    const double q = -0.25 * y * y;
    double t = pow(0.5 * y, mu) / tgamma(mu + 1.0);
    double s = t, sd = mu * t;
    for (int m = 1; m < 40; ++m) {
        t *= q / ((double)m * ((double)m + mu));
        s += t;
        sd += (2.0 * m + mu) * t;
    }
    J = s;
    yJp = sd;
}

// ---------------------------------------------------------------------------
// The classical trajectory.  Sample i is the state after i steps of kBgStep.
//
// An extrapolated step (Gragg, Bulirsch and Stoer): column c integrates the step by the modified
// midpoint rule with 2 (c + 1) substeps, whose error is a series in the substep's square, and the
// columns' polynomial extrapolation to substep 0 has order 16 with eight columns.  The states are
// held as differences from the step's start, so that the extrapolation's weights (up to 50) do not
// multiply the rounding of the state itself.
// ---------------------------------------------------------------------------
// 1/x for normal x, to about an ulp: the hardware reciprocal and two Newton steps.
__device__ __forceinline__ double recip(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}

__device__ inline Bg bg_deriv(const Pot &p, double phi, double pi_, bool upper)
{
    double V, dV, d2V;
    pot_eval(p, phi, upper, V, dV, d2V);
    return Bg{pi_, -(3.0 - 0.5 * pi_ * pi_) * fma(dV, recip(V), pi_)};
}

// The difference (dphi, dpi) over H by the modified midpoint rule with n (even) substeps.
__device__ inline Bg midpoint(const Pot &p, Bg y, double H, int n, bool upper)
{
    const double h = H / n;
    Bg a{0.0, 0.0}, f = bg_deriv(p, y.phi, y.pi_, upper);
    Bg b{h * f.phi, h * f.pi_};
    for (int m = 1; m < n; ++m) {
        f = bg_deriv(p, y.phi + b.phi, y.pi_ + b.pi_, upper);
        const Bg t{a.phi + 2.0 * h * f.phi, a.pi_ + 2.0 * h * f.pi_};
        a = b;
        b = t;
    }
    return b;
}

// Weight of column c in the extrapolation over the first `cols` columns: prod_{j != c} n_c^2/(n_c^2 - n_j^2).
__host__ __device__ constexpr double col_weight(int c, int cols)
{
    double w = 1.0;
    for (int j = 0; j < cols; ++j)
        if (j != c) w *= (double)((c + 1) * (c + 1)) / (double)((c + 1) * (c + 1) - (j + 1) * (j + 1));
    return w;
}

__device__ constexpr double kColWeight[kCols] = {col_weight(0, kCols), col_weight(1, kCols), col_weight(2, kCols),
                                                 col_weight(3, kCols), col_weight(4, kCols), col_weight(5, kCols),
                                                 col_weight(6, kCols), col_weight(7, kCols)};

// The state after H by the extrapolated step, one thread.
__device__ inline Bg extrapolated(const Pot &p, Bg y, double H, bool upper)
{
    Bg s{0.0, 0.0};
#pragma unroll 1
    for (int c = 0; c < kCols; ++c) {
        const Bg d = midpoint(p, y, H, 2 * (c + 1), upper);
        s.phi += kColWeight[c] * d.phi;
        s.pi_ += kColWeight[c] * d.pi_;
    }
    return Bg{y.phi + s.phi, y.pi_ + s.pi_};
}

// A stride of the trajectory: from the state (phi, pi_) at sample `first` to sample `last` on one
// smooth branch (`upper`: the piecewise-linear potential's phi >= phi_T one, continued).
struct MacroRec {
    int first, last, upper, pad;
    double phi, pi_;
};
constexpr int kMacroCap = 1 << 16;
static_assert(kBgLast < kMatchCap, "room for every sample");

// The last sample and the number of strides; the first sample at which the trajectory ended, and the
// first at or below phi_ref (INT_MAX if none).
struct BgEnd {
    int last, nrec, stop, ref;
};

// Where the trajectory's samples are and how far they go.
struct BgStore {
    double *N, *phi, *pi_;   // samples (kMatchCap)
    MacroRec *rec;           // strides of more than one sample (kMacroCap)
    BgEnd *end;
};

__device__ inline void put_sample(const BgStore &b, int i, double N, Bg y)
{
    b.N[i] = N;
    b.phi[i] = y.phi;
    b.pi_[i] = y.pi_;
}

// The trajectory by strides, one wave.  A stride of m samples is an extrapolated step; it is halved
// while the order-14 result differs from the order-16 one by more than kTol (the order-16 error is
// far smaller still) or while it would cross the kink of the piecewise-linear potential, and doubled
// again where that difference is down at the rounding, kHold accepted strides after a refusal.  A stride of one sample is a plain
// RK4 step, which also cuts its step on the kink (advance), so whatever the potential does, the
// samples are at least those of a sequential RK4 solve.  On the upper branch with A_+ > 0 the field
// cannot dip below the kink and return within a stride (V' > 0 keeps pi < 0); with A_+ <= 0 every
// stride is one sample.  So it is on the Gaussian bump: there V'/V changes over 0.016 in phi, so the
// rounding of phi at every sample moves the trajectory by some 1e-13, and tables from sequential
// solves that share it agree to 1e-14, which a stride's more accurate path would not.
// The chain is bound by latency: 3.3e5 dependent RK4 steps (33 e-folds) took 314 ms on one thread; the
// strides of 16 dependent evaluations take 0.29 ms, and the samples between them 0.03 ms (bg_fill_kernel).
// stop_phi: the samples end once phi < stop_phi (phi nodes; -inf for time nodes).  ref_phi: they
// end N_after e-folds after phi first reached ref_phi (time nodes; -inf for phi nodes).  A stride may pass
// these ends (bg_scan_kernel finds the sample), but the last one is cut at kBgLast: what lies beyond is
// not part of the trajectory.
template <int KIND>
__global__ void __launch_bounds__(64) bg_macro_kernel(Pot pot, double phi_start, double pi_start, double stop_phi,
                                                      double ref_phi, double N_after, BgStore b)
{
    constexpr double kTol = 1e-12, kSmooth = 3e-14;
    constexpr int kHold = 6;
    const int lane = threadIdx.x;
    Pot p = pot;
    p.kind = KIND;
    constexpr bool linear = KIND == kPotPiecewiseLinear;
    const int m_max = (KIND == kPotGaussianBump || (linear && !(p.Ap > 0.0))) ? 1 : kMacroMax;
    Bg y{phi_start, pi_start};
    int i = 0, m = m_max, nrec = 0, hold = 0;
    double N = 0.0, N_end = INFINITY;
    if (lane == 0) put_sample(b, 0, N, y);
    while (!(y.phi < stop_phi || 0.5 * y.pi_ * y.pi_ >= 1.0 || i >= kBgLast || N >= N_end)) {
        const bool upper = linear && y.phi > p.phi_T;
        // a state that is no number stays one: the remaining samples are filled with it
        const bool lost = nrec < kMacroCap && !(fabs(y.phi) < INFINITY && fabs(y.pi_) < INFINITY);
        const int room = kBgLast - i;
        if (m > room) m = room;
        if (nrec >= kMacroCap) m = 1;
        Bg z = y;
        bool take = m == 1 || lost;
        double err = 0.0;
        if (!take) {
            const double H = (double)m * kBgStep;
            const Bg d = midpoint(p, y, H, 2 * ((lane & (kCols - 1)) + 1), upper);
            Bg s8{0.0, 0.0}, s7{0.0, 0.0};
#pragma unroll
            for (int c = 0; c < kCols; ++c) {
                const double dp = __shfl(d.phi, c), dq = __shfl(d.pi_, c);
                s8.phi += col_weight(c, kCols) * dp;
                s8.pi_ += col_weight(c, kCols) * dq;
                if (c < kCols - 1) {
                    s7.phi += col_weight(c, kCols - 1) * dp;
                    s7.pi_ += col_weight(c, kCols - 1) * dq;
                }
            }
            z = Bg{y.phi + s8.phi, y.pi_ + s8.pi_};
            const double e_phi = fabs(s8.phi - s7.phi) / (fabs(s8.phi) + 1e-3 * fabs(y.phi) + 1e-300);
            const double e_pi = fabs(s8.pi_ - s7.pi_) / (fabs(y.pi_) + fabs(s8.pi_) + 1e-300);
            err = fmax(e_phi, e_pi);
            take = e_phi <= kTol && e_pi <= kTol && !(upper && z.phi <= p.phi_T);
            if (!take) {
                m >>= 1;
                hold = kHold;
                continue;
            }
            if (lane == 0) b.rec[nrec] = MacroRec{i, i + m, upper ? 1 : 0, 0, y.phi, y.pi_};
            ++nrec;
            N += H;
        } else if (lost) {
            m = room;
            if (lane == 0) b.rec[nrec] = MacroRec{i, i + m, 0, 0, y.phi, y.pi_};
            ++nrec;
            N += (double)m * kBgStep;
        } else {
            advance(p, N, N + kBgStep, z, kBgStep);
        }
        i += m;
        y = z;
        if (lane == 0) put_sample(b, i, N, y);
        if (y.phi <= ref_phi && N_end == INFINITY) N_end = N + N_after;
        if (hold > 0) --hold;
        else if (err <= kSmooth && 2 * m <= m_max) m *= 2;
    }
    if (lane == 0) *b.end = BgEnd{i, nrec, i, INT_MAX};
}

// The samples between the strides' ends: a thread takes kFillChunk samples, reaches the first one of
// them inside a stride by one extrapolated step from the stride's start, and goes on by RK4 steps of
// kBgStep.
__global__ void __launch_bounds__(256) bg_fill_kernel(Pot p, BgStore b)
{
    const int i0 = (blockIdx.x * blockDim.x + threadIdx.x) * kFillChunk + 1;
    const int last = min(i0 + kFillChunk - 1, b.end->last - 1), nrec = b.end->nrec;
    if (i0 > last || nrec == 0) return;
    int lo = 0, hi = nrec;                    // the last stride that starts before i0
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (b.rec[mid].first < i0) lo = mid;
        else hi = mid;
    }
    MacroRec r = b.rec[lo];
    bool have = false;
    Bg y{0.0, 0.0};
    for (int i = i0; i <= last; ++i) {
        while (i >= r.last && lo + 1 < nrec && b.rec[lo + 1].first < i) {
            r = b.rec[++lo];
            have = false;
        }
        if (i <= r.first || i >= r.last) {    // a stride's end, or a single step: written already
            have = false;
            continue;
        }
        if (have || i == r.first + 1) {
            if (!have) y = Bg{r.phi, r.pi_};
            y = rk4(p, kBgStep, y, r.upper != 0);
        } else {
            y = extrapolated(p, Bg{r.phi, r.pi_}, (double)(i - r.first) * kBgStep, r.upper != 0);
        }
        have = true;
        put_sample(b, i, b.N[r.first] + (double)(i - r.first) * kBgStep, y);
    }
}

// Per sample: where the trajectory ends (the first sample below stop_phi or with eps_1 >= 1), the
// first passage of ref_phi, and the first sample at or below each phi node (first_idx, all ones
// where none is; n = 0 for time nodes).
__global__ void __launch_bounds__(256) bg_scan_kernel(BgStore b, double stop_phi, double ref_phi, double phi_lo,
                                                      double h_node, int n, int *first_idx)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i > b.end->last) return;
    const double phi = b.phi[i], pi_ = b.pi_[i];
    if (phi < stop_phi || 0.5 * pi_ * pi_ >= 1.0) atomicMin(&b.end->stop, i);
    if (i == 0) return;
    const double before = b.phi[i - 1];
    if (before > ref_phi && phi <= ref_phi) atomicMin(&b.end->ref, i);
    // nodes first reached by this sample: phi <= phi_j < before and phi_j < phi_start
    const double hi_phi = fmin(before, b.phi[0]);
    if (n == 0 || !(phi < hi_phi)) return;
    int j0 = 0, j1 = n - 1;
    if (h_node > 0.0) {   // candidate range, clamped in FP64 before the conversion
        j0 = (int)fmin(fmax(floor((phi - phi_lo) / h_node) - 1.0, 0.0), (double)n);
        j1 = (int)fmin(fmax(ceil((hi_phi - phi_lo) / h_node) + 1.0, -1.0), (double)(n - 1));
    }
    for (int j = j0; j <= j1; ++j) {
        const double pj = grid_node(phi_lo, j, h_node);
        if (phi <= pj && pj < hi_phi) atomicMin(reinterpret_cast<unsigned *>(&first_idx[j]), (unsigned)i);
    }
}

// The Bunch-Davies node of eq. (covariance_constant_nu) at phi: sqrt(Xi_phiphi), nu.  False where
// V <= 0 or nu^2 <= 0.
__device__ inline bool bd_node(const Pot &p, double sigma, double phi, double &S_bd, double &nu, double &V)
{
    double dV, d2V;
    pot_eval(p, phi, false, V, dV, d2V);
    const double nu2 = nu2_of(p, phi);
    if (!(V > 0.0) || !(nu2 > 0.0)) return false;
    nu = sqrt(nu2);
    S_bd = sqrt(V / 3.0) / (2.0 * M_PI) * (tgamma(nu) / (0.5 * sqrt(M_PI))) * pow(0.5 * sigma, 1.5 - nu);
    return true;
}

// ---------------------------------------------------------------------------
// Modes.  The mode that crosses k = sigma a H at N_sigma starts at the last sample with k >= 100 aH
// and is solved to N_sigma in P segments whose ends are samples: equal shares of the RK4 steps that
// the step rule of mode_segment_kernel asks for, with y = k/(aH) falling as e^-N from 100.
// ---------------------------------------------------------------------------
// One node's mode: status 0 none (no matching), else start sample i0 and end time Ns.
struct ModeJob {
    double Ns, k, phi_j;
    int i0, on;
};

// Fill in a job that ends at Ns, where the classical trajectory is at (phi_j, pis) with V = V(phi_j).
// Status bit 2: the mode would start before N = 0 (no job).
__device__ inline ModeJob mode_job(const Pot &p, double sigma, double phi_j, double pis, double Ns, double V,
                                   const BgStore &b, int nb, int *status)
{
    ModeJob q{Ns, sigma * exp(Ns) * sqrt(V / (3.0 - 0.5 * pis * pis)), phi_j, 0, 0};
    // start at the last sample with k >= 100 aH (aH grows while eps1 < 1)
    auto aH = [&](int ii) { return exp(b.N[ii]) * sqrt(hubble2(p, b.phi[ii], b.pi_[ii])); };
    if (q.k < kStartRatio * aH(0)) {
        atomicOr(status, 2);
        return q;
    }
    int lo = 0, hi = nb;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (q.k < kStartRatio * aH(mid)) hi = mid;
        else lo = mid;
    }
    q.i0 = lo;
    q.on = 1;
    return q;
}

// RK4 steps of the step rule over the first tau e-folds of a mode (a load estimate), and its inverse.
constexpr double kStepsPerRad = kStepsPerPeriod / (2.0 * M_PI);
__device__ inline double mode_cost(double tau)
{
    const double tau1 = log(kStartRatio * kStepsPerRad * kModeMaxStep);   // the step reaches kModeMaxStep
    const double t = fmin(tau, tau1);
    return kStepsPerRad * kStartRatio * (1.0 - exp(-t)) + (tau - t) / kModeMaxStep;
}

__device__ inline double mode_cost_inv(double c)
{
    const double tau1 = log(kStartRatio * kStepsPerRad * kModeMaxStep);
    const double c1 = mode_cost(tau1);
    return c < c1 ? -log(1.0 - c / (kStepsPerRad * kStartRatio)) : tau1 + (c - c1) * kModeMaxStep;
}

// Sample at which segment s of P begins (INT_MAX: at Ns itself, an empty segment).  A sample next to
// a downward passage of the kink moves past it, so that the passage lies well inside one segment
// whatever the last bits of the two segments' own backgrounds are.
__device__ inline int segment_start(const Pot &p, const ModeJob &q, const BgStore &b, int s, int P)
{
    if (s <= 0) return q.i0;
    if (s >= P) return INT_MAX;
    const double tau = q.Ns - b.N[q.i0];
    const double c = mode_cost(tau) * (double)s / (double)P;
    int i = q.i0 + (int)rint(fmin(mode_cost_inv(c), tau) / kBgStep);
    if (p.kind == kPotPiecewiseLinear && i > 0) {
        const int top = b.end->last;
        const double at = b.phi[min(i, top)];
        if (b.phi[min(i, top) - 1] > p.phi_T && at <= p.phi_T) i += 1;
        else if (at > p.phi_T && b.phi[min(i + 1, top)] <= p.phi_T) i += 2;
    }
    return (i > b.end->last || !(b.N[min(i, b.end->last)] < q.Ns)) ? INT_MAX : i;
}

// Background (phi, pi), the mode dphi = (fr, fi) and d dphi/dN = (gr, gi).
struct St {
    double phi, pi_, fr, fi, gr, gi;
};

__device__ inline St axpy(const St &s, const St &k, double c)
{
    return St{s.phi + c * k.phi, s.pi_ + c * k.pi_, s.fr + c * k.fr, s.fi + c * k.fi, s.gr + c * k.gr,
              s.gi + c * k.gi};
}

// The time derivative of background and mode with E = k^2 e^(-2N) given: deriv's, and eq. (full_delta_phi) over
// H^2, whose last term, a^-3 d/dt(a^3 phidot^2/H), is H^2 (pi^2 (3 - eps1) + 2 pi dpi/dN), with one reciprocal in
// place of the divisions.  w = q/V = 1/H^2.
__device__ __forceinline__ St mode_deriv(const Pot &p, double E, const St &s, bool upper, double &w)
{
    double V, dV, d2V;
    pot_eval(p, s.phi, upper, V, dV, d2V);
    const double iV = recip(V);
    const double q = 3.0 - 0.5 * s.pi_ * s.pi_;
    const double dpi = -q * (s.pi_ + dV * iV);
    w = q * iV;
    const double m2 = (E + d2V) * w - s.pi_ * (s.pi_ * q + 2.0 * dpi);
    return St{s.pi_, dpi, s.gr, s.gi, -q * s.gr - m2 * s.fr, -q * s.gi - m2 * s.fi};
}

// One RK4 step of h <= kModeMaxStep from the derivative k1 at its start; E0, E1, E2 are E at its
// start, middle and end.
__device__ __forceinline__ St mode_rk4(const Pot &p, double E1, double E2, double h, const St &s, const St &k1,
                                       bool upper)
{
    double w;
    const St k2 = mode_deriv(p, E1, axpy(s, k1, 0.5 * h), upper, w);
    const St k3 = mode_deriv(p, E1, axpy(s, k2, 0.5 * h), upper, w);
    const St k4 = mode_deriv(p, E2, axpy(s, k3, h), upper, w);
    const double c = h * (1.0 / 6.0);
    return St{s.phi + c * (k1.phi + 2.0 * (k2.phi + k3.phi) + k4.phi),
              s.pi_ + c * (k1.pi_ + 2.0 * (k2.pi_ + k3.pi_) + k4.pi_),
              s.fr + c * (k1.fr + 2.0 * (k2.fr + k3.fr) + k4.fr), s.fi + c * (k1.fi + 2.0 * (k2.fi + k3.fi) + k4.fi),
              s.gr + c * (k1.gr + 2.0 * (k2.gr + k3.gr) + k4.gr), s.gi + c * (k1.gi + 2.0 * (k2.gi + k3.gi) + k4.gi)};
}

// The propagator of one segment of one mode: the solutions that start as (f, g) = (1, 0) and (0, 1),
// carried as the real and imaginary parts of one state.  RK4 steps of at most kModeMaxStep and at most 1/800
// of the mode's period 2 pi aH/k; the step that takes phi over the kink of the piecewise-linear potential ends
// on it, where the delta function (A_+ - A_-) delta(phi - phi_T) in V'' adds -(A_+ - A_-) dphi/(H^2 |pi|) to
// d dphi/dN, and phi continues one ulp below phi_T.
// E = k^2 e^(-2N) is carried along by the series of e^(-x) (at the step's middle x = h, at its end x = 2 h <=
// 5e-4: x^5/120 < 3e-19).
// Node j, segment s is thread s n + j, so that a wave's lanes hold neighbouring nodes in the same
// segment and step alike.
// One thread per mode left 64 waves on the chip, each a chain of 2.3e4 steps: 25.0 ms for 4096 nodes.
// Split over 64 segments the solve is bound by FP64 issue (about 150 operations a step): 0.64 ms.
template <int KIND>
__global__ void __launch_bounds__(256) mode_segment_kernel(Pot pot, int n, int P, const ModeJob *jobs, BgStore b,
                                                           double4 *prop)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n * P) return;
    const int j = t % n, seg = t / n;
    Pot p = pot;
    p.kind = KIND;
    const ModeJob q = jobs[j];
    if (!q.on) return;
    St s{0.0, 0.0, 1.0, 0.0, 0.0, 1.0};
    const int ia = segment_start(p, q, b, seg, P), ib = segment_start(p, q, b, seg + 1, P);
    if (ia != INT_MAX) {
        double N = b.N[ia];
        const double N_stop = ib == INT_MAX ? q.Ns : b.N[ib];
        s.phi = b.phi[ia];
        s.pi_ = b.pi_[ia];
        const bool has_kink = KIND == kPotPiecewiseLinear && q.phi_j < p.phi_T;
        double E = q.k * q.k * exp(-2.0 * N);
        while (N < N_stop) {
            double w;
            St k1 = mode_deriv(p, E, s, false, w);
            // (the floor of 1e-6 e-folds is below any step of a regular mode and ends the loop for one that is not)
            const double h_rule = (1.0 / kStepsPerRad) * __builtin_amdgcn_rsq(E * w);
            const double h = fmin(fmin(kModeMaxStep, N_stop - N), fmax(h_rule, 1e-6));
            auto decay = [](double x) {
                return fma(x, fma(x, fma(x, fma(x, 1.0 / 24.0, -1.0 / 6.0), 0.5), -1.0), 1.0);
            };
            double e1 = decay(h), e2 = decay(2.0 * h);
            const St u = mode_rk4(p, E * e1, E * e2, h, s, k1, false);
            if (!(has_kink && s.phi > p.phi_T && u.phi <= p.phi_T)) {
                s = u;
                N += h;
                E *= e2;
                continue;
            }
            // the step that crosses the kink ends on it: Newton on its length from the chord (phi is
            // nearly straight over 2.5e-4 e-folds, so four steps reach the rounding; the lanes of a wave
            // cross at steps of their own, so this part runs once per lane and a bisection's 256
            // evaluations there took three quarters of the kernel)
            const Bg s0{s.phi, s.pi_};
            double hi = h * (s.phi - p.phi_T) / (s.phi - u.phi);
            for (int it = 0; it < 4; ++it) {
                const Bg v = rk4(p, hi, s0, true);
                hi = fmin(fmax(hi - (v.phi - p.phi_T) / v.pi_, 0.0), h);
            }
            e1 = decay(hi);
            e2 = decay(2.0 * hi);
            k1 = mode_deriv(p, E, s, true, w);
            s = mode_rk4(p, E * e1, E * e2, hi, s, k1, true);
            N += hi;
            E *= e2;
            double V, dV, d2V;
            pot_eval(p, p.phi_T, true, V, dV, d2V);
            const double H2 = V / (3.0 - 0.5 * s.pi_ * s.pi_);
            const double kick = -(p.Ap - p.Am) / (H2 * fabs(s.pi_));
            s.gr += kick * s.fr;
            s.gi += kick * s.fi;
            s.phi = nextafter(p.phi_T, -INFINITY);
        }
    }
    prop[(size_t)seg * n + j] = make_double4(s.fr, s.gr, s.fi, s.gi);
}

// 4|B_k|^2/pi of a solved mode with nu = nu(phi_j).  Status bit 4: non-finite or zero B_k (NaN).
__device__ double matched_factor(const Pot &p, double sigma, const ModeJob &q, double nu, const BgStore &b,
                                 const double4 *prop, int n, int P, int *status)
{
    const double N = b.N[q.i0], k = q.k;
    double fr, fi, gr, gi;
    {
        // Bunch-Davies: e^(iy)(1 + i c/y)/(a sqrt(2k)), c = (4 nu^2 - 1)/8, y = k/(aH), overall phase
        // dropped; d/dN of it is [(-1 - iy)(1 + ic/y) + ic/y]/(a sqrt(2k))
        const double a = exp(N);
        const double y = k / (a * sqrt(hubble2(p, b.phi[q.i0], b.pi_[q.i0])));
        const double c = (4.0 * nu2_of(p, b.phi[q.i0]) - 1.0) * 0.125;
        const double amp = 1.0 / (a * sqrt(2.0 * k));
        fr = amp;
        fi = amp * c / y;
        gr = amp * (-1.0 + c);        // Re[(-1 - iy)(1 + ic/y) + ic/y]
        gi = amp * (-y);              // Im[...] = -c/y - y + c/y
    }
#pragma unroll 4
    for (int s = 0; s < P; ++s) {
        const double4 m = prop[(size_t)s * n];          // columns (x, y) of f, (z, w) of g
        const double r0 = m.x * fr + m.z * gr, r1 = m.y * fr + m.w * gr;
        const double i0 = m.x * fi + m.z * gi, i1 = m.y * fi + m.w * gi;
        fr = r0;
        gr = r1;
        fi = i0;
        gi = i1;
    }
    // eq. (bessel_matching) at -k eta = sigma with nu(phi_j); a/sqrt(-eta) = e^N sqrt(k/sigma).  The
    // denominator J_nu dY_nu/dN - Y_nu dJ_nu/dN is -y W[J_nu, Y_nu](y) = -2/pi (the Bessel Wronskian),
    // so B_k = (pi/2) pref (dphi dJ/dN - g J) with g = 3/2 dphi + d dphi/dN, for every nu > 0.
    double Jn, yJn;
    bessel_j(nu, sigma, Jn, yJn);
    const double dJ = -yJn;
    const double pref = exp(q.Ns) * sqrt(k / sigma);
    const double g_r = 1.5 * fr + gr, g_i = 1.5 * fi + gi;
    const double b_r = 0.5 * M_PI * pref * (fr * dJ - g_r * Jn);
    const double b_i = 0.5 * M_PI * pref * (fi * dJ - g_i * Jn);
    const double fac = 4.0 * (b_r * b_r + b_i * b_i) / M_PI;
    if (!(fac > 0.0) || !isfinite(fac)) {
        atomicOr(status, 4);
        return NAN;
    }
    return fac;
}

// The time at which phi(N) reaches target inside samples [i-1, i]: Newton on the cubic Hermite
// interpolant of phi; pi there interpolated linearly.
__device__ inline void hermite_root(const double *bN, const double *bphi, const double *bpi, int i, double target,
                                    double &Ns, double &pis)
{
    const double dn = bN[i] - bN[i - 1];
    const double p0 = bphi[i - 1], p1 = bphi[i], m0 = bpi[i - 1] * dn, m1 = bpi[i] * dn;
    double t = (p0 - target) / (p0 - p1);
    for (int it = 0; it < 50; ++it) {
        const double t2 = t * t, t3 = t2 * t;
        const double v = (2.0 * t3 - 3.0 * t2 + 1.0) * p0 + (t3 - 2.0 * t2 + t) * m0 + (3.0 * t2 - 2.0 * t3) * p1 +
                         (t3 - t2) * m1 - target;
        const double dv = 6.0 * (t2 - t) * (p0 - p1) + (3.0 * t2 - 4.0 * t + 1.0) * m0 + (3.0 * t2 - 2.0 * t) * m1;
        const double step = v / dv;
        t -= step;
        if (fabs(step) < 1e-16) break;
    }
    Ns = bN[i - 1] + t * dn;
    pis = bpi[i - 1] + t * (bpi[i] - bpi[i - 1]);
}

// Samples that belong to the trajectory: up to the first one at which it ended.
__device__ inline int bg_count(const BgStore &b) { return min(b.end->last, b.end->stop) + 1; }

// The phi nodes: Bunch-Davies noise, the crossing time and the mode's job.
__global__ void match_node_kernel(Pot p, double sigma, int n, double phi_lo, double h_node, BgStore b,
                                  const int *first_idx, double *S, double *tan_out, double *fac_out, ModeJob *jobs,
                                  int *status)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    const double phi_j = grid_node(phi_lo, j, h_node);
    jobs[j].on = 0;
    double S_bd, nu, V;
    if (!bd_node(p, sigma, phi_j, S_bd, nu, V)) {
        atomicOr(status, 1);
        S[j] = tan_out[j] = fac_out[j] = 0.0;
        return;
    }
    tan_out[j] = nu - 1.5;
    S[j] = S_bd;
    fac_out[j] = 1.0;
    const int i = first_idx[j], nb = bg_count(b);
    if (i > 0 && i < nb) {
        double Ns, pis;
        hermite_root(b.N, b.phi, b.pi_, i, phi_j, Ns, pis);
        jobs[j] = mode_job(p, sigma, phi_j, pis, Ns, V, b, nb, status);
        if (!jobs[j].on) S[j] = fac_out[j] = NAN;
    }
}

// Nodes with a solved mode: the factor, and the noise scaled by it.
__global__ void match_finish_kernel(Pot p, double sigma, int n, const ModeJob *jobs, BgStore b, const double4 *prop,
                                    int P, double *S, const double *tan_out, double *fac_out, int *status)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n || !jobs[j].on) return;
    const double fac = matched_factor(p, sigma, jobs[j], tan_out[j] + 1.5, b, prop + j, n, P, status);
    fac_out[j] = fac;
    S[j] *= sqrt(fac);
}

// The time at which the trajectory passes phi_ref (NaN if it does not).
__device__ inline double ref_time(const BgStore &b, double phi_ref)
{
    const int i = b.end->ref;
    if (i >= bg_count(b)) return NAN;
    double N_ref, pr;
    hermite_root(b.N, b.phi, b.pi_, i, phi_ref, N_ref, pr);
    return N_ref;
}

// The trajectory at N_sigma = N_ref + tau (tau = t_lo + j h, formed without a fused multiply-add):
// phi by the cubic Hermite interpolant of the samples, pi linearly; tau = 0 is the reference point,
// phi_ref exactly (on a kink at phi_ref, the branch before it).  False where the trajectory does
// not pass phi_ref (N_ref NaN) or N_sigma lies outside the followed samples.
__device__ inline bool time_node(double t_lo, int j, double h, double phi_ref, const double *bN, const double *bphi,
                                 const double *bpi, int nb, double N_ref, double &Ns, double &phi_j, double &pi_j)
{
    const double tau = grid_node(t_lo, j, h);
    Ns = N_ref + tau;
    if (!(Ns >= bN[0]) || !(Ns <= bN[nb - 1]) || nb < 2) return false;
    // first sample at or after Ns (from 1, at most nb - 1)
    int lo = 0, hi = nb - 1;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (bN[mid] < Ns) lo = mid;
        else hi = mid;
    }
    const int i = hi;
    const double dn = bN[i] - bN[i - 1], t = (Ns - bN[i - 1]) / dn;
    const double t2 = t * t, t3 = t2 * t;
    phi_j = tau == 0.0 ? phi_ref
                       : (2.0 * t3 - 3.0 * t2 + 1.0) * bphi[i - 1] + (t3 - 2.0 * t2 + t) * bpi[i - 1] * dn +
                             (3.0 * t2 - 2.0 * t3) * bphi[i] + (t3 - t2) * bpi[i] * dn;
    pi_j = bpi[i - 1] + t * (bpi[i] - bpi[i - 1]);
    return true;
}

// Node j at N_sigma = N_ref + t_lo + j h: the trajectory's phi_j and pi_j there (time_node), the
// Bunch-Davies node and the mode's job.  Status 16: the trajectory does not pass phi_ref, or the node
// lies outside the followed trajectory.
__global__ void match_node_time_kernel(Pot p, double sigma, int n, double t_lo, double h, double phi_ref, BgStore b,
                                       double *S, double *tan_out, double *fac_out, double *phi_out, ModeJob *jobs,
                                       int *status)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    const int nb = bg_count(b);
    jobs[j].on = 0;
    S[j] = tan_out[j] = fac_out[j] = phi_out[j] = NAN;
    double Ns, phi_j, pi_j;
    if (!time_node(t_lo, j, h, phi_ref, b.N, b.phi, b.pi_, nb, ref_time(b, phi_ref), Ns, phi_j, pi_j)) {
        atomicOr(status, 16);
        return;
    }
    phi_out[j] = phi_j;
    double S_bd, nu, V;
    if (!bd_node(p, sigma, phi_j, S_bd, nu, V)) {
        atomicOr(status, 1);
        return;
    }
    tan_out[j] = nu - 1.5;
    jobs[j] = mode_job(p, sigma, phi_j, pi_j, Ns, V, b, nb, status);
    if (jobs[j].on) S[j] = S_bd;
}

// 2D node j in time: the covariance of noise_node.hpp at the trajectory's phi there.  Status 16 as
// above, 1 where the covariance rejects the node.
__global__ void bessel2d_time_node_kernel(Pot p, double sigma, int n, double t_lo, double h, double phi_ref, BgStore b,
                                          double *Xpp, double *Xpq, double *Xqq, double *phi_out, int *status)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    Xpp[j] = Xpq[j] = Xqq[j] = phi_out[j] = NAN;
    double Ns, phi_j, pi_j;
    if (!time_node(t_lo, j, h, phi_ref, b.N, b.phi, b.pi_, bg_count(b), ref_time(b, phi_ref), Ns, phi_j, pi_j)) {
        atomicOr(status, 16);
        return;
    }
    phi_out[j] = phi_j;
    if (!bessel2d_node(p, sigma, phi_j, Xpp[j], Xpq[j], Xqq[j])) atomicOr(status, 1);
}

// The trajectory's part of the scratch memory.
BgStore carve_bg(void *scratch, size_t &off)
{
    unsigned char *base = static_cast<unsigned char *>(scratch);
    BgStore b;
    b.N = reinterpret_cast<double *>(base);
    b.phi = b.N + kMatchCap;
    b.pi_ = b.phi + kMatchCap;
    b.rec = reinterpret_cast<MacroRec *>(b.pi_ + kMatchCap);
    b.end = reinterpret_cast<BgEnd *>(b.rec + kMacroCap);
    off = (size_t)kMatchCap * 3 * sizeof(double) + (size_t)kMacroCap * sizeof(MacroRec) + 256;
    return b;
}

hipError_t bg_launch(const PotParams &p, double phi_start, double pi_start, double stop_phi, double ref_phi,
                     double N_after, const BgStore &b, double phi_lo, double h_node, int n, int *first_idx,
                     hipStream_t stream)
{
    auto macro = p.kind == kPotPiecewiseLinear ? bg_macro_kernel<kPotPiecewiseLinear>
                 : p.kind == kPotExponential   ? bg_macro_kernel<kPotExponential>
                                               : bg_macro_kernel<kPotGaussianBump>;
    hipLaunchKernelGGL(macro, dim3(1), dim3(64), 0, stream, p, phi_start, pi_start, stop_phi, ref_phi, N_after,
                       b);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // the sample count is on the device: grids for the longest trajectory, whose excess blocks end at once
    const int most = kBgLast + 1;
    const int per_block = 256 * kFillChunk;
    hipLaunchKernelGGL(bg_fill_kernel, dim3((most + per_block - 1) / per_block), dim3(256), 0, stream, p, b);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(bg_scan_kernel, dim3((most + 255) / 256), dim3(256), 0, stream, b, stop_phi, ref_phi, phi_lo,
                       h_node, n, first_idx);
    return hipGetLastError();
}

// Segments per mode: 64 give four waves on each SIMD at 4096 nodes; fewer nodes take more segments, up
// to 256, where some 90 steps are left and a segment's set-up (two logarithms, two searches) shows.
int mode_segments(int n)
{
    int P = 64;
    while (P < 256 && (size_t)n * P < (size_t)1 << 18) P *= 2;
    return P;
}

hipError_t mode_launch(const PotParams &p, int n, int P, const ModeJob *jobs, const BgStore &b, double4 *prop,
                       hipStream_t stream)
{
    const dim3 grid((unsigned)(((size_t)n * P + 255) / 256)), block(256);
    if (p.kind == kPotPiecewiseLinear)
        hipLaunchKernelGGL(mode_segment_kernel<kPotPiecewiseLinear>, grid, block, 0, stream, p, n, P, jobs, b, prop);
    else if (p.kind == kPotExponential)
        hipLaunchKernelGGL(mode_segment_kernel<kPotExponential>, grid, block, 0, stream, p, n, P, jobs, b, prop);
    else
        hipLaunchKernelGGL(mode_segment_kernel<kPotGaussianBump>, grid, block, 0, stream, p, n, P, jobs, b, prop);
    return hipGetLastError();
}

}  // namespace

size_t matched_scratch_bytes(int n)
{
    size_t off;
    (void)carve_bg(nullptr, off);
    return off + (size_t)n * (sizeof(ModeJob) + sizeof(double4) * mode_segments(n) + sizeof(int)) + 256;
}

hipError_t matched_table_launch(const PotParams &p, double sigma, int n, double phi_lo, double h_node,
                                double phi_start, double pi_start, void *scratch, double *d_S, double *d_tan,
                                double *d_fac, int *d_status, hipStream_t stream)
{
    size_t off;
    const BgStore b = carve_bg(scratch, off);
    const int P = mode_segments(n);
    double4 *prop = reinterpret_cast<double4 *>(static_cast<unsigned char *>(scratch) + off);
    ModeJob *jobs = reinterpret_cast<ModeJob *>(prop + (size_t)n * P);
    int *first_idx = reinterpret_cast<int *>(jobs + n);
    hipError_t e = hipMemsetAsync(first_idx, 0xff, sizeof(int) * n, stream);   // -1: not reached
    if (e != hipSuccess) return e;
    e = bg_launch(p, phi_start, pi_start, phi_lo, -INFINITY, 0.0, b, phi_lo, h_node, n, first_idx, stream);
    if (e != hipSuccess) return e;
    const dim3 grid((n + 63) / 64), block(64);
    hipLaunchKernelGGL(match_node_kernel, grid, block, 0, stream, p, sigma, n, phi_lo, h_node, b, first_idx, d_S,
                       d_tan, d_fac, jobs, d_status);
    e = hipGetLastError();
    if (e == hipSuccess) e = mode_launch(p, n, P, jobs, b, prop, stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(match_finish_kernel, grid, block, 0, stream, p, sigma, n, jobs, b, prop, P, d_S, d_tan, d_fac,
                       d_status);
    return hipGetLastError();
}

hipError_t matched_time_launch(const PotParams &p, double sigma, int n, double t_lo, double h, double phi_start,
                               double pi_start, double phi_ref, double N_after, void *scratch, double *d_S,
                               double *d_tan, double *d_fac, double *d_phi, int *d_status, hipStream_t stream)
{
    size_t off;
    const BgStore b = carve_bg(scratch, off);
    const int P = mode_segments(n);
    double4 *prop = reinterpret_cast<double4 *>(static_cast<unsigned char *>(scratch) + off);
    ModeJob *jobs = reinterpret_cast<ModeJob *>(prop + (size_t)n * P);
    hipError_t e = bg_launch(p, phi_start, pi_start, -INFINITY, phi_ref, N_after, b, 0.0, 0.0, 0, nullptr, stream);
    if (e != hipSuccess) return e;
    const dim3 grid((n + 63) / 64), block(64);
    hipLaunchKernelGGL(match_node_time_kernel, grid, block, 0, stream, p, sigma, n, t_lo, h, phi_ref, b, d_S, d_tan,
                       d_fac, d_phi, jobs, d_status);
    e = hipGetLastError();
    if (e == hipSuccess) e = mode_launch(p, n, P, jobs, b, prop, stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(match_finish_kernel, grid, block, 0, stream, p, sigma, n, jobs, b, prop, P, d_S, d_tan, d_fac,
                       d_status);
    return hipGetLastError();
}

size_t bessel2d_time_scratch_bytes()
{
    size_t off;
    (void)carve_bg(nullptr, off);
    return off;
}

hipError_t bessel2d_time_launch(const PotParams &p, double sigma, int n, double t_lo, double h, double phi_start,
                                double pi_start, double phi_ref, double N_after, void *scratch, double *d_Xpp,
                                double *d_Xpq, double *d_Xqq, double *d_phi, int *d_status, hipStream_t stream)
{
    size_t off;
    const BgStore b = carve_bg(scratch, off);
    hipError_t e = bg_launch(p, phi_start, pi_start, -INFINITY, phi_ref, N_after, b, 0.0, 0.0, 0, nullptr, stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(bessel2d_time_node_kernel, dim3((n + 63) / 64), dim3(64), 0, stream, p, sigma, n, t_lo, h,
                       phi_ref, b, d_Xpp, d_Xpq, d_Xqq, d_phi, d_status);
    return hipGetLastError();
}

}  // namespace fpt
