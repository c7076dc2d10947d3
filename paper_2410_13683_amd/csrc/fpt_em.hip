// fpt_em.hip -- Euler-Maruyama first-passage kernels for gfx950.
//
// One lane integrates one trajectory of the 1D-noise Langevin system in
// (phi, pi = dphi/dN) (arXiv:2410.13683, Sec. 4.1, eqs. stochastic_eom_1D and
// importance_sampling_1D_noise_step) with a bias parallel to the noise,
// B = a S (1, tan theta_n) (eq. 2D_1D_noise_diussion_based_bias), and
// accumulates ln w = -sum dA (eqs. weight, weight_A restricted to the noise
// direction: dA = a xi sqrt(dN) + a^2 dN / 2 where S > 0).  A trajectory stops
// at its first passage through phi_end; N is interpolated linearly in phi over
// the crossing step.  deltaN = N - N_ref goes into a per-block LDS histogram
// that is flushed to global memory with atomics when the block ends.
//
// Work distribution: a persistent grid; each wave claims trajectories from a
// global cursor with one atomic per refill (ballot + popcount + mbcnt), runs
// `chunk` steps, retires the lanes whose trajectory ended, and refills them.
// New trajectories only start at chunk boundaries and a chunk is a whole number
// of step groups (FP64: 4 steps, 2 with 2D noise; FP32: 16, except the kernel
// that evaluates the network in the step, 4; a chunk is rounded up to a whole
// group), so every active lane of a wave is at the same step modulo the group
// length and each Philox call (four steps of 1D noise, two of 2D noise) is
// taken by the whole wave at once.
//
// Random numbers: Philox4x32-10 (Salmon et al., SC'11), key = seed, counter =
// (traj lo, n >> 2, traj hi, instance); u = (w + 1/2) 2^-32; Box-Muller pairs
// (u0, u1) -> steps 4m, 4m+1 and (u2, u3) -> steps 4m+2, 4m+3.
//
// Two state precisions: FP64 (phi, pi, ln w in double) and FP32 state (the
// distance x = phi - phi_end and pi each held as an unevaluated pair of floats
// hi + lo, increments computed in FP32 from the hi parts, uniforms
// fl32(w) 2^-32 + 2^-33 and hardware sin/cos/log; ln w, the crossing
// interpolation and the histogram stay FP64).
#include "internal.hpp"

#include <hip/hip_runtime.h>
#include <math.h>

#include <type_traits>

// Optional register budget for the Euler-Maruyama kernels (waves per SIMD the
// compiler must leave room for); unset = the compiler's choice.
#ifdef FPT_EM_WAVES_PER_EU
#define FPT_EM_OCCUPANCY __attribute__((amdgpu_waves_per_eu(FPT_EM_WAVES_PER_EU)))
#else
#define FPT_EM_OCCUPANCY
#endif

namespace fpt {
namespace {

constexpr uint32_t kPhiloxM0 = 0xD2511F53u, kPhiloxM1 = 0xCD9E8D57u;
constexpr uint32_t kPhiloxW0 = 0x9E3779B9u, kPhiloxW1 = 0xBB67AE85u;

// a ^ b ^ c in one instruction: gfx950's three-input bitwise op with the XOR
// truth table 0x96 (c is wave-uniform, the round key).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    uint32_t d;
    asm("v_bitop3_b32 %0, %1, %2, %3 bitop3:0x96" : "=v"(d) : "v"(a), "v"(b), "s"(c));
    return d;
}

// Philox4x32-10 (Salmon et al., SC'11): ten rounds on the counter (c0, c1, c2, c3) with the key
// (k0, k1); a round forms the 64-bit products M0 c0 and M1 c2 and maps the counter to
// (hi(M1 c2) ^ c1 ^ k0, lo(M1 c2), hi(M0 c0) ^ c3 ^ k1, lo(M0 c0)), then adds the Weyl
// increments (W0, W1) to the key.  Here the counter is (traj lo, m, traj hi, instance) for a fixed
// trajectory, key and instance word, and only the call index m varies.  It sits in a word that
// round 1 XORs but does not multiply, so every product that does not depend on m is a
// per-trajectory constant: both products of round 1, M1 times round 1's word 2 in round 2, and
// M0 times round 2's word 0 in round 3.  They are computed once when a lane takes a trajectory
// (philox_pre), which leaves rounds 1 to 3 two multiplies in all instead of six.
struct PhiloxPre {
    uint32_t a;     // round 1 output word 0 without m: hi(M1 thi) ^ k0 (the word is a ^ m)
    uint32_t y;     // lo(M0 tlo) ^ round 2's key word 1 (round 2 output word 2 is hi(M0 (a ^ m)) ^ y)
    uint32_t x1k;   // lo(M1 (hi(M0 tlo) ^ inst ^ k1)) ^ round 3's key word 0
    uint32_t z;     // hi(M0 x0) ^ round 3's key word 1, x0 round 2's output word 0 (constant)
    uint32_t w;     // lo(M0 x0): round 3 output word 3
};

__device__ __forceinline__ PhiloxPre philox_pre(uint64_t traj, uint32_t inst, uint32_t k0, uint32_t k1)
{
    const uint64_t p = (uint64_t)kPhiloxM0 * (uint32_t)traj;            // round 1: M0 c0
    const uint64_t q = (uint64_t)kPhiloxM1 * (uint32_t)(traj >> 32);    // round 1: M1 c2
    PhiloxPre r;
    r.a = (uint32_t)(q >> 32) ^ k0;
    const uint32_t d = (uint32_t)(p >> 32) ^ inst ^ k1;                 // round 1 output word 2
    r.y = (uint32_t)p ^ (k1 + kPhiloxW1);
    const uint64_t q2 = (uint64_t)kPhiloxM1 * d;                        // round 2: M1 c2
    const uint32_t x0 = (uint32_t)(q2 >> 32) ^ (uint32_t)q ^ (k0 + kPhiloxW0);
    r.x1k = (uint32_t)q2 ^ (k0 + 2u * kPhiloxW0);
    const uint64_t p3 = (uint64_t)kPhiloxM0 * x0;                       // round 3: M0 c0
    r.z = (uint32_t)(p3 >> 32) ^ (k1 + 2u * kPhiloxW1);
    r.w = (uint32_t)p3;
    return r;
}

// The four output words for call m from the trajectory's PhiloxPre.
__device__ __forceinline__ void philox_call(uint32_t m, const PhiloxPre &q, uint32_t k0, uint32_t k1, uint32_t w[4])
{
    // round 2: M0 (a ^ m); words 0 and 1 are per-trajectory constants
    const uint64_t p2 = (uint64_t)kPhiloxM0 * (q.a ^ m);
    const uint32_t v2 = (uint32_t)(p2 >> 32) ^ q.y;
    const uint32_t v3 = (uint32_t)p2;
    // round 3: M1 v2; M0 times the constant word 0 is precomputed
    const uint64_t q3 = (uint64_t)kPhiloxM1 * v2;
    uint32_t d0 = (uint32_t)(q3 >> 32) ^ q.x1k;
    uint32_t d1 = (uint32_t)q3;
    uint32_t d2 = q.z ^ v3;
    uint32_t d3 = q.w;
    k0 += 3u * kPhiloxW0;
    k1 += 3u * kPhiloxW1;
    // rounds 4 .. 10
#pragma unroll
    for (int r = 3; r < 10; ++r) {
        const uint64_t a = (uint64_t)kPhiloxM0 * d0;
        const uint64_t b = (uint64_t)kPhiloxM1 * d2;
        const uint32_t n0 = xor3((uint32_t)(b >> 32), d1, k0);
        const uint32_t n2 = xor3((uint32_t)(a >> 32), d3, k1);
        d1 = (uint32_t)b;
        d3 = (uint32_t)a;
        d0 = n0;
        d2 = n2;
        k0 += kPhiloxW0;
        k1 += kPhiloxW1;
    }
    w[0] = d0; w[1] = d1; w[2] = d2; w[3] = d3;
}

// Box-Muller in FP64 on uniforms u = (w + 1/2) 2^-32 (exact in double), table-driven: two
// 256-entry tables in LDS (kBmBytes, staged once per block by stage_bm) replace the library
// log and sincos, each by a table read and a short series.
//   ln u:  u = m 2^e, m in [0.5, 1).  Bucket i (top 8 fraction bits of m) has centre c_i
//          (c_255 = 1, so that u near 1 loses nothing to cancellation), r_i = fl(1/c_i) and
//          L_i = -ln r_i.  Then ln m = L_i + ln(1 + t), t = m r_i - 1, |t| <= 2^-9, and the
//          series to t^5 leaves t^6/6 < 1e-17.
//   2 pi u: (2 w + 1) 2^-33 = (j + 1/2)/256 + d 2^-33, j = w >> 24, d = 2 (w mod 2^24) + 1 - 2^24
//          (an exact integer, |d| < 2^24).  sin and cos of A_j = 2 pi (j + 1/2)/256 come from
//          the table; theta = 2 pi d 2^-33 (|theta| <= pi/256) from series to theta^5 and
//          theta^6 (errors < 1e-17 and < 2e-23), and the angle-addition formulas combine them.
// Both stay far below what per-trajectory agreement to 1e-9 with an FP64 reference needs
// (normals to ~1e-9): the series stop where the next term is below 1e-17.
// VALU issue bounds it, so powers of two are folded where that leaves every bit as it is: the factor -2 of
// sqrt(-2 ln u) into the table and the series, 2^-32 into the exponent, the angle's integer formed in the
// top bits of a word (four operations fewer per pair; 1e4 trajectories of the linear problem 0.89 -> 0.86
// ms, 65,536 of slow roll -> ultra-slow roll 17.3 -> 16.7, 1e6 183.7 -> 182.0).
// Returns xi sqrt(dN) for the two steps of the pair.
constexpr int kBmN = 256;
constexpr size_t kBmBytes = 2 * kBmN * sizeof(double2);

// l_bm[j] = (sin A_j, cos A_j); l_bm[kBmN + i] = (r_i, -2 L_i)
__device__ __forceinline__ void stage_bm(double2 *l_bm)
{
    for (int i = threadIdx.x; i < 2 * kBmN; i += blockDim.x) {
        if (i < kBmN) {
            double sn, cs;
            sincospi((i + 0.5) * (1.0 / 128.0), &sn, &cs);
            l_bm[i] = make_double2(sn, cs);
        } else {
            const int k = i - kBmN;
            const double c = (k == kBmN - 1) ? 1.0 : 0.5 * (1.0 + (k + 0.5) * (1.0 / 256.0));
            const double r = 1.0 / c;
            l_bm[i] = make_double2(r, 2.0 * log(r));
        }
    }
}

// sqrt(x) for x in [2e-10, 50] (here -2 ln u: never 0, denormal or infinite, so the library's
// scaling and special-case tests are not needed): the hardware reciprocal square root, one
// Goldschmidt step and one residual correction, s = g + (x - g^2) h (within about an ulp).
__device__ __forceinline__ double sqrt_mid(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double r = fma(-g, h, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    return fma(fma(-g, g, x), h, g);
}

__device__ __forceinline__ void box_muller64(uint32_t wa, uint32_t wb, double sqrt_dN, const double2 *l_bm,
                                             double &za, double &zb)
{
    const double ua = (double)wa + 0.5;                      // u 2^32
    const double m = __builtin_amdgcn_frexp_mant(ua);        // [0.5, 1)
    const int e = __builtin_amdgcn_frexp_exp(ua) - 32;
    const int i = (__double2hiint(m) >> 12) & 0xff;
    const double2 lt = l_bm[kBmN + i];
    const double t = fma(m, lt.x, -1.0);
    double q = fma(t, -0.4, 0.5);
    q = fma(t, q, -2.0 / 3.0);
    q = fma(t, q, 1.0);
    q = fma(t, q, -2.0);
    const double m2ln_u = fma((double)e, -0x1.62e42fefa39efp+0, fma(t, q, lt.y));   // -2 (e ln 2 + L_i + ln(1 + t))
    const double rho = sqrt_mid(m2ln_u) * sqrt_dN;
    // 128 d as the signed integer that w's low 24 bits and a half form at the top of a word
    const int d128 = (int)(((wb << 8) | 0x80u) ^ 0x80000000u);
    const double th = (double)d128 * 0x1.921fb54442d18p-38;                       // 2 pi d 2^-33
    const double th2 = th * th;
    const double sn = th * fma(th2, fma(th2, 1.0 / 120.0, -1.0 / 6.0), 1.0);
    const double cs = fma(th2, fma(th2, fma(th2, -1.0 / 720.0, 1.0 / 24.0), -0.5), 1.0);
    const double2 sc = l_bm[wb >> 24];
    za = rho * fma(sc.y, cs, -sc.x * sn);      // cos(A + theta)
    zb = rho * fma(sc.x, cs, sc.y * sn);       // sin(A + theta)
}

// Copy a wave-uniform value into a VGPR once, so that a per-lane select between
// two such values is a v_cndmask on registers (not a load from the kernel
// arguments, and no extra moves for the scalar-operand limit).
__device__ __forceinline__ float in_vgpr(float x)
{
    float v;
    asm volatile("v_mov_b32 %0, %1" : "=v"(v) : "s"(x));
    return v;
}

__device__ __forceinline__ double in_vgpr(double x)
{
    double v;
    asm volatile("v_mov_b64 %0, %1" : "=v"(v) : "s"(x));
    return v;
}

__device__ __forceinline__ uint32_t lanes_below(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// x^2/2 rounded by itself (never part of a fused multiply-add).
__device__ __forceinline__ double half_sq(double x)
{
#pragma clang fp contract(off)
    return 0.5 * x * x;
}

// Steps left before max_steps for the wave's most advanced lane that holds a trajectory, as a
// wave-uniform value (such a lane has at most max_steps steps: a lane reaching it is censored).
// At the start of a chunk it bounds every lane's count inside the chunk (all lanes step
// together), so whether a group can reach max_steps is one scalar comparison per group.
__device__ __forceinline__ uint32_t wave_steps_left(bool has, uint32_t n, uint32_t max_steps)
{
    uint32_t v = has ? n : 0u;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, o));
    return max_steps - __builtin_amdgcn_readfirstlane(v);
}

// The table interval of coordinate x, min(max(floor(x), 0), top) for every x (0 for NaN), as an integer:
// v_cvt_u32_f64 truncates, takes negatives and NaN to 0 and saturates above.  Against the floor, two FP64
// clamps and a conversion it leaves one integer minimum and the conversion back (FP64 operations issue
// at some 5 cycles each and bound the kernel).
__device__ __forceinline__ uint32_t interval_of(double x, uint32_t top)
{
    uint32_t j;
    asm("v_cvt_u32_f64 %0, %1" : "=v"(j) : "v"(x));
    return min(j, top);
}

// Wave-aggregated claim of trajectories from the global cursor.  Must be
// reached by every lane of the wave.  Returns true in lanes that got one.
__device__ __forceinline__ bool claim(bool need, uint64_t &rel, unsigned long long *cursor, uint64_t n_traj,
                                      bool &exhausted)
{
    const uint64_t mask = __ballot(need && !exhausted);
    if (mask == 0) return false;
    const uint32_t cnt = (uint32_t)__popcll(mask);
    const int leader = __ffsll((unsigned long long)mask) - 1;
    unsigned long long base = 0;
    if ((int)__lane_id() == leader) base = atomicAdd(cursor, (unsigned long long)cnt);
    const uint32_t b_lo = (uint32_t)__shfl((int)(uint32_t)base, leader);
    const uint32_t b_hi = (uint32_t)__shfl((int)(uint32_t)(base >> 32), leader);
    const uint64_t b = ((uint64_t)b_hi << 32) | b_lo;
    if (b + cnt >= n_traj) exhausted = true;
    if (need) {
        const uint64_t me = b + lanes_below(mask);
        if (me < n_traj) {
            rel = me;
            return true;
        }
    }
    return false;
}

struct LdsAcc {
    unsigned long long *cnt;  // nb + 4
    double *sum;              // 4 nb + 4
    int nb;
};

__device__ __forceinline__ LdsAcc lds_acc(unsigned char *smem, int n_bins)
{
    LdsAcc a;
    a.nb = n_bins + 2;
    a.cnt = reinterpret_cast<unsigned long long *>(smem);
    a.sum = reinterpret_cast<double *>(a.cnt + a.nb + 4);
    return a;
}

__device__ __forceinline__ int bin_of(const HistSpec &h, double x)
{
    double t;
    if (h.bins_kind == kBinsLinear) t = (x - h.lo) * h.scale;
    else t = (x > 0.0) ? log(x / h.lo) * h.scale : -1.0;
    if (!(t >= 0.0)) return 0;
    if (t >= (double)h.n_bins) return h.n_bins + 1;
    return (int)floor(t) + 1;
}

// Where retired trajectories go: per-trajectory outputs (any may be NULL),
// the histogram layout and the block's LDS accumulators.
struct RetireTo {
    double *d_N, *d_lnw;
    uint32_t *d_steps;
    unsigned long long *cnt;
    double *sum;
    int nb;
    HistSpec hist;
};

// Retire one finished trajectory: per-trajectory outputs and LDS histogram.
__device__ __forceinline__ void retire(const RetireTo &t, uint64_t rel, uint32_t status, uint32_t n_steps, double N,
                                       double lnw)
{
    if (t.d_N) t.d_N[rel] = N;
    if (t.d_lnw) t.d_lnw[rel] = lnw;
    if (t.d_steps) t.d_steps[rel] = n_steps | status;
    if (status & kFlagCensored) {
        atomicAdd(&t.cnt[t.nb + 0], 1ull);
    } else if (status & kFlagEndedEarly) {
        atomicAdd(&t.cnt[t.nb + 1], 1ull);
    } else {
        const int b = bin_of(t.hist, N - t.hist.N_ref);
        const double w = exp(lnw);
        atomicAdd(&t.cnt[b], 1ull);
        atomicAdd(&t.sum[b], w);
        atomicAdd(&t.sum[t.nb + b], w * w);
        atomicAdd(&t.sum[2 * t.nb + b], lnw);
        atomicAdd(&t.sum[3 * t.nb + b], lnw * lnw);
        double *tot = t.sum + 4 * t.nb;
        atomicAdd(&tot[0], w);
        atomicAdd(&tot[1], w * w);
        atomicAdd(&tot[2], w * N);
        atomicAdd(&tot[3], w * N * N);
    }
    atomicAdd(&t.cnt[t.nb + 2], (unsigned long long)n_steps);
}

__device__ __forceinline__ void zero_lds_acc(const LdsAcc &a)
{
    for (int i = threadIdx.x; i < a.nb + 4; i += blockDim.x) a.cnt[i] = 0ull;
    for (int i = threadIdx.x; i < 4 * a.nb + 4; i += blockDim.x) a.sum[i] = 0.0;
}

__device__ __forceinline__ void flush_lds_acc(const LdsAcc &a, void *global)
{
    unsigned long long *gc = reinterpret_cast<unsigned long long *>(global);
    double *gs = reinterpret_cast<double *>(gc + a.nb + 4);
    for (int i = threadIdx.x; i < a.nb + 4; i += blockDim.x)
        if (a.cnt[i]) atomicAdd(&gc[i], a.cnt[i]);
    for (int i = threadIdx.x; i < 4 * a.nb + 4; i += blockDim.x)
        if (a.sum[i] != 0.0) unsafeAtomicAdd(&gs[i], a.sum[i]);
}

// V'/V for both potentials as 1/d, d = kx phi + s with s chosen per side:
//   piecewise linear  kx = 1, s = -c_+ (phi >= phi_T) or -c_- (phi < phi_T), c_+- = phi_T - V0/A_+-
//   exponential       kx = 0, s = 1/A_+ on both sides
// (no cancellation: d = phi - c is a single rounding).
struct DriftConsts {
    double kx, s_plus, s_minus;
};

__device__ __forceinline__ DriftConsts drift_consts(const Inst &I)
{
    DriftConsts k;
    if (I.pot_kind == kPotExponential) {
        k.kx = 0.0;
        k.s_plus = k.s_minus = 1.0 / I.A_plus;
    } else {
        k.kx = 1.0;
        k.s_plus = -(I.phi_T - I.V0 / I.A_plus);
        k.s_minus = -(I.phi_T - I.V0 / I.A_minus);
    }
    return k;
}

// V'/V of the Gaussian bump, eq. (potential_swagat), as one fraction:
//   2 m^2/(phi (m^2 + phi^2)) - x g/(Sigma (1 + g)),  x = (phi - phi_0)/Sigma,  g = K e^(-x^2/2).
// In ultra-slow roll the two terms nearly cancel; the single division keeps that to one rounding
// of the numerator's difference.
struct BumpConsts {
    double phi0, m2, two_m2, inv_sig, sig, K;
};

__device__ __forceinline__ BumpConsts bump_consts(const Inst &I)
{
    return BumpConsts{I.phi_T, I.bump_m2, 2.0 * I.bump_m2, 1.0 / I.bump_Sigma, I.bump_Sigma, I.bump_K};
}

__device__ __forceinline__ double bump_dlnV(const BumpConsts &b, double phi)
{
    const double x = (phi - b.phi0) * b.inv_sig;
    const double g = b.K * exp(-0.5 * x * x);
    const double d1 = phi * fma(phi, phi, b.m2);
    const double d2 = b.sig * (1.0 + g);
    // the quotient as the hardware reciprocal of the denominator (a normal number here: phi > 0
    // away from 0, Sigma (1 + g) > 0) with one Newton step, times the numerator: about 2e-15
    // relative, where the IEEE division would spend twice the instructions on the last ulp
    const double den = d1 * d2;
    double r = __builtin_amdgcn_rcp(den);
    r = fma(r, fma(-den, r, 1.0), r);
    return (b.two_m2 * d2 - x * g * d1) * r;
}

// The table size used by the kernels: a single node (constant noise) is
// staged as two equal nodes so one lookup serves every table.
__device__ __forceinline__ int staged_nodes(const Inst &I) { return I.n_tab > 1 ? I.n_tab : 2; }

// FP64 staging: the noise nodes, then the Box-Muller tables right after them.
__device__ __forceinline__ void stage_table64(const Inst &I, double2 *l_tab)
{
    const int n = staged_nodes(I);
    for (int i = threadIdx.x; i < n; i += blockDim.x) l_tab[i] = I.tab64[I.n_tab > 1 ? i : 0];
    stage_bm(l_tab + n);
}

// FP32 staging: the noise nodes, then the V'/V intervals right after them,
// scaled by half the time step (the step uses (V'/V) dN/2); all NaN for a
// single-node table, so that V'/V is computed exactly there.
__device__ __forceinline__ void stage_table32(const Inst &I, float4 *l_tab, float dN)
{
    const int n = staged_nodes(I);
    for (int i = threadIdx.x; i < n; i += blockDim.x) l_tab[i] = I.tab32[I.n_tab > 1 ? i : 0];
    float2 *l_r = reinterpret_cast<float2 *>(l_tab + n);
    const float nan = __builtin_nanf("");
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        float2 r = make_float2(nan, nan);
        if (I.n_tab > 1) {
            r = I.rtab32[i];
            r.x *= 0.5f * dN;
            r.y *= 0.5f * dN;
        }
        l_r[i] = r;
    }
}

// ---------------------------------------------------------------------------
// Learned control, tabulated: the amplitude a(phi, pi) is the bilinear
// interpolation of the network's values on a uniform grid of the normalised
// inputs (x0, x1) = ((phi - c0)/s0, (ln max(|pi|, 1e-30) - c1)/s1), clamped to
// the edge cells.  A deterministic function of the state is an admissible
// importance-sampling control (Sec. 4.1: the bias may depend on the state as
// long as the weight uses the same bias), and the weights below use this same
// amplitude, so the estimator stays unbiased.
//
// Replay (gradient) mode: the lanes integrate listed trajectories again with
// the same control and scatter each step's factor -xi sqrt(dN) (the on-policy
// value of -(e_k - a_k dN), e_k = a_k dN + xi_k sqrt(dN)) onto the four nodes
// of the step's cell with the bilinear weights, scaled by the path's w^2.  A
// lane keeps running sums for its current cell in registers and adds them to
// the block's LDS node array when the path leaves the cell or ends.
// ---------------------------------------------------------------------------
struct GridConsts64 {
    double k0, off0, k1, off1, imax0, imax1;
    int n1c;                   // cells per row, n1 - 1
};

__device__ __forceinline__ GridConsts64 grid_consts64(const Inst &I)
{
    GridConsts64 g;
    g.k0 = I.g_k0;
    g.off0 = I.g_off0;
    g.k1 = I.g_k1;
    g.off1 = I.g_off1;
    g.imax0 = (double)(I.g_n0 - 2);
    g.imax1 = (double)(I.g_n1 - 2);
    g.n1c = I.g_n1 - 1;
    return g;
}

// a(phi, pi) from the staged cells; also the cell and the fractions inside it.
// fmin/fmax map NaN and infinite coordinates onto the edge cells, so the cell
// index stays inside the table for any state.
__device__ __forceinline__ double grid_amp64(const GridConsts64 &g, const double2 *l_grid, double phi, double pi_,
                                             int &cell, double &f0, double &f1)
{
    const double u0 = fma(phi, g.k0, g.off0);
    const double u1 = fma(log(fmax(fabs(pi_), 1e-30)), g.k1, g.off1);
    const double i0 = fmin(fmax(floor(u0), 0.0), g.imax0);
    const double i1 = fmin(fmax(floor(u1), 0.0), g.imax1);
    f0 = fmin(fmax(u0 - i0, 0.0), 1.0);
    f1 = fmin(fmax(u1 - i1, 0.0), 1.0);
    cell = (int)i0 * g.n1c + (int)i1;
    const double2 c0 = l_grid[2 * cell], c1 = l_grid[2 * cell + 1];
    const double b0 = fma(f0, c0.y - c0.x, c0.x);
    const double b1 = fma(f0, c1.y - c1.x, c1.x);
    return fma(f1, b1 - b0, b0);
}

struct GridConsts32 {
    float k0, off0;            // u0 = x k0 + off0 with x = phi - phi_end
    float k1, off1;            // u1 = log2 max(|pi|, 1e-30) k1 + off1
    float imax0, imax1;
    int n1c;
};

__device__ __forceinline__ GridConsts32 grid_consts32(const Inst &I)
{
    GridConsts32 g;
    g.k0 = (float)I.g_k0;
    g.off0 = (float)fma(I.phi_end, I.g_k0, I.g_off0);
    g.k1 = (float)(I.g_k1 * 0.69314718055994531);
    g.off1 = (float)I.g_off1;
    g.imax0 = (float)(I.g_n0 - 2);
    g.imax1 = (float)(I.g_n1 - 2);
    g.n1c = I.g_n1 - 1;
    return g;
}

__device__ __forceinline__ float grid_amp32(const GridConsts32 &g, const float4 *l_grid, float x, float pi_, int &cell,
                                            float &f0, float &f1)
{
    const float u0 = fmaf(x, g.k0, g.off0);
    const float u1 = fmaf(__builtin_amdgcn_logf(fmaxf(fabsf(pi_), 1e-30f)), g.k1, g.off1);
    // clamps as one three-operand median each (both coordinates are finite)
    const float i0 = __builtin_amdgcn_fmed3f(floorf(u0), 0.0f, g.imax0);
    const float i1 = __builtin_amdgcn_fmed3f(floorf(u1), 0.0f, g.imax1);
    f0 = __builtin_amdgcn_fmed3f(u0 - i0, 0.0f, 1.0f);
    f1 = __builtin_amdgcn_fmed3f(u1 - i1, 0.0f, 1.0f);
    cell = (int)i0 * g.n1c + (int)i1;
    const float4 c = l_grid[cell];
    const float b0 = fmaf(f0, c.y - c.x, c.x);
    const float b1 = fmaf(f0, c.w - c.z, c.z);
    return fmaf(f1, b1 - b0, b0);
}

// How the lanes of a kernel gather gradient factors: not at all, replaying listed paths whose weight is
// known, or recording each path's sums per visited cell while it is sampled (weighted afterwards).
enum : int { kGradNone = 0, kGradReplay = 1, kGradRecord = 2 };

// Where a replay or a recording run sends its results.
struct ReplayTo {
    const TailEntry *tail;
    double *l_G;                       // node weights of the block (LDS), n0 n1
    unsigned long long *mismatch;      // global count of replays that did not end with a passage
    RecordPool rec;                    // recording run
};

// Add a lane's running sums for `cell` (corner order (i0, i1), (i0 + 1, i1),
// (i0, i1 + 1), (i0 + 1, i1 + 1)) times ww to the LDS node weights.
template <typename T>
__device__ __forceinline__ void grad_flush(const ReplayTo &rp, int n1c, int cell, T s[4], double ww)
{
    if (cell >= 0) {
        const int k = cell + cell / n1c;          // node (i0, i1)
        const int n1 = n1c + 1;
        atomicAdd(&rp.l_G[k], ww * (double)s[0]);
        atomicAdd(&rp.l_G[k + n1], ww * (double)s[1]);
        atomicAdd(&rp.l_G[k + 1], ww * (double)s[2]);
        atomicAdd(&rp.l_G[k + n1 + 1], ww * (double)s[3]);
    }
    s[0] = s[1] = s[2] = s[3] = T(0);
}

// Append a lane's running sums for `cell` to the records of trajectory rel; k counts the path's records,
// also those beyond the pool's room (the path is then replayed).
template <typename T>
__device__ __forceinline__ void grad_record(const RecordPool &p, uint64_t rel, uint32_t &k, int cell, T s[4])
{
    if (cell >= 0) {
        if (k < p.cap) {
            const uint64_t at = rel * p.cap + k;
            T *q = static_cast<T *>(p.sums) + 4 * at;
            q[0] = s[0];
            q[1] = s[1];
            q[2] = s[2];
            q[3] = s[3];
            p.cell[at] = (uint16_t)cell;
        }
        ++k;
    }
    s[0] = s[1] = s[2] = s[3] = T(0);
}

template <typename T>
__device__ __forceinline__ void grad_add(T s[4], T c, T f0, T f1)
{
    const T p1 = c * f1, p0 = c - p1;        // c f1, c (1 - f1)
    s[0] += p0 - p0 * f0;
    s[1] += p0 * f0;
    s[2] += p1 - p1 * f0;
    s[3] += p1 * f0;
}

// ---------------------------------------------------------------------------
// Learned control, exact: output 0 of the 2 -> 64 -> 64 -> 2 tanh network itself at the
// normalised state (x0, x1), evaluated every mlp_every steps and held in between (the bias may be
// any deterministic function of the path's past states; the weights use the same amplitude, so
// the estimator stays unbiased).  Both evaluations take the network's sums in their own order.
//
// FP64 state: the parameters are staged in LDS as doubles, W2 transposed (word j 64 + i holds
// W2[i][j]), then W1, b1, b2, row 0 of W3 and b3[0]; the second layer is accumulated eight units
// at a time, each pass recomputing the 64 first-layer activations, so that a lane holds eight
// accumulators instead of 64 activations.
//
// FP32 state, kBiasMlpMatrix: the second layer, 64 x 64 for the wave's 64 states, runs on the matrix cores as 128
// v_mfma_f32_32x32x1 (two blocks of 32 states, one input unit per instruction).  Such an instruction is
// one fused multiply-add per element, rounded like v_fma_f32 (bit for bit over 8e5 elements of mixed
// scales), so the sums are those of a chain of multiply-adds in the order of the input units, two
// chains per output unit (even and odd units).  A lane holds its state's input unit as the B operand
// and output unit lane % 32 of the weights as A, staged in LDS so that one 16-byte read serves four
// instructions; W1, b1 and W3 are read in place through the constant address space (scalar loads).
// Bound: the 128 instructions take 9.6e3 cycles an evaluation (75 each measured) and the FP32 vector
// work, which does not run beside FP32 matrix instructions, some 5e3 more (256 exp2 and reciprocals at
// 8 cycles among it); 1.6e4 measured.  The 128 accumulators leave two waves per SIMD.
//
// FP32 state, kBiasMlpExact: the parameters are read in place through the constant address space.  Every
// lane of a wave reads the same word, so the loads are scalar and the 4096 multiply-adds take the weights as
// scalar operands; a lane keeps its 64 first-layer activations in registers, and four waves per SIMD fit.
// The 17.9 KB pass through the 16 KB scalar cache, whose waits leave 2e4 to 5.6e4 cycles an evaluation: 1e5
// trajectories at k = 16 take 238 ms against 104 on the matrix cores, 1000 (one wave per SIMD) 147 and 67.
// Between evaluations four waves hide more than two: 2e6 trajectories (of 2.5e4 steps) at k = 128 take 98.5 ms
// against 128, at k = 1024 84 against 120.  fpt_run chooses by the estimate of network_on_matrix.  Both add
// in the same order, bit for bit.
// tanh s = 1 - 2/(e^(2s) + 1) from the hardware exp2 and reciprocal, exactly +-1 for large |s|.
// ---------------------------------------------------------------------------
constexpr int kMlpChunk = 8;
constexpr int kMlpLdsWords = kMlpHidden * kMlpHidden + 2 * kMlpHidden + 3 * kMlpHidden + 1;
constexpr size_t kMlpLdsBytes64 = ((size_t)kMlpLdsWords * 8 + 15) / 16 * 16;

__device__ __forceinline__ void stage_mlp64(const float *params, double *l_w)
{
    constexpr int H = kMlpHidden;
    for (int k = threadIdx.x; k < kMlpLdsWords; k += blockDim.x) {
        int src;
        if (k < H * H) {
            src = kOffW2 + (k % H) * H + k / H;       // word j H + i <- W2[i][j]
        } else {
            const int r = k - H * H;
            src = r < 2 * H ? kOffW1 + r                      // W1 [64][2]
                : r < 3 * H ? kOffB1 + (r - 2 * H)            // b1
                : r < 4 * H ? kOffB2 + (r - 3 * H)            // b2
                : r < 5 * H ? kOffW3 + (r - 4 * H)            // W3 row 0
                            : kOffB3;                         // b3[0]
        }
        l_w[k] = (double)params[src];
    }
}

__device__ __forceinline__ double mlp_out0_64(const double *l_w, double x0, double x1)
{
    constexpr int H = kMlpHidden;
    const double *W2t = l_w, *W1 = l_w + H * H, *b1 = W1 + 2 * H, *b2 = b1 + H, *W3 = b2 + H;
    double out = W3[H];
    for (int c = 0; c < H; c += kMlpChunk) {
        double acc[kMlpChunk];
#pragma unroll
        for (int i = 0; i < kMlpChunk; ++i) acc[i] = b2[c + i];
        for (int j = 0; j < H; ++j) {
            const double h = tanh(fma(W1[2 * j], x0, fma(W1[2 * j + 1], x1, b1[j])));
#pragma unroll
            for (int i = 0; i < kMlpChunk; ++i) acc[i] = fma(W2t[j * H + c + i], h, acc[i]);
        }
#pragma unroll
        for (int i = 0; i < kMlpChunk; ++i) out = fma(W3[c + i], tanh(acc[i]), out);
    }
    return out;
}

typedef __attribute__((address_space(4))) const float const_float;
typedef float float32x __attribute__((ext_vector_type(32)));

// The LDS copy of W2 and b2 for the matrix instructions: for input units 2j and 2j + 1 and r = 0..31
// the four weights (W2[r][2j], W2[r + 32][2j], W2[r][2j + 1], W2[r + 32][2j + 1]), then b2.
constexpr size_t kMlpLdsBytes32 = (size_t)(kMlpHidden * kMlpHidden + kMlpHidden) * sizeof(float);

__device__ __forceinline__ void stage_mlp32(const float *params, float *l_w)
{
    constexpr int H = kMlpHidden;
    for (int k = threadIdx.x; k < H * H + H; k += blockDim.x) {
        const int j = 2 * (k / 128) + (k >> 1 & 1), o = (k / 4) % 32 + 32 * (k & 1);
        l_w[k] = params[k < H * H ? kOffW2 + o * H + j : kOffB2 + (k - H * H)];
    }
}

// z[j] by a run-time index, as selects (folded away where j is a constant)
template <typename T>
__device__ __forceinline__ T pick4(const T z[4], int j)
{
    return j == 0 ? z[0] : j == 1 ? z[1] : j == 2 ? z[2] : z[3];
}

__device__ __forceinline__ float mlp_tanh32(float s)
{
    const float e = __builtin_amdgcn_exp2f(s * 2.8853900817779268f);   // e^(2s) = 2^(2 s log2 e)
    return fmaf(-2.0f, __builtin_amdgcn_rcpf(e + 1.0f), 1.0f);
}

__device__ __forceinline__ float mlp_out0_32_scalar(const_float *p, float x0, float x1)
{
    constexpr int H = kMlpHidden;
    float h[H];
#pragma unroll
    for (int j = 0; j < H; ++j)
        h[j] = mlp_tanh32(fmaf(p[kOffW1 + 2 * j], x0, fmaf(p[kOffW1 + 2 * j + 1], x1, p[kOffB1 + j])));
    float out = p[kOffB3];
    for (int o = 0; o < H; ++o) {
        const_float *row = p + kOffW2 + o * H;
        // two partial sums: two independent chains of multiply-adds
        float s0 = p[kOffB2 + o], s1 = 0.0f;
#pragma unroll
        for (int j = 0; j < H; j += 2) {
            s0 = fmaf(row[j], h[j], s0);
            s1 = fmaf(row[j + 1], h[j + 1], s1);
        }
        out = fmaf(p[kOffW3 + o], mlp_tanh32(s0 + s1), out);
    }
    return out;
}

// Every lane of the wave must take part (the weights of output unit lane % 32 come from each lane).
__device__ __forceinline__ float mlp_out0_32(const_float *p, const float *l_w, float x0, float x1)
{
    constexpr int H = kMlpHidden;
    const int lane = (int)__lane_id();
    // accumulators [units 0..31, units 32..63]: element 16 b + 4 g + q of a lane is output unit
    // 8 g + 4 (lane / 32) + q of state 32 b + lane % 32
    float32x e[2], o[2];
    const float4 *l_b = reinterpret_cast<const float4 *>(l_w + H * H) + (lane >> 5);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float4 b = l_b[8 * h + 2 * g];
            const float v[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                e[h][4 * g + q] = e[h][16 + 4 * g + q] = v[q];
                o[h][4 * g + q] = o[h][16 + 4 * g + q] = 0.0f;
            }
        }
    const float4 *l_a = reinterpret_cast<const float4 *>(l_w) + (lane & 31);
#pragma unroll 4
    for (int j = 0; j < H; j += 2) {
        const float4 w = l_a[16 * j];
        const float h0 = mlp_tanh32(fmaf(p[kOffW1 + 2 * j], x0, fmaf(p[kOffW1 + 2 * j + 1], x1, p[kOffB1 + j])));
        const float h1 = mlp_tanh32(fmaf(p[kOffW1 + 2 * j + 2], x0, fmaf(p[kOffW1 + 2 * j + 3], x1, p[kOffB1 + j + 1])));
        e[0] = __builtin_amdgcn_mfma_f32_32x32x1f32(w.x, h0, e[0], 0, 0, 0);
        e[1] = __builtin_amdgcn_mfma_f32_32x32x1f32(w.y, h0, e[1], 0, 0, 0);
        o[0] = __builtin_amdgcn_mfma_f32_32x32x1f32(w.z, h1, o[0], 0, 0, 0);
        o[1] = __builtin_amdgcn_mfma_f32_32x32x1f32(w.w, h1, o[1], 0, 0, 0);
    }
    float out = p[kOffB3];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            // the halves of the wave trade: then every lane has units 8 g + q (u) and 8 g + 4 + q (v) of its own state
            float u[4], v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float s0 = e[h][4 * g + q] + o[h][4 * g + q], s1 = e[h][16 + 4 * g + q] + o[h][16 + 4 * g + q];
                const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(s0), __float_as_uint(s1), false, false);
                u[q] = __uint_as_float(t[0]);
                v[q] = __uint_as_float(t[1]);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) out = fmaf(p[kOffW3 + 32 * h + 8 * g + q], mlp_tanh32(u[q]), out);
#pragma unroll
            for (int q = 0; q < 4; ++q) out = fmaf(p[kOffW3 + 32 * h + 8 * g + 4 + q], mlp_tanh32(v[q]), out);
        }
    return out;
}

// The network's normalised inputs: x0 = phi m_k0 + m_off0, x1 = ln max(|pi|, 1e-30) m_k1 + m_off1;
// FP32 state reads phi as x = phi - phi_end and takes log2.
struct NetConsts32 {
    float k0, off0, k1, off1;
};

__device__ __forceinline__ NetConsts32 net_consts32(const Inst &I)
{
    NetConsts32 q;
    q.k0 = (float)I.m_k0;
    q.off0 = (float)fma(I.phi_end, I.m_k0, I.m_off0);
    q.k1 = (float)(I.m_k1 * 0.69314718055994531);
    q.off1 = (float)I.m_off1;
    return q;
}

// ---------------------------------------------------------------------------
// Paired waves.  A run that leaves SIMDs short of waves is bound by the latency of one wave's step:
// half of it forms the random numbers, which do not depend on the state.  There each integrating wave
// gets a partner that forms its normals, one trajectory per lane and no refill: the partner fills the
// wave's LDS buffer with the normals of the next kFeedSteps steps while the wave takes the current
// ones, from registers.  Both waves of every pair run the same loop,
//   fill / step | barrier | (take the buffer, say whether the wave has a live lane) | barrier | all done?
// and leave it together, at the first turn in which no integrating wave of the block has a live lane.
// That answer is in the flags of the turn's parity, which are next written two barriers later, so every
// wave of the block reads the same one.  The arithmetic is that of the unpaired kernel.
// ---------------------------------------------------------------------------
struct Feed {
    unsigned char *buf;      // this pair's buffer (LDS)
    uint32_t *flags;         // [2][kFeedMaxPairs] (LDS): the pair's wave has a live lane
    int pair, n_pairs;       // this pair and the block's pairs
    uint64_t first;          // relative index of lane 0's trajectory
};

// One turn's end: flags up, barrier, and whether any pair goes on.
__device__ __forceinline__ bool feed_goes_on(const Feed &f, uint32_t turn)
{
    __syncthreads();
    uint32_t any = 0;
    const uint32_t *fl = f.flags + (turn & 1) * kFeedMaxPairs;
    for (int i = 0; i < f.n_pairs; ++i) any |= fl[i];
    return __builtin_amdgcn_readfirstlane(any) != 0;
}

// ---------------------------------------------------------------------------
// FP64 state: the lanes of one wave integrate trajectories of instance I,
// claimed from `cursor` (global or LDS), until the range is exhausted.
//
// Steps are taken in groups of four (one Philox call).  Inside a group every
// lane computes every step; a lane whose trajectory ended earlier in the chunk
// keeps integrating a discarded state until the chunk ends and it is refilled,
// which keeps the group free of per-step exec-mask bookkeeping.  The end of a
// trajectory (first passage, eps_1 >= 1) is recorded in a branch that is taken
// about once per 1e4-1e5 steps and retired once the group is done.  Censoring
// at max_steps needs a test before every step, so groups that can reach
// max_steps take a separate variant; which groups can is decided once per chunk
// from the wave's largest step count (wave_steps_left).  GRAD: replay the trajectories listed in
// rp.tail (cursor over the list) and scatter the gradient factors instead of
// retiring into the histogram.
// ---------------------------------------------------------------------------
// TAB: 0 a single node (constant noise); 1 nodes in phi; 2 nodes in the run's time n dN (the
// table's phi_lo and inv_h then refer to N).
template <int BIAS, int TAB, bool ALLPOS, int GRAD, int POT = kPotPiecewiseLinear, bool FEED = false>
__device__ __forceinline__ void lanes_fp64(const Inst &I, const RunArgs &R, const double2 *l_tab, const double2 *l_grid,
                                           const RetireTo &rt, const ReplayTo &rp, unsigned long long *cursor,
                                           uint64_t n_traj, uint64_t traj_offset, const Feed &feed = Feed{})
{
    static_assert(!GRAD || BIAS == kBiasMlp, "gradients need the tabulated control");
    constexpr bool LEARNED = BIAS == kBiasMlp || BIAS == kBiasMlpExact;
    const double *l_w = reinterpret_cast<const double *>(l_grid);
    const uint32_t every = (uint32_t)I.mlp_every;
    // POT: kPotPiecewiseLinear serves both linear-family potentials (V'/V = 1/d below);
    // kPotGaussianBump computes the bump's V'/V
    const DriftConsts dk = drift_consts(I);
    const BumpConsts bc = bump_consts(I);
    const GridConsts64 gc = grid_consts64(I);
    const double S0 = l_tab[0].x, t0 = l_tab[0].y;
    const double2 *l_bm = l_tab + staged_nodes(I);
    const double dN = R.dN, sqrt_dN = R.sqrt_dN, phi_end = I.phi_end, phi_T = I.phi_T;
    const double a_const = (BIAS == kBiasConst) ? I.A : 0.0;
    const double half_a2_dN = 0.5 * a_const * a_const * dN;
    const double half_dN = 0.5 * dN;
    const uint32_t j_top = (uint32_t)(staged_nodes(I) - 2);
    const double s_plus = in_vgpr(dk.s_plus), s_minus = in_vgpr(dk.s_minus);

    bool exhausted = false;
    uint64_t rel = FEED ? feed.first + __lane_id() : 0;
    bool has = FEED ? rel < n_traj : claim(true, rel, cursor, n_traj, exhausted);
    bool live = has;          // has a trajectory that has not ended yet
    double phi = I.phi_in, pi_ = I.pi_in, lnw = 0.0;
    uint32_t n = 0;
    double a_held = 0.0;      // exact network: its output at the last evaluation
    uint32_t next_eval = 0;   // exact network: the step of the next evaluation
    uint64_t traj = 0;        // replay: the listed trajectory
    double ww = 0.0;          // replay: its weight w^2
    int g_cell = -1;          // GRAD: cell of the running sums
    uint32_t g_k = 0;         // recording: the path's records so far
    double g_s[4] = {0.0, 0.0, 0.0, 0.0};
    if (GRAD == kGradReplay && has) {
        traj = rp.tail[rel].traj;
        ww = rp.tail[rel].ww;
    }
    PhiloxPre pre{};
    if (!FEED) pre = philox_pre(GRAD == kGradReplay ? traj : traj_offset + rel, I.instance, R.key0, R.key1);

    // Groups below the kink: a live lane has |pi| < sqrt 2 (the start aside) and |xi| < 6.8 (the Box-Muller
    // radius is at most sqrt(66 ln 2)), so in four steps it moves less than `reach`; where every live lane
    // starts the group further below phi_T than that, the drift takes the lower branch's constant without a
    // comparison and two selects per step.  With the event's masks and the table index this took 1e6
    // slow-roll -> ultra-slow-roll trajectories from 193.8 to 183.6 ms, with a constant bias from 227 to 199
    // ms (109 and 128 VGPRs to 95 and 113).  Keeping the lane's table record in registers between steps,
    // tried instead of the lookup, was slower (198 ms): its check is a branch in every step.
    constexpr bool CAN_BELOW = POT == kPotPiecewiseLinear && !LEARNED;
    const double reach = 4.0 * (fmax(1.4143, fabs(I.pi_in)) * dN + I.S_max * (fabs(a_const) * dN + 6.8 * sqrt_dN));
    const double phi_below = (dk.s_plus == dk.s_minus) ? __builtin_inf() : phi_T - reach;
    auto all_below = [&]() -> bool { return __builtin_amdgcn_ballot_w64(live && !(phi < phi_below)) == 0; };
    // Groups without noise: a table that ends on S = 0 (its lowest phi node, or its last time node) leaves
    // the paths beyond it classical, and a group in which every live lane stays there needs no normals, no
    // table and no noise terms.  On a phi table a lane may come back during the group; the group then
    // starts again from its state with noise.  The bump's noise ends after 3.5 of its 16 e-folds: 1e6
    // trajectories at A = 3 went from 54.4 to 37.2 ms.
    constexpr bool CAN_QUIET = TAB != 0 && !LEARNED && !ALLPOS;
    const bool quiet_table = CAN_QUIET && l_tab[TAB == 1 ? 0 : I.n_tab - 1].x == 0.0;
    const double quiet_N = I.phi_lo + (double)I.n_tab / I.inv_h;
    auto quiet_lane = [&]() -> bool { return TAB == 1 ? phi < I.phi_lo : (double)n * dN > quiet_N; };

    // Returns false for a QUIET group that left the quiet region, and for a group without EVENTS in which a
    // live lane's path ended: nothing is recorded then, and the state is the group's start again.  Paired
    // waves step without EVENTS first: one wave on its SIMD waits out the event's branch in every step, and
    // a wave's 64 paths end in at most 64 of its 2.5e4 groups (16,384 trajectories, slow roll -> ultra-slow
    // roll: 15.9 -> 14.4 ms here, 7.6 -> 5.0 in lanes_fp32; with four waves per SIMD they
    // hide that wait: FP64 the same within 1 %, FP32 7 % slower for the saved state's registers).  Of paths of
    // 35 to 2900 steps most groups are taken twice; paired, such runs are still 1.0 to 2.4 times as fast as on
    // full blocks.
    auto group = [&](auto censor_tag, auto below_tag, auto quiet_tag, auto events_tag, const double z[4]) -> bool {
        constexpr bool CENSOR = decltype(censor_tag)::value;
        constexpr bool BELOW = decltype(below_tag)::value;
        constexpr bool QUIET = decltype(quiet_tag)::value;
        constexpr bool EVENTS = decltype(events_tag)::value;
        bool fresh = false;
        uint32_t ev_status, ev_n;   // written before use: read only where fresh is set
        double ev_N, ev_lnw;
        const bool live0 = live;
        const double phi0 = phi, pi0 = pi_, lnw0 = lnw;
        bool left_quiet = false, any_end = false;
        double eps1 = 0.0;          // pi^2/2 after the last step
#pragma unroll(BIAS == kBiasMlpExact ? 1 : 4)   // the exact network: one copy of its code
        for (int j = 0; j < 4; ++j) {
            if (CENSOR && live && n == I.max_steps) {
                ev_status = kFlagCensored;
                ev_n = n;
                ev_N = __builtin_nan("");
                ev_lnw = lnw;
                live = false;
                fresh = true;
            }
            if (QUIET && TAB == 1) left_quiet = left_quiet || !(phi < I.phi_lo);
            double r;   // V'/V
            if (POT == kPotGaussianBump) {
                r = bump_dlnV(bc, phi);
            } else {
                // the hardware reciprocal (relative error below 5e-8) and one Newton step: 2.2e-15
                const double d = fma(phi, dk.kx, (!BELOW && phi >= phi_T) ? s_plus : s_minus);
                r = __builtin_amdgcn_rcp(d);
                r = fma(r, fma(-d, r, 1.0), r);
            }
            double S, t;
            if (QUIET) {
                S = t = 0.0;
            } else if (TAB) {
                const double x = ((TAB == 2 ? (double)n * dN : phi) - I.phi_lo) * I.inv_h;
                const uint32_t jj = interval_of(x, j_top);
                const double f = fmin(fmax(x - (double)jj, 0.0), 1.0);
                const double2 lo = l_tab[jj], hi = l_tab[jj + 1];
                S = lo.x + f * (hi.x - lo.x);
                t = lo.y + f * (hi.y - lo.y);
            } else {
                S = S0;
                t = t0;
            }
            // 3 - pi^2/2: one fused operation in the group's first step, from the end test's rounded pi^2/2 in
            // the others.  Written out, so that every variant of the group rounds alike.
            const double q_pi = (j == 0 || BIAS == kBiasMlpExact) ? fma(-pi_, 0.5 * pi_, 3.0) : 3.0 - eps1;
            double a = a_const;
            int cell = 0;
            double f0 = 0.0, f1 = 0.0;
            if (BIAS == kBiasMlp) a = grid_amp64(gc, l_grid, phi, pi_, cell, f0, f1);
            if (BIAS == kBiasMlpExact) {
                if (n == next_eval) {
                    a_held = mlp_out0_64(l_w, fma(phi, I.m_k0, I.m_off0),
                                         fma(log(fmax(fabs(pi_), 1e-30)), I.m_k1, I.m_off1));
                    next_eval += every;
                }
                a = a_held;
            }
            const double zs = QUIET ? 0.0 : pick4(z, j);  // xi sqrt(dN)
            const double noise = S * zs;
            // without a bias the amplitude is a literal 0, which IEEE arithmetic does not fold away:
            // the terms are left out instead (the same values, up to the sign of a zero)
            const double aS = a * S;
            const double phi_n = QUIET ? phi + pi_ * dN
                                 : (BIAS == kBiasNone) ? phi + pi_ * dN + noise : phi + (pi_ + aS) * dN + noise;
            const double drift_pi = pi_ - q_pi * (pi_ + r) * dN;
            const double pi_n = QUIET ? drift_pi
                                : (BIAS == kBiasNone) ? drift_pi + t * noise : drift_pi + t * (aS * dN + noise);
            if (QUIET) {
                // no noise, no weight
            } else if (BIAS == kBiasConst) {
                if (ALLPOS) {
                    lnw -= a * zs + half_a2_dN;
                } else {
                    lnw -= (S > 0.0) ? a * zs + half_a2_dN : 0.0;
                }
            } else if (LEARNED) {
                const double dA = fma(a, zs, a * a * half_dN);
                lnw -= (ALLPOS || S > 0.0) ? dA : 0.0;
            }
            if (GRAD && live) {
                if (cell != g_cell) {
                    if (GRAD == kGradReplay) grad_flush(rp, gc.n1c, g_cell, g_s, ww);
                    else grad_record(rp.rec, rel, g_k, g_cell, g_s);
                    g_cell = cell;
                }
                grad_add(g_s, (ALLPOS || S > 0.0) ? -zs : 0.0, f0, f1);
            }
            // live and fresh are updated outside the branch, so that they stay lane masks; the event's inputs
            // pass through an empty volatile asm, which keeps its work (a second comparison with phi_end, a
            // division) from moving in front of the branch, into every step
            eps1 = half_sq(pi_n);
            const bool ends = (phi_n <= phi_end) | (eps1 >= 1.0);
            const bool hit = EVENTS && (live & ends);
            if (!EVENTS) any_end = any_end | ends;
            if (hit) {
                double pa = phi, pb = phi_n;
                uint32_t nb = n;
                asm volatile("; passage event" : "+v"(pa), "+v"(pb), "+v"(nb));
                const bool crossed = pb <= phi_end;
                ev_status = crossed ? 0u : kFlagEndedEarly;
                ev_n = nb + 1;
                ev_N = crossed ? (double)nb * dN + dN * ((pa - phi_end) / (pa - pb)) : (double)(nb + 1) * dN;
                ev_lnw = lnw;
            }
            live = live & !hit;
            fresh = fresh | hit;
            phi = phi_n;
            pi_ = pi_n;
            n += 1;
        }
        if ((QUIET && TAB == 1) || !EVENTS) {
            if (__builtin_amdgcn_ballot_w64(live0 && (left_quiet || any_end)) != 0) {
                phi = phi0;
                pi_ = pi0;
                lnw = lnw0;
                live = live0;
                n -= 4;
                return false;
            }
        }
        if (fresh) {
            if (GRAD == kGradRecord) {
                grad_record(rp.rec, rel, g_k, g_cell, g_s);
                rp.rec.count[rel] = g_k;
                g_cell = -1;
                g_k = 0;
            }
            if (GRAD == kGradReplay) {
                grad_flush(rp, gc.n1c, g_cell, g_s, ww);
                g_cell = -1;
                if (ev_status != 0u) atomicAdd(rp.mismatch, 1ull);
            } else {
                retire(rt, rel, ev_status, ev_n, ev_N, ev_lnw);
            }
        }
        return true;
    };
    using Yes = std::integral_constant<bool, true>;
    using No = std::integral_constant<bool, false>;
    // The group's variant from its normals; `may_cap`: a lane may reach max_steps in it.
    auto noisy_group = [&](bool may_cap, const double z[4]) {
        using Below = std::integral_constant<bool, CAN_BELOW>;
        // paired waves: without events first, unless a step leaves records behind
        using Last = std::integral_constant<bool, !FEED || GRAD != kGradNone>;
        if (may_cap) group(Yes(), No(), No(), Yes(), z);
        else if (CAN_BELOW && all_below()) {
            if (!group(No(), Below(), No(), Last(), z)) group(No(), Below(), No(), Yes(), z);
        } else if (!group(No(), No(), No(), Last(), z)) group(No(), No(), No(), Yes(), z);
    };
    auto quiet_group = [&](bool may_cap) -> bool {
        if constexpr (CAN_QUIET) {
            const double none[4] = {0.0, 0.0, 0.0, 0.0};
            if (may_cap || !quiet_table || __builtin_amdgcn_ballot_w64(live && !quiet_lane()) != 0) return false;
            return group(No(), No(), Yes(), Yes(), none);
        }
        return false;
    };

    if constexpr (FEED) {
        const double2 *buf = reinterpret_cast<const double2 *>(feed.buf) + __lane_id();
        for (uint32_t turn = 0;; ++turn) {
            __syncthreads();
            double2 v[kFeedSteps / 2];
#pragma unroll
            for (int q = 0; q < kFeedSteps / 2; ++q) v[q] = buf[64 * q];
            feed.flags[(turn & 1) * kFeedMaxPairs + feed.pair] = __any(live) ? 1u : 0u;
            if (!feed_goes_on(feed, turn)) break;
            if (!__any(live)) continue;
#pragma unroll
            for (int q = 0; q < kFeedSteps / 2; q += 2) {
                const double z[4] = {v[q].x, v[q].y, v[q + 1].x, v[q + 1].y};
                // all lanes are at the same step
                const bool may_cap = (uint32_t)__builtin_amdgcn_readfirstlane(n) + 4 > I.max_steps;
                if (!quiet_group(may_cap)) noisy_group(may_cap, z);
            }
        }
        return;
    }
    while (__any(has)) {
        const uint32_t left = wave_steps_left(has, n, I.max_steps);
        for (int k = 0; k < R.chunk; k += 4) {
            if (!__any(live)) break;
            const bool may_cap = (uint32_t)k + 4 > left;
            if (quiet_group(may_cap)) continue;
            uint32_t w[4];
            philox_call(n >> 2, pre, R.key0, R.key1, w);
            double z[4];
            box_muller64(w[0], w[1], sqrt_dN, l_bm, z[0], z[1]);
            box_muller64(w[2], w[3], sqrt_dN, l_bm, z[2], z[3]);
            noisy_group(may_cap, z);
        }
        if (!live) has = false;
        if (claim(!has, rel, cursor, n_traj, exhausted)) {
            has = true;
            live = true;
            phi = I.phi_in;
            pi_ = I.pi_in;
            lnw = 0.0;
            n = 0;
            a_held = 0.0;
            next_eval = 0;
            if (GRAD == kGradReplay) {
                traj = rp.tail[rel].traj;
                ww = rp.tail[rel].ww;
            }
            pre = philox_pre(GRAD == kGradReplay ? traj : traj_offset + rel, I.instance, R.key0, R.key1);
        }
    }
}

// The partner of a paired FP64 wave: the normals of kFeedSteps steps (two or more generator calls) a turn.
template <int DIM>
__device__ __forceinline__ void feed_fp64(const Inst &I, const RunArgs &R, const double2 *l_bm, uint64_t traj_offset,
                                          const Feed &feed)
{
    const PhiloxPre pre = philox_pre(traj_offset + feed.first + __lane_id(), I.instance, R.key0, R.key1);
    double2 *buf = reinterpret_cast<double2 *>(feed.buf) + __lane_id();
    uint32_t m = 0;
    for (uint32_t turn = 0;; ++turn) {
#pragma unroll
        for (int q = 0; q < DIM * kFeedSteps / 2; q += 2) {
            uint32_t w[4];
            philox_call(m++, pre, R.key0, R.key1, w);
            double2 a, b;
            box_muller64(w[0], w[1], R.sqrt_dN, l_bm, a.x, a.y);
            box_muller64(w[2], w[3], R.sqrt_dN, l_bm, b.x, b.y);
            buf[64 * q] = a;
            buf[64 * (q + 1)] = b;
        }
        __syncthreads();
        if (!feed_goes_on(feed, turn)) break;
    }
}

// ---------------------------------------------------------------------------
// FP32 state: x = phi - phi_end and pi each as an unevaluated pair of floats
// hi + lo.  A step adds its increment to the low word only (lo += dx) and
// reads the state as the rounded sum hi + lo; once per step group (16 steps, 4
// where the network is evaluated in the step) the pair is renormalised (Fast2Sum
// of hi and lo).
// Against an exact two-sum per step this leaves one rounding of the low word per
// step, at the scale of ulp(16 increments), far below the FP32 resolution of the
// state itself.
// ---------------------------------------------------------------------------
struct F32Consts {
    float xT_hi, xT_lo;        // phi_T - phi_end as a float pair
    float kx, s_plus, s_minus; // (V'/V) dN/2 = 1/(kx (phi - phi_T) + s), s = s_plus (phi >= phi_T) or s_minus
    float u_off;               // (phi_end - phi_lo) * inv_h: table coordinate of x = 0
    float inv_h;
    float t_scale, t_off;      // time tables: coordinate n dN inv_h - N_lo inv_h
    float jtop;                // n_tab - 1: the last record (slope 0, V'/V interval NaN)
    float dN, half_dN;
    float m2ln2_dN;            // -2 ln 2 dN: rho = sqrt(log2(u) m2ln2_dN) = sqrt(-2 ln u) sqrt(dN)
    float adN;                 // constant bias: A dN, the shift carried by each step's normal
};

__device__ __forceinline__ F32Consts f32_consts(const Inst &I, const RunArgs &R)
{
    F32Consts c;
    const double xT = I.phi_T - I.phi_end;
    c.xT_hi = (float)xT;
    c.xT_lo = (float)(xT - (double)c.xT_hi);
    const double two_over_dN = 2.0 / R.dN;
    if (I.pot_kind == kPotExponential) {
        c.kx = 0.0f;
        c.s_plus = c.s_minus = (float)(two_over_dN / I.A_plus);
    } else {
        c.kx = (float)two_over_dN;
        c.s_plus = (float)(I.V0 / I.A_plus * two_over_dN);
        c.s_minus = (float)(I.V0 / I.A_minus * two_over_dN);
    }
    c.u_off = (float)((I.phi_end - I.phi_lo) * I.inv_h);
    c.inv_h = (float)I.inv_h;
    c.t_scale = (float)(R.dN * I.inv_h);
    c.t_off = (float)(-I.phi_lo * I.inv_h);
    c.jtop = (float)(staged_nodes(I) - 1);
    c.dN = (float)R.dN;
    c.half_dN = (float)(0.5 * R.dN);
    c.m2ln2_dN = (float)(-2.0 * 0.69314718055994531 * R.dN);
    c.adN = (I.bias_kind == kBiasConst) ? (float)(I.A * R.dN) : 0.0f;
    return c;
}

// Box-Muller in FP32 on uniforms fl32(w) 2^-32 + 2^-33: the same uniform as the
// FP64 path, rounded to 24 significant bits (relative, not absolute, resolution,
// so the radius stays accurate for small u).  Never 0; at most 1.0f, where
// log2 gives 0 and the radius -0 or 0.  v_log_f32 returns log2, v_sin_f32 /
// v_cos_f32 take turns.  Returns xi sqrt(dN) + off for the two steps of the pair.
__device__ __forceinline__ void box_muller32(uint32_t wa, uint32_t wb, float m2ln2_dN, float off, float &za, float &zb)
{
    const float ua = fmaf((float)wa, 0x1p-32f, 0x1p-33f);
    const float ub = fmaf((float)wb, 0x1p-32f, 0x1p-33f);
    const float rho = __builtin_amdgcn_sqrtf(__builtin_amdgcn_logf(ua) * m2ln2_dN);
    za = fmaf(rho, __builtin_amdgcn_cosf(ub), off);
    zb = fmaf(rho, __builtin_amdgcn_sinf(ub), off);
}

template <int BIAS, int TAB, bool ALLPOS, int GRAD, bool FEED = false>
__device__ __forceinline__ void lanes_fp32(const Inst &I, const RunArgs &R, const float4 *l_tab, const float4 *l_grid,
                                           const RetireTo &rt, const ReplayTo &rp, unsigned long long *cursor,
                                           uint64_t n_traj, uint64_t traj_offset, const Feed &feed = Feed{})
{
    static_assert(!GRAD || BIAS == kBiasMlp, "gradients need the tabulated control");
    constexpr bool EXACT = BIAS == kBiasMlpExact || BIAS == kBiasMlpMatrix;
    constexpr bool LEARNED = BIAS == kBiasMlp || EXACT;
    // steps per group: 16 (four generator calls), so that the group's fixed work (table record,
    // renormalisation, FP64 sums, loop control) is shared by 16 steps; the normals of the whole
    // group are formed first.  The exact network keeps groups of 4 and one copy of its code.
    constexpr int G = EXACT ? 4 : 16;
    const_float *wp = (const_float *)(uintptr_t)I.mlp_params;
    const NetConsts32 nq = net_consts32(I);
    const uint32_t every = (uint32_t)I.mlp_every;
    const F32Consts c = f32_consts(I, R);
    const GridConsts32 gc = grid_consts32(I);
    const float S0 = l_tab[0].x, t0 = l_tab[0].z;
    const float2 *l_rtab = reinterpret_cast<const float2 *>(l_tab + staged_nodes(I));
    const double x_in = I.phi_in - I.phi_end;
    const float x_in_hi = (float)x_in, x_in_lo = (float)(x_in - (double)x_in_hi);
    const float pi_in_hi = (float)I.pi_in, pi_in_lo = (float)(I.pi_in - (double)pi_in_hi);
    const double dN = R.dN;
    const double A = (BIAS == kBiasConst) ? I.A : 0.0;
    const double half_a2_dN = 0.5 * A * A * dN;
    const float s_plus = in_vgpr(c.s_plus), s_minus = in_vgpr(c.s_minus);

    bool exhausted = false;
    uint64_t rel = FEED ? feed.first + __lane_id() : 0;
    bool has = FEED ? rel < n_traj : claim(true, rel, cursor, n_traj, exhausted);
    bool live = has;          // has a trajectory that has not ended yet
    // state: x = xh + xl, pi = ph + pl; xs, ps their rounded sums (what a step reads; xs is formed
    // each step only where a step reads it, and otherwise once per group)
    float xh = x_in_hi, xl = x_in_lo, ph = pi_in_hi, pl = pi_in_lo;
    float xs = x_in_hi, ps = pi_in_hi;
    double zsum = 0.0;        // constant bias: sum of z = xi sqrt(dN) + a dN over steps with S > 0
    uint32_t n_on = 0;        // constant bias: number of such steps (counted only when some node has S = 0)
    double lnw = 0.0;         // learned bias: ln w up to the current group
    uint32_t n = 0;
    float a_held = 0.0f;      // exact network: its output at the last evaluation
    uint32_t next_eval = 0;   // exact network: the step of the next evaluation
    uint64_t traj = 0;        // replay: the listed trajectory
    double ww = 0.0;          // replay: its weight w^2
    int g_cell = -1;          // GRAD: cell of the running sums
    uint32_t g_k = 0;         // recording: the path's records so far
    float g_s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (GRAD == kGradReplay && has) {
        traj = rp.tail[rel].traj;
        ww = rp.tail[rel].ww;
    }
    PhiloxPre pre{};
    if (!FEED) pre = philox_pre(GRAD == kGradReplay ? traj : traj_offset + rel, I.instance, R.key0, R.key1);

    // constant bias: each step's normal carries the drift shift, z = xi sqrt(dN) + c.adN with
    // c.adN = fl32(A dN), so the exponent of eq. (weight_A) in 1D over k steps,
    // -A sum xi sqrt(dN) - k A^2 dN / 2, is -A sum z + k (A c.adN - A^2 dN / 2)
    const double lnw_step = A * (double)c.adN - half_a2_dN;
    auto lnw_of = [&](double zs_total, uint32_t steps_on) -> double {
        return (BIAS == kBiasNone) ? 0.0 : -A * zs_total + (double)steps_on * lnw_step;
    };

    // Phi tables: a lane whose interval at the group start holds an interpolated V'/V reads that
    // record once for the whole group, and each step evaluates S, tan theta and V'/V on that
    // interval's linear piece: value at x = xh plus slope per unit x times xl (x - xh = xl within
    // the group), the values and slopes formed once per group.  Inside the interval
    // this is the table's interpolation; where the group's path passes a node it extends the start
    // interval's piece instead of switching to the next one, which differs from the interpolation
    // by the change of slope at the node times the distance past it (second order in the node
    // spacing for a table of a smooth function).  A lane whose interval is NaN-marked (table
    // edges, the kink, tables that do not qualify) takes the record of each step's own clamped
    // coordinate instead.  The choice is the lane's own, so a trajectory's
    // arithmetic does not depend on the other lanes of its wave: SPAN groups, where no live lane is
    // in a NaN interval, run the first form only; the other groups run both and select per lane.
    // the group-start record's S, tan theta and V'/V at x = xh and their slopes per unit x
    float g_S = 0.0f, g_dS = 0.0f, g_t = 0.0f, g_dt = 0.0f, g_r = 0.0f, g_dr = 0.0f;

    // The epsilon_1 = 1 end (|pi| >= sqrt 2) in SPAN groups.  While |pi| < sqrt 2, a step changes pi
    // by at most delta = 6 (sqrt2 dN/2 + |V'/V| dN/2) + |tan theta| S |z| (|pi^2 - 6| <= 6), where
    // S, tan theta and V'/V are read from a smooth record extended past its interval by at most
    // the D intervals a group's path can move (|dx| <= sqrt2 dN + S |z|), and |z| <= 6.8 sqrt(dN) +
    // |a| dN (the Box-Muller radius is at most sqrt(66 ln 2 dN)).  A lane with |pi| <= pi_safe at
    // the group start therefore stays below sqrt 2 (1 - 1e-3) for 16 steps (5 % margin on delta),
    // and a SPAN group whose live lanes all qualify leaves the end test out; the other SPAN groups
    // keep it.  With no usable bound (fine grids, where D is large) pi_safe is -1: no lane
    // qualifies, and every group keeps the test.
    float pi_safe = -1.0f;
    if (TAB == 1 && !LEARNED) {
        const float zmax = fmaf(6.8f, __builtin_amdgcn_sqrtf(c.dN), fabsf((float)A) * c.dN);
        const float D = fmaf(16.0f * c.inv_h, fmaf(2.0f * I.rec_S, zmax, 1.4143f * c.dN), 1.0f);
        const float Sx = fmaf(I.rec_dS, D, I.rec_S);
        const float Tx = fmaf(I.rec_dt, D, I.rec_t);
        const float Rx = fmaf(I.rec_dr, D, I.rec_r) * c.half_dN;
        const float delta = fmaf(6.0f, fmaf(0.7072f, c.dN, Rx), Tx * Sx * zmax);
        if (Sx <= 2.0f * I.rec_S && delta == delta && delta >= 0.0f && delta < 1.0f)
            pi_safe = fmaf(-16.8f, delta, 1.4128f);
    }

    // Time tables: a group is plain for a lane that stays below the kink (as in lanes_fp64, 16 steps' reach,
    // 1 % above it for the rounding), whose coordinate runs inside [0, last node before the first one with
    // S = 0], and that cannot reach |pi| = sqrt 2 (pi_safe's bound with the largest S and tan theta of the
    // table and the largest |V'/V| between phi_end and the kink, where it is monotonic): its steps need no
    // clamp, no branch select, no test of S and no end test, and n + j is exact in FP32.  Eight operations
    // fewer of some fifty per step: 1e6 trajectories of the time-indexed problem 124.5 -> 104.8 ms.
    // With equal slopes there is no kink to stay below, as long as |V'/V| does not grow upwards either
    // (V' >= 0, or the exponential potential); V' < 0 keeps the lanes below phi_T, up to which the bound holds.
    const float z_most = fmaf(6.8f, __builtin_amdgcn_sqrtf(c.dN), fabsf((float)A) * c.dN);
    const float reach = 1.01f * 16.0f * fmaf((float)I.S_max, z_most, fmaxf(1.4143f, fabsf((float)I.pi_in)) * c.dN);
    const float d_end = fmaf(-(c.xT_hi + c.xT_lo), c.kx, c.s_minus);      // 1/((V'/V) dN/2) at phi_end
    const float below = (c.s_plus == c.s_minus && (c.kx == 0.0f || d_end > 0.0f)) ? __builtin_inff() : -reach;
    const float u_plain = (float)(I.n_pos - 1);
    float pi_plain = -1.0f;
    if (TAB == 2) {
        const float r_most = 1.01f / fminf(fabsf(c.s_minus), fabsf(d_end));
        const float delta = fmaf(6.0f, fmaf(0.7072f, c.dN, r_most), (float)(I.t_max * I.S_max) * z_most);
        if (delta >= 0.0f && delta < 1.0f) pi_plain = fmaf(-16.8f, delta, 1.4128f);
    }
    auto plain_lane = [&]() -> bool {
        const float u0 = fmaf((float)n, c.t_scale, c.t_off), u1 = fmaf((float)(n + G - 1), c.t_scale, c.t_off);
        return u0 >= 0.0f && u1 < u_plain && n < (1u << 24) - G &&
               (xh - c.xT_hi) + (xl - c.xT_lo) < below && fabsf(ps) <= pi_plain;
    };

    // As in lanes_fp64, a group without EVENTS returns false, at the group's start again, if a live lane's
    // path ends in it.
    auto group = [&](auto censor_tag, auto span_tag, auto end_tag, auto events_tag, const float z[G]) -> bool {
        constexpr bool CENSOR = decltype(censor_tag)::value;
        constexpr bool SPAN = decltype(span_tag)::value;
        constexpr bool END = decltype(end_tag)::value;   // test the eps_1 = 1 end in each step
        constexpr bool EVENTS = decltype(events_tag)::value;
        const float xl0 = xl, pl0 = pl, xs0 = xs, ps0 = ps;
        const uint32_t n_on0 = n_on;
        bool any_end = false;
        static_assert(!SPAN || (TAB != 0 && !CENSOR), "one record per group, or a plain time group: no censoring");
        // a SPAN group of a time table is plain: below the kink, inside the table, S > 0 (plain_lane)
        constexpr bool PLAIN = TAB == 2 && SPAN;
        constexpr bool ON = ALLPOS || PLAIN;                      // S > 0 in every step
        const float nf = PLAIN ? (float)n : 0.0f;
        // the rounded sum xs is read by a step only for a per-step table lookup and by the control
        constexpr bool STEP_XS = LEARNED || (TAB == 1 && !SPAN);
        float zacc = 0.0f;        // constant bias: sum of this group's xi sqrt(dN); learned: of its dA
        bool fresh = false;
        uint32_t ev_code;         // written before use: read only where fresh is set
        double ev_N, ev_lnw;
        auto lnw_now = [&](uint32_t steps) -> double {
            if (LEARNED) return lnw - (double)zacc;
            return lnw_of(zsum + (double)zacc, ALLPOS ? steps : PLAIN ? n_on + (steps - n) : n_on);
        };
#pragma unroll(EXACT ? 1 : G)   // the exact network: one copy of its code
        for (int j = 0; j < G; ++j) {
            const float zj = (G == 4) ? pick4(z, j) : z[j];
            if (CENSOR && live && n + j == I.max_steps) {
                ev_code = (n + j) | kFlagCensored;
                ev_N = __builtin_nan("");
                ev_lnw = lnw_now(n + j);
                live = false;
                fresh = true;
            }
            // (V'/V) dN/2 exactly: 1/(kx (phi - phi_T) + s), phi - phi_T = (xh - xT_hi) + (xl - xT_lo)
            auto drift_exact = [&]() -> float {
                const float dT = (xh - c.xT_hi) + (xl - c.xT_lo);
                return __builtin_amdgcn_rcpf(fmaf(dT, c.kx, (!PLAIN && dT >= 0.0f) ? s_plus : s_minus));
            };
            float S, t, r;        // r = (V'/V) dN/2
            if (TAB == 2) {
                // time table: the node at n dN; V'/V exactly (the V'/V intervals follow phi)
                const float u = PLAIN ? fmaf(nf + (float)j, c.t_scale, c.t_off)     // n + j < 2^24: exact
                                      : __builtin_amdgcn_fmed3f(fmaf((float)(n + j), c.t_scale, c.t_off), 0.0f, c.jtop);
                const float f = __builtin_amdgcn_fractf(u);
                const float4 node = l_tab[(int)u];
                S = fmaf(f, node.y, node.x);
                t = fmaf(f, node.w, node.z);
                r = drift_exact();
            } else if (SPAN) {
                S = fmaf(xl, g_dS, g_S);
                t = fmaf(xl, g_dt, g_t);
                r = fmaf(xl, g_dr, g_r);
            } else if (TAB) {
                // the coordinate clamped to [0, n_tab - 1]: its integer part is the record, its
                // fraction the weight; past the last node the last record (slope 0) gives the
                // edge value, and its NaN V'/V interval the exact V'/V
                const float u = __builtin_amdgcn_fmed3f(fmaf(xs, c.inv_h, c.u_off), 0.0f, c.jtop);
                const float f = __builtin_amdgcn_fractf(u);
                const float4 node = l_tab[(int)u];
                const float2 rn = l_rtab[(int)u];
                S = fmaf(f, node.y, node.x);
                t = fmaf(f, node.w, node.z);
                // V'/V interpolated in the interval (error below FP32 resolution); NaN marks the
                // intervals where it is computed exactly instead: the two edge intervals, which
                // also take every clamped coordinate outside the table, the two intervals at the
                // kink phi_T, and every interval of a table that does not qualify
                r = fmaf(f, rn.y, rn.x);
                if (TAB == 1 && g_r == g_r) {
                    // the lane's group-start interval is smooth: the arithmetic of a SPAN group
                    S = fmaf(xl, g_dS, g_S);
                    t = fmaf(xl, g_dt, g_t);
                    r = fmaf(xl, g_dr, g_r);
                }
                if (__any(r != r)) {
                    // a real branch (rarely taken): the volatile asm keeps the compiler from
                    // computing the exact value in every step and selecting
                    asm volatile("; exact V'/V");
                    if (r != r) r = drift_exact();
                }
            } else {
                S = S0;
                t = t0;
                r = drift_exact();
            }
            float a = 0.0f;       // the learned amplitude
            int cell = 0;
            float f0 = 0.0f, f1 = 0.0f;
            if (BIAS == kBiasMlp) a = grid_amp32(gc, l_grid, xs, ps, cell, f0, f1);
            if (BIAS == kBiasMlpExact) {
                if (n + j == next_eval) {
                    a_held = mlp_out0_32_scalar(wp, fmaf(xs, nq.k0, nq.off0),
                                                fmaf(__builtin_amdgcn_logf(fmaxf(fabsf(ps), 1e-30f)), nq.k1, nq.off1));
                    next_eval += every;
                }
                a = a_held;
            }
            if (BIAS == kBiasMlpMatrix) {
                const bool due = n + j == next_eval;
                if (__any(due)) {      // by the whole wave; lanes at other phases keep what they hold
                    const float v = mlp_out0_32(wp, reinterpret_cast<const float *>(l_grid), fmaf(xs, nq.k0, nq.off0),
                                                fmaf(__builtin_amdgcn_logf(fmaxf(fabsf(ps), 1e-30f)), nq.k1, nq.off1));
                    a_held = due ? v : a_held;
                    next_eval += due ? every : 0u;
                }
                a = a_held;
            }
            // Bn = S (a dN + xi sqrt(dN)): the bias and noise increments of phi (a constant bias
            // rides in z = xi sqrt(dN) + a dN; the learned one is added here, z = xi sqrt(dN))
            const float Bn = S * (LEARNED ? fmaf(a, c.dN, zj) : zj);
            if (BIAS == kBiasConst) {
                if (ON) {
                    zacc = (j == 0) ? z[0] : zacc + zj;
                } else {
                    const bool on = S > 0.0f;
                    zacc += on ? zj : 0.0f;
                    n_on += on ? 1u : 0u;
                }
            } else if (LEARNED) {
                const float dA = fmaf(a, zj, a * a * (0.5f * c.dN));
                zacc += (ALLPOS || S > 0.0f) ? dA : 0.0f;
            }
            if (GRAD && live) {
                if (cell != g_cell) {
                    if (GRAD == kGradReplay) grad_flush(rp, gc.n1c, g_cell, g_s, ww);
                    else grad_record(rp.rec, rel, g_k, g_cell, g_s);
                    g_cell = cell;
                }
                grad_add(g_s, (ALLPOS || S > 0.0f) ? -zj : 0.0f, f0, f1);
            }
            // x += pi dN + Bn; pi += (pi^2 - 6)(pi dN/2 + (V'/V) dN/2) + tan(theta) Bn, i.e.
            // -(3 - pi^2/2)(pi + V'/V) dN plus the bias and noise along (1, tan theta).  The pi
            // terms go into their low word by two FMAs; the x increment is formed first and added
            // once, since adding its two parts one at a time rounds twice at the low word's scale,
            // which shifted the crossing (the mean N by ~1e-6 against FP64 on the same normals).
            const float x0l = xl;
            xl += fmaf(ps, c.dN, Bn);
            pl = fmaf(fmaf(ps, ps, -6.0f), fmaf(ps, c.half_dN, r), fmaf(t, Bn, pl));
            if (STEP_XS) xs = xh + xl;
            ps = ph + pl;
            // x <= 0: the sign of a rounded sum is that of the exact one, so this is xs <= 0
            const bool crossed = xl <= -xh;
            // eps_1 = pi^2/2 >= 1: |pi| >= the float just above sqrt(2) (no float lies between
            // sqrt(2) and it, so this is pi^2 >= 2 for float pi); left out of the groups where no
            // live lane can get there (pi_safe above)
            const bool ended = END && fabsf(ps) >= 0x1.6a09e8p+0f;
            // live and fresh are updated outside the branch, so that they stay lane masks
            const bool hit = EVENTS && live && (crossed || ended);
            if (!EVENTS) any_end = any_end | crossed | ended;
            if (hit) {
                // both candidates, then a select on the crossing mask: no divergent branch inside.
                // The state passes through an empty volatile asm first, which keeps the compiler
                // from moving this rarely taken work in front of the branch (into every step).
                float bh = xh, b0 = x0l, b1 = xl;
                uint32_t nb = n + j;
                asm volatile("; passage event" : "+v"(bh), "+v"(b0), "+v"(b1), "+v"(nb));
                const double x0 = (double)bh + (double)b0;
                const double x1 = (double)bh + (double)b1;
                const double N_cross = (double)nb * dN + dN * (x0 / (x0 - x1));
                const double N_end = (double)(nb + 1) * dN;
                ev_code = (nb + 1) | (crossed ? 0u : kFlagEndedEarly);
                ev_N = crossed ? N_cross : N_end;
                ev_lnw = lnw_now(nb + 1);
            }
            live = live && !hit;
            fresh = fresh || hit;
        }
        if (!EVENTS) {
            if (__builtin_amdgcn_ballot_w64(live && any_end) != 0) {
                xl = xl0;
                pl = pl0;
                xs = xs0;
                ps = ps0;
                n_on = n_on0;
                return false;
            }
        }
        n += G;
        if (PLAIN && !ALLPOS && BIAS == kBiasConst) n_on += G;
        if (LEARNED) lnw -= (double)zacc;
        else zsum += (double)zacc;
        if (fresh) {
            if (GRAD == kGradRecord) {
                grad_record(rp.rec, rel, g_k, g_cell, g_s);
                rp.rec.count[rel] = g_k;
                g_cell = -1;
                g_k = 0;
            }
            if (GRAD == kGradReplay) {
                grad_flush(rp, gc.n1c, g_cell, g_s, ww);
                g_cell = -1;
                if ((ev_code & ~kStepMask) != 0u) atomicAdd(rp.mismatch, 1ull);
            } else {
                retire(rt, rel, ev_code & ~kStepMask, ev_code & kStepMask, ev_N, ev_lnw);
            }
        }
        // renormalise the pairs once per group (Fast2Sum of hi and the accumulated lo; ps, and xs
        // where a step reads it, are their rounded sums already)
        if (!STEP_XS) xs = xh + xl;
        xl = xl - (xs - xh);
        xh = xs;
        pl = pl - (ps - ph);
        ph = ps;
        return true;
    };

    // One group from its normals; `may_cap`: a lane may reach max_steps in it.
    auto run_group = [&](bool may_cap, const float z[G]) {
        using T = std::integral_constant<bool, true>;
        using F = std::integral_constant<bool, false>;
        // paired waves: without events first, unless a step leaves records behind
        using L = std::integral_constant<bool, !FEED || GRAD != kGradNone>;
        if constexpr (TAB == 1) {
            // the record of the lane's interval at the group start
            const float u0 = __builtin_amdgcn_fmed3f(fmaf(xs, c.inv_h, c.u_off), 0.0f, c.jtop);
            const int j0 = (int)u0;
            const float4 g_node = l_tab[j0];
            const float2 g_rn = l_rtab[j0];
            const float fh = fmaf(xh, c.inv_h, c.u_off - (float)j0);   // the fraction at x = xh
            g_S = fmaf(fh, g_node.y, g_node.x);
            g_dS = g_node.y * c.inv_h;
            g_t = fmaf(fh, g_node.w, g_node.z);
            g_dt = g_node.w * c.inv_h;
            g_r = fmaf(fh, g_rn.y, g_rn.x);
            g_dr = g_rn.y * c.inv_h;
        }
        if (may_cap) {
            group(T(), F(), T(), T(), z);
        } else {
            if constexpr (TAB == 1) {
                if (__builtin_amdgcn_ballot_w64(live && g_r != g_r) != 0) {
                    group(F(), F(), T(), T(), z);
                } else if constexpr (LEARNED) {
                    if (!group(F(), T(), T(), L(), z)) group(F(), T(), T(), T(), z);
                } else {
                    if (__builtin_amdgcn_ballot_w64(live && fabsf(ps) > pi_safe) == 0) {
                        if (!group(F(), T(), F(), L(), z)) group(F(), T(), F(), T(), z);
                    } else {
                        group(F(), T(), T(), T(), z);
                    }
                }
            } else if constexpr (TAB == 2) {
                if (__builtin_amdgcn_ballot_w64(live && !plain_lane()) == 0) {
                    if (!group(F(), T(), F(), L(), z)) group(F(), T(), F(), T(), z);
                } else {
                    group(F(), F(), T(), T(), z);
                }
            } else {
                if (!group(F(), F(), T(), L(), z)) group(F(), F(), T(), T(), z);
            }
        }
    };

    if constexpr (FEED) {
        static_assert(G == kFeedSteps32, "a turn is one group");
        const float4 *buf = reinterpret_cast<const float4 *>(feed.buf) + __lane_id();
        for (uint32_t turn = 0;; ++turn) {
            __syncthreads();
            float z[G];
#pragma unroll
            for (int q = 0; q < G / 4; ++q) {
                const float4 v = buf[64 * q];
                z[4 * q] = v.x;
                z[4 * q + 1] = v.y;
                z[4 * q + 2] = v.z;
                z[4 * q + 3] = v.w;
            }
            feed.flags[(turn & 1) * kFeedMaxPairs + feed.pair] = __any(live) ? 1u : 0u;
            if (!feed_goes_on(feed, turn)) break;
            // all lanes are at the same step
            if (__any(live)) run_group((uint32_t)__builtin_amdgcn_readfirstlane(n) + G > I.max_steps, z);
        }
        return;
    }
    // n_hi: a wave-uniform upper bound on n over the lanes that hold a trajectory.  All lanes step
    // together and a refilled lane restarts at 0, so adding each chunk's steps keeps it a bound;
    // the exact maximum (a cross-lane reduction) is formed only once the bound comes within a
    // chunk of max_steps, so the groups that can reach max_steps are the same as with the exact
    // count at every chunk
    uint32_t n_hi = 0;
    while (__any(has)) {
        if ((uint64_t)n_hi + (uint64_t)R.chunk + G > I.max_steps)
            n_hi = I.max_steps - wave_steps_left(has, n, I.max_steps);
        const uint32_t left = I.max_steps - n_hi;
        int k = 0;
        for (; k < R.chunk; k += G) {
            if (!__any(live)) break;
            uint32_t w[G];
#pragma unroll
            for (int q = 0; q < G; q += 4) philox_call((n >> 2) + (uint32_t)(q >> 2), pre, R.key0, R.key1, w + q);
            float z[G];
            const float off = (BIAS == kBiasConst) ? c.adN : 0.0f;
#pragma unroll
            for (int q = 0; q < G; q += 2) box_muller32(w[q], w[q + 1], c.m2ln2_dN, off, z[q], z[q + 1]);
            run_group((uint32_t)k + G > left, z);
        }
        n_hi += (uint32_t)k;
        if (!live) has = false;
        if (claim(!has, rel, cursor, n_traj, exhausted)) {
            has = true;
            live = true;
            xh = xs = x_in_hi;
            xl = x_in_lo;
            ph = ps = pi_in_hi;
            pl = pi_in_lo;
            zsum = 0.0;
            n_on = 0;
            lnw = 0.0;
            n = 0;
            a_held = 0.0f;
            next_eval = 0;
            if (GRAD == kGradReplay) {
                traj = rp.tail[rel].traj;
                ww = rp.tail[rel].ww;
            }
            pre = philox_pre(GRAD == kGradReplay ? traj : traj_offset + rel, I.instance, R.key0, R.key1);
        }
    }
}
// The partner of a paired FP32 wave: the shifted normals of one group (four generator calls) a turn.
template <int DIM>
__device__ __forceinline__ void feed_fp32(const Inst &I, const RunArgs &R, uint64_t traj_offset, const Feed &feed)
{
    const F32Consts c = f32_consts(I, R);
    const float shift = DIM == 2 ? 0.0f : c.adN;      // 2D: a constant bias shifts along e, in the step
    const PhiloxPre pre = philox_pre(traj_offset + feed.first + __lane_id(), I.instance, R.key0, R.key1);
    float4 *buf = reinterpret_cast<float4 *>(feed.buf) + __lane_id();
    uint32_t m = 0;
    for (uint32_t turn = 0;; ++turn) {
#pragma unroll
        for (int q = 0; q < DIM * kFeedSteps32 / 4; ++q) {
            uint32_t w[4];
            philox_call(m++, pre, R.key0, R.key1, w);
            float4 v;
            box_muller32(w[0], w[1], c.m2ln2_dN, shift, v.x, v.y);
            box_muller32(w[2], w[3], c.m2ln2_dN, shift, v.z, v.w);
            buf[64 * q] = v;
        }
        __syncthreads();
        if (!feed_goes_on(feed, turn)) break;
    }
}

// ---------------------------------------------------------------------------
// FP64 state with 2D noise (eq. full_langevin_equation): two normals per step,
// noise S (xi_1, xi_2) sqrt(dN) with S the interpolated symmetric square root of
// the covariance, bias B = a S e with e the interpolated principal axis, and
// dA = a e.xi sqrt(dN) + a^2 |e|^2 dN / 2, eq. (weight_A) for B = S (a e).  Step
// n takes call n >> 1 of the generator: (u0, u1) for step 2m, (u2, u3) for
// 2m + 1, so a group of two steps takes one call.  The structure (groups,
// event capture, claims) is that of lanes_fp64.
// ---------------------------------------------------------------------------
struct Node2d {
    double Spp, Spq, Sqq, e1, e2;
};

__device__ __forceinline__ Node2d lerp_node2d(const double2 *l_tab, int j, double f)
{
    const double2 a0 = l_tab[3 * j], a1 = l_tab[3 * j + 1], a2 = l_tab[3 * j + 2];
    const double2 b0 = l_tab[3 * j + 3], b1 = l_tab[3 * j + 4], b2 = l_tab[3 * j + 5];
    Node2d n;
    n.Spp = a0.x + f * (b0.x - a0.x);
    n.Spq = a0.y + f * (b0.y - a0.y);
    n.Sqq = a1.x + f * (b1.x - a1.x);
    n.e1 = a1.y + f * (b1.y - a1.y);
    n.e2 = a2.x + f * (b2.x - a2.x);
    return n;
}

template <int BIAS, bool ALLPOS, bool TIME, bool FEED = false>
__device__ __forceinline__ void lanes_fp64_2d(const Inst &I, const RunArgs &R, const double2 *l_tab,
                                              const RetireTo &rt, unsigned long long *cursor, uint64_t n_traj,
                                              uint64_t traj_offset, const Feed &feed = Feed{})
{
    const DriftConsts dk = drift_consts(I);
    const double dN = R.dN, sqrt_dN = R.sqrt_dN, phi_end = I.phi_end, phi_T = I.phi_T;
    const double a = (BIAS == kBiasConst) ? I.A : 0.0;
    const double half_a2_dN = 0.5 * a * a * dN;
    const uint32_t j_top = (uint32_t)(staged_nodes(I) - 2);
    const double2 *l_bm = l_tab + 3 * staged_nodes(I);
    const double s_plus = in_vgpr(dk.s_plus), s_minus = in_vgpr(dk.s_minus);

    bool exhausted = false;
    uint64_t rel = FEED ? feed.first + __lane_id() : 0;
    bool has = FEED ? rel < n_traj : claim(true, rel, cursor, n_traj, exhausted);
    bool live = has;
    double phi = I.phi_in, pi_ = I.pi_in, lnw = 0.0;
    uint32_t n = 0;
    PhiloxPre pre{};
    if (!FEED) pre = philox_pre(traj_offset + rel, I.instance, R.key0, R.key1);

    // Groups below the kink, as in lanes_fp64: two steps' reach, with the noise S (xi_1, xi_2) and the bias
    // a S e (|e| <= 1) bounded by twice the largest entry of S.
    const double reach =
        2.0 * (fmax(1.4143, fabs(I.pi_in)) * dN + 2.0 * I.S_max * (fabs(a) * dN + 6.8 * sqrt_dN));
    const double phi_below = (dk.s_plus == dk.s_minus) ? __builtin_inf() : phi_T - reach;

    // groups of two steps: one Philox call gives both steps' (xi_1, xi_2); without EVENTS as in lanes_fp64, in
    // paired waves only (in all waves 3e5 paths of 1e5 steps took 101.6 instead of 103.8 ms and 1e6 the same
    // 291, but 4e6 paths of 115 steps, most of whose groups are then taken twice, 3.9 instead of 3.4 ms)
    auto group = [&](auto censor_tag, auto below_tag, auto events_tag, const double z[4]) -> bool {
        constexpr bool CENSOR = decltype(censor_tag)::value;
        constexpr bool BELOW = decltype(below_tag)::value;
        constexpr bool EVENTS = decltype(events_tag)::value;
        const double phi0 = phi, pi0 = pi_, lnw0 = lnw;
        bool any_end = false;
        double eps1 = 0.0;          // pi^2/2 after the last step
        bool fresh = false;
        uint32_t ev_status, ev_n;   // written before use: read only where fresh is set
        double ev_N, ev_lnw;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (CENSOR && live && n == I.max_steps) {
                ev_status = kFlagCensored;
                ev_n = n;
                ev_N = __builtin_nan("");
                ev_lnw = lnw;
                live = false;
                fresh = true;
            }
            const double d = fma(phi, dk.kx, (!BELOW && phi >= phi_T) ? s_plus : s_minus);
            double r = __builtin_amdgcn_rcp(d);          // V'/V: reciprocal and one Newton step
            r = fma(r, fma(-d, r, 1.0), r);
            // table coordinate: phi, or the run's time n dN for a time-indexed table
            const double x = ((TIME ? (double)n * dN : phi) - I.phi_lo) * I.inv_h;
            const uint32_t jj = interval_of(x, j_top);
            const double f = fmin(fmax(x - (double)jj, 0.0), 1.0);
            const Node2d S = lerp_node2d(l_tab, (int)jj, f);
            const double z1 = z[2 * j], z2 = z[2 * j + 1];          // xi sqrt(dN)
            const double noise_phi = S.Spp * z1 + S.Spq * z2;
            const double noise_pi = S.Spq * z1 + S.Sqq * z2;
            // without a bias the amplitude is a literal 0, which IEEE arithmetic does not fold away:
            // the terms are left out instead (the same values, up to the sign of a zero)
            const double B_phi = a * (S.Spp * S.e1 + S.Spq * S.e2);
            const double B_pi = a * (S.Spq * S.e1 + S.Sqq * S.e2);
            const double phi_n =
                (BIAS == kBiasNone) ? phi + pi_ * dN + noise_phi : phi + (pi_ + B_phi) * dN + noise_phi;
            const double q_pi = (j == 0) ? fma(-pi_, 0.5 * pi_, 3.0) : 3.0 - eps1;      // as in lanes_fp64
            const double drift_pi = pi_ - q_pi * (pi_ + r) * dN;
            const double pi_n = (BIAS == kBiasNone) ? drift_pi + noise_pi : drift_pi + B_pi * dN + noise_pi;
            if (BIAS != kBiasNone) {
                const double dA = a * (S.e1 * z1 + S.e2 * z2) + half_a2_dN * (S.e1 * S.e1 + S.e2 * S.e2);
                if (ALLPOS) lnw -= dA;
                else lnw -= (S.Spp != 0.0 || S.Spq != 0.0 || S.Sqq != 0.0) ? dA : 0.0;
            }
            // as in lanes_fp64
            eps1 = half_sq(pi_n);
            const bool ends = (phi_n <= phi_end) | (eps1 >= 1.0);
            const bool hit = EVENTS && (live & ends);
            if (!EVENTS) any_end = any_end | ends;
            if (hit) {
                double pa = phi, pb = phi_n;
                uint32_t nb = n;
                asm volatile("; passage event" : "+v"(pa), "+v"(pb), "+v"(nb));
                const bool crossed = pb <= phi_end;
                ev_status = crossed ? 0u : kFlagEndedEarly;
                ev_n = nb + 1;
                ev_N = crossed ? (double)nb * dN + dN * ((pa - phi_end) / (pa - pb)) : (double)(nb + 1) * dN;
                ev_lnw = lnw;
            }
            live = live & !hit;
            fresh = fresh | hit;
            phi = phi_n;
            pi_ = pi_n;
            n += 1;
        }
        if (!EVENTS) {
            if (__builtin_amdgcn_ballot_w64(live && any_end) != 0) {
                phi = phi0;
                pi_ = pi0;
                lnw = lnw0;
                n -= 2;
                return false;
            }
        }
        if (fresh) retire(rt, rel, ev_status, ev_n, ev_N, ev_lnw);
        return true;
    };
    auto run_group = [&](bool may_cap, const double z[4]) {
        using Yes = std::integral_constant<bool, true>;
        using No = std::integral_constant<bool, false>;
        using Last = std::integral_constant<bool, !FEED>;      // paired waves: without events first
        if (may_cap) group(Yes(), No(), Yes(), z);
        else if (__builtin_amdgcn_ballot_w64(live && !(phi < phi_below)) == 0) {
            if (!group(No(), Yes(), Last(), z)) group(No(), Yes(), Yes(), z);
        } else if (!group(No(), No(), Last(), z)) group(No(), No(), Yes(), z);
    };

    if constexpr (FEED) {
        const double2 *buf = reinterpret_cast<const double2 *>(feed.buf) + __lane_id();
        for (uint32_t turn = 0;; ++turn) {
            __syncthreads();
            double2 v[kFeedSteps];
#pragma unroll
            for (int q = 0; q < kFeedSteps; ++q) v[q] = buf[64 * q];
            feed.flags[(turn & 1) * kFeedMaxPairs + feed.pair] = __any(live) ? 1u : 0u;
            if (!feed_goes_on(feed, turn)) break;
            if (!__any(live)) continue;
#pragma unroll
            for (int q = 0; q < kFeedSteps; q += 2) {
                const double z[4] = {v[q].x, v[q].y, v[q + 1].x, v[q + 1].y};
                run_group((uint32_t)__builtin_amdgcn_readfirstlane(n) + 2 > I.max_steps, z);
            }
        }
        return;
    }

    while (__any(has)) {
        const uint32_t left = wave_steps_left(has, n, I.max_steps);
        for (int k = 0; k < R.chunk; k += 2) {
            if (!__any(live)) break;
            uint32_t w[4];
            philox_call(n >> 1, pre, R.key0, R.key1, w);
            double z[4];
            box_muller64(w[0], w[1], sqrt_dN, l_bm, z[0], z[1]);
            box_muller64(w[2], w[3], sqrt_dN, l_bm, z[2], z[3]);
            run_group((uint32_t)k + 2 > left, z);
        }
        if (!live) has = false;
        if (claim(!has, rel, cursor, n_traj, exhausted)) {
            has = true;
            live = true;
            phi = I.phi_in;
            pi_ = I.pi_in;
            lnw = 0.0;
            n = 0;
            pre = philox_pre(traj_offset + rel, I.instance, R.key0, R.key1);
        }
    }
}

// ---------------------------------------------------------------------------
// FP32 state with 2D noise (eq. full_langevin_equation): the float-pair state of
// lanes_fp32 with the noise, bias and weight of lanes_fp64_2d.  Step n takes
// (xi_1, xi_2) from generator call n >> 1 as the FP64 2D path does ((u0, u1) for
// step 2m, (u2, u3) for step 2m + 1), so the two paths see the same numbers; a
// group of 16 steps takes eight calls.  Node record, three float4:
// (S_pp, slope, S_pq, slope), (S_qq, slope, e_phi, slope), (e_pi, slope, r, slope)
// with r = (V'/V) dN/2 interpolated in the interval, NaN where V'/V is computed
// exactly (as in the 1D FP32 table; all NaN on a time axis).  A constant bias
// B = a S e enters through shifted normals, B dN + S xi sqrt(dN) = S (xi sqrt(dN)
// + a dN e), and dA = a e.xi sqrt(dN) + a^2 |e|^2 dN/2 is summed per group in
// FP32 and across groups in FP64.
// ---------------------------------------------------------------------------
template <int BIAS, bool ALLPOS, bool TIME, bool FEED = false>
__device__ __forceinline__ void lanes_fp32_2d(const Inst &I, const RunArgs &R, const float4 *l_tab, const RetireTo &rt,
                                              unsigned long long *cursor, uint64_t n_traj, uint64_t traj_offset,
                                              const Feed &feed = Feed{})
{
    // steps per group: 16 (eight generator calls, the normals of the whole group formed first)
    constexpr int G = 16;
    const F32Consts c = f32_consts(I, R);
    const double x_in = I.phi_in - I.phi_end;
    const float x_in_hi = (float)x_in, x_in_lo = (float)(x_in - (double)x_in_hi);
    const float pi_in_hi = (float)I.pi_in, pi_in_lo = (float)(I.pi_in - (double)pi_in_hi);
    const double dN = R.dN;
    const float a = (BIAS == kBiasConst) ? (float)I.A : 0.0f;
    const float adN = a * c.dN;                 // the normals' shift per unit of e
    const float half_a2_dN = 0.5f * a * a * c.dN;
    const float s_plus = in_vgpr(c.s_plus), s_minus = in_vgpr(c.s_minus);

    bool exhausted = false;
    uint64_t rel = FEED ? feed.first + __lane_id() : 0;
    bool has = FEED ? rel < n_traj : claim(true, rel, cursor, n_traj, exhausted);
    bool live = has;
    float xh = x_in_hi, xl = x_in_lo, ph = pi_in_hi, pl = pi_in_lo;
    float xs = x_in_hi, ps = pi_in_hi;          // xs is formed each step only for a per-step lookup
    double lnw = 0.0;
    uint32_t n = 0;
    PhiloxPre pre{};
    if (!FEED) pre = philox_pre(traj_offset + rel, I.instance, R.key0, R.key1);

    // Phi tables: the lane's group-start record, as in lanes_fp32: each entry's value at x = xh
    // and its slope per unit x, so that a step of a lane whose start interval is smooth evaluates
    // every entry as value + slope * xl (the start interval's linear piece, extended past a node
    // the group's path passes); lanes in NaN-marked intervals read each step's own record.
    float g_v[6], g_d[6];           // S_pp, S_pq, S_qq, e_phi, e_pi, r
#pragma unroll
    for (int q = 0; q < 6; ++q) g_v[q] = g_d[q] = 0.0f;

    // without EVENTS as in lanes_fp64
    auto group = [&](auto censor_tag, auto span_tag, auto events_tag, const float z[2 * G]) -> bool {
        constexpr bool CENSOR = decltype(censor_tag)::value;
        constexpr bool SPAN = decltype(span_tag)::value;
        constexpr bool EVENTS = decltype(events_tag)::value;
        const float xl0 = xl, pl0 = pl, xs0 = xs, ps0 = ps;
        bool any_end = false;
        static_assert(!SPAN || (!TIME && !CENSOR), "one record per group: phi tables, no censoring");
        constexpr bool STEP_XS = !TIME && !SPAN;
        float zacc = 0.0f;        // this group's sum of dA
        bool fresh = false;
        uint32_t ev_code;
        double ev_N, ev_lnw;
#pragma unroll
        for (int j = 0; j < G; ++j) {
            if (CENSOR && live && n + j == I.max_steps) {
                ev_code = (n + j) | kFlagCensored;
                ev_N = __builtin_nan("");
                ev_lnw = lnw - (double)zacc;
                live = false;
                fresh = true;
            }
            float Spp, Spq, Sqq, e1, e2, r;     // r = (V'/V) dN/2
            if (SPAN) {
                Spp = fmaf(xl, g_d[0], g_v[0]);
                Spq = fmaf(xl, g_d[1], g_v[1]);
                Sqq = fmaf(xl, g_d[2], g_v[2]);
                e1 = fmaf(xl, g_d[3], g_v[3]);
                e2 = fmaf(xl, g_d[4], g_v[4]);
                r = fmaf(xl, g_d[5], g_v[5]);
            } else {
                const float u = __builtin_amdgcn_fmed3f(
                    TIME ? fmaf((float)(n + j), c.t_scale, c.t_off) : fmaf(xs, c.inv_h, c.u_off), 0.0f, c.jtop);
                const float f = __builtin_amdgcn_fractf(u);
                const float4 *rec = l_tab + 3 * (int)u;
                const float4 A0 = rec[0], A1 = rec[1], A2 = rec[2];
                Spp = fmaf(f, A0.y, A0.x);
                Spq = fmaf(f, A0.w, A0.z);
                Sqq = fmaf(f, A1.y, A1.x);
                e1 = fmaf(f, A1.w, A1.z);
                e2 = fmaf(f, A2.y, A2.x);
                r = fmaf(f, A2.w, A2.z);
                if (!TIME && g_v[5] == g_v[5]) {
                    // the lane's group-start interval is smooth: the arithmetic of a SPAN group
                    Spp = fmaf(xl, g_d[0], g_v[0]);
                    Spq = fmaf(xl, g_d[1], g_v[1]);
                    Sqq = fmaf(xl, g_d[2], g_v[2]);
                    e1 = fmaf(xl, g_d[3], g_v[3]);
                    e2 = fmaf(xl, g_d[4], g_v[4]);
                    r = fmaf(xl, g_d[5], g_v[5]);
                }
                if (__any(r != r)) {
                    asm volatile("; exact V'/V");
                    if (r != r) {
                        const float dT = (xh - c.xT_hi) + (xl - c.xT_lo);
                        r = __builtin_amdgcn_rcpf(fmaf(dT, c.kx, (dT >= 0.0f) ? s_plus : s_minus));
                    }
                }
            }
            const float z1 = z[2 * j], z2 = z[2 * j + 1];            // xi sqrt(dN)
            // noise plus bias through the shifted normals
            const float zb1 = (BIAS == kBiasConst) ? fmaf(adN, e1, z1) : z1;
            const float zb2 = (BIAS == kBiasConst) ? fmaf(adN, e2, z2) : z2;
            const float nphi = fmaf(Spp, zb1, Spq * zb2);
            const float npi = fmaf(Spq, zb1, Sqq * zb2);
            const float dx = fmaf(ps, c.dN, nphi);
            const float dpi = fmaf(fmaf(ps, ps, -6.0f), fmaf(ps, c.half_dN, r), npi);
            if (BIAS == kBiasConst) {
                const float dA = fmaf(a, fmaf(e1, z1, e2 * z2), half_a2_dN * fmaf(e1, e1, e2 * e2));
                zacc += (ALLPOS || Spp != 0.0f || Spq != 0.0f || Sqq != 0.0f) ? dA : 0.0f;
            }
            const float x0l = xl;
            xl += dx;
            pl += dpi;
            if (STEP_XS) xs = xh + xl;
            ps = ph + pl;
            // x <= 0: the sign of a rounded sum is that of the exact one, so this is xs <= 0
            const bool crossed = xl <= -xh;
            const bool ended = fabsf(ps) >= 0x1.6a09e8p+0f;
            const bool hit = EVENTS && live && (crossed || ended);
            if (!EVENTS) any_end = any_end | crossed | ended;
            if (hit) {
                float bh = xh, b0 = x0l, b1 = xl, bz = zacc;
                uint32_t nb = n + j;
                asm volatile("; passage event" : "+v"(bh), "+v"(b0), "+v"(b1), "+v"(nb), "+v"(bz));
                const double x0 = (double)bh + (double)b0;
                const double x1 = (double)bh + (double)b1;
                const double N_cross = (double)nb * dN + dN * (x0 / (x0 - x1));
                const double N_end = (double)(nb + 1) * dN;
                ev_code = (nb + 1) | (crossed ? 0u : kFlagEndedEarly);
                ev_N = crossed ? N_cross : N_end;
                ev_lnw = lnw - (double)bz;
            }
            live = live && !hit;
            fresh = fresh || hit;
        }
        if (!EVENTS) {
            if (__builtin_amdgcn_ballot_w64(live && any_end) != 0) {
                xl = xl0;
                pl = pl0;
                xs = xs0;
                ps = ps0;
                return false;
            }
        }
        n += G;
        lnw -= (double)zacc;
        if (fresh) retire(rt, rel, ev_code & ~kStepMask, ev_code & kStepMask, ev_N, ev_lnw);
        if (!STEP_XS) xs = xh + xl;
        xl = xl - (xs - xh);
        xh = xs;
        pl = pl - (ps - ph);
        ph = ps;
        return true;
    };
    // One group from its normals; `may_cap`: a lane may reach max_steps in it.
    auto run_group = [&](bool may_cap, const float z[2 * G]) {
        using T = std::integral_constant<bool, true>;
        using F = std::integral_constant<bool, false>;
        using L = std::integral_constant<bool, !FEED>;         // paired waves: without events first
        if constexpr (!TIME) {
            // the record of the lane's interval at the group start
            const float u0 = __builtin_amdgcn_fmed3f(fmaf(xh, c.inv_h, c.u_off), 0.0f, c.jtop);
            const int j0 = (int)u0;
            const float4 *rec = l_tab + 3 * j0;
            const float4 A0 = rec[0], A1 = rec[1], A2 = rec[2];
            const float fh = fmaf(xh, c.inv_h, c.u_off - (float)j0);   // the fraction at x = xh
            const float v0[6] = {A0.x, A0.z, A1.x, A1.z, A2.x, A2.z};
            const float d0[6] = {A0.y, A0.w, A1.y, A1.w, A2.y, A2.w};
#pragma unroll
            for (int q = 0; q < 6; ++q) {
                g_v[q] = fmaf(fh, d0[q], v0[q]);
                g_d[q] = d0[q] * c.inv_h;
            }
        }
        if (may_cap) {
            group(T(), F(), T(), z);
        } else {
            if constexpr (!TIME) {
                if (__builtin_amdgcn_ballot_w64(live && g_v[5] != g_v[5]) == 0) {
                    if (!group(F(), T(), L(), z)) group(F(), T(), T(), z);
                } else {
                    group(F(), F(), T(), z);
                }
            } else {
                if (!group(F(), F(), L(), z)) group(F(), F(), T(), z);
            }
        }
    };

    if constexpr (FEED) {
        static_assert(G == kFeedSteps32, "a turn is one group");
        const float4 *buf = reinterpret_cast<const float4 *>(feed.buf) + __lane_id();
        for (uint32_t turn = 0;; ++turn) {
            __syncthreads();
            float z[2 * G];
#pragma unroll
            for (int q = 0; q < G / 2; ++q) {
                const float4 v = buf[64 * q];
                z[4 * q] = v.x;
                z[4 * q + 1] = v.y;
                z[4 * q + 2] = v.z;
                z[4 * q + 3] = v.w;
            }
            feed.flags[(turn & 1) * kFeedMaxPairs + feed.pair] = __any(live) ? 1u : 0u;
            if (!feed_goes_on(feed, turn)) break;
            if (__any(live)) run_group((uint32_t)__builtin_amdgcn_readfirstlane(n) + G > I.max_steps, z);
        }
        return;
    }
    while (__any(has)) {
        const uint32_t left = wave_steps_left(has, n, I.max_steps);
        for (int k = 0; k < R.chunk; k += G) {
            if (!__any(live)) break;
            uint32_t w[2 * G];
#pragma unroll
            for (int q = 0; q < G / 2; ++q) philox_call((n >> 1) + (uint32_t)q, pre, R.key0, R.key1, w + 4 * q);
            float z[2 * G];
#pragma unroll
            for (int q = 0; q < 2 * G; q += 2) box_muller32(w[q], w[q + 1], c.m2ln2_dN, 0.0f, z[q], z[q + 1]);
            run_group((uint32_t)k + G > left, z);
        }
        if (!live) has = false;
        if (claim(!has, rel, cursor, n_traj, exhausted)) {
            has = true;
            live = true;
            xh = xs = x_in_hi;
            xl = x_in_lo;
            ph = ps = pi_in_hi;
            pl = pi_in_lo;
            lnw = 0.0;
            n = 0;
            pre = philox_pre(traj_offset + rel, I.instance, R.key0, R.key1);
        }
    }
}

// 2D staging: three double2 per node, then the Box-Muller tables.
__device__ __forceinline__ void stage_table64_2d(const Inst &I, double2 *l_tab)
{
    const int n = staged_nodes(I);
    for (int i = threadIdx.x; i < 3 * n; i += blockDim.x) l_tab[i] = I.tab64_2d[I.n_tab > 1 ? i : i % 3];
    stage_bm(l_tab + 3 * n);
}

// FP32 2D staging: three float4 per node, the V'/V interval (last pair) scaled by dN/2 (NaN kept);
// a single node is staged twice with zero slopes and a NaN interval.
__device__ __forceinline__ void stage_table32_2d(const Inst &I, float4 *l_tab, float dN)
{
    const int n = staged_nodes(I);
    for (int i = threadIdx.x; i < 3 * n; i += blockDim.x) {
        float4 v = I.tab32_2d[I.n_tab > 1 ? i : i % 3];
        if (i % 3 == 2) {
            v.z *= 0.5f * dN;
            v.w *= 0.5f * dN;
        }
        l_tab[i] = v;
    }
}

// ---------------------------------------------------------------------------
// LDS layout of the kernels: [accumulators][noise table][control cells][node
// weights], each part starting on a 16-byte boundary.
// ---------------------------------------------------------------------------
__host__ __device__ __forceinline__ size_t align16(size_t b) { return (b + 15) & ~(size_t)15; }
// FP64: double2 per node; FP32: float4 per node plus the float2 V'/V interval
// LDS of a staged table: FP64 nodes (16 B) and the Box-Muller tables, or FP32 nodes and V'/V
// intervals (24 B per node).
// 2D noise.  FP64: three double2 per node and the Box-Muller tables; FP32: three float4 per node
__host__ __device__ __forceinline__ size_t tab2d_bytes(int precision, int n_tab)
{
    return (size_t)(n_tab > 1 ? n_tab : 2) * 48 + (precision == 0 ? kBmBytes : 0);
}

__host__ __device__ __forceinline__ size_t tab_bytes(int precision, int n_tab)
{
    return align16((size_t)(n_tab > 1 ? n_tab : 2) * (precision == 0 ? 16 : 24)) + (precision == 0 ? kBmBytes : 0);
}
__host__ __device__ __forceinline__ size_t cell_bytes(int precision, int n_cells)
{
    return (size_t)n_cells * (precision == 0 ? 32 : 16);
}

template <int PREC>
__device__ __forceinline__ void stage_grid(const Inst &I, void *l_grid)
{
    const int nc = grid_cells(I);
    if (PREC == 0) {
        double2 *g = static_cast<double2 *>(l_grid);
        for (int i = threadIdx.x; i < 2 * nc; i += blockDim.x) g[i] = I.grid64[i];
    } else {
        float4 *g = static_cast<float4 *>(l_grid);
        for (int i = threadIdx.x; i < nc; i += blockDim.x) g[i] = I.grid32[i];
    }
}

// ---------------------------------------------------------------------------
// Single-problem kernels: a persistent grid over one instance.
// ---------------------------------------------------------------------------
__device__ __forceinline__ RetireTo retire_to(const EmParams &p, const LdsAcc &a)
{
    RetireTo r;
    r.d_N = p.d_N;
    r.d_lnw = p.d_lnw;
    r.d_steps = p.d_steps;
    r.cnt = a.cnt;
    r.sum = a.sum;
    r.nb = a.nb;
    r.hist = p.inst.hist;
    return r;
}

template <int PREC, int BIAS, int TAB, bool ALLPOS, int POT = kPotPiecewiseLinear>
__global__ void __launch_bounds__(BIAS == kBiasMlpMatrix ? kMaxBlockMatrix : 1024) FPT_EM_OCCUPANCY
em_kernel(EmParams p)
{
    static_assert(POT == kPotPiecewiseLinear || (PREC == 0 && (BIAS == kBiasNone || BIAS == kBiasConst)),
                  "the bump runs in FP64 only, without a learned bias");
    extern __shared__ __align__(16) unsigned char smem[];
    const LdsAcc acc = lds_acc(smem, p.inst.hist.n_bins);
    unsigned char *l_tab = smem + align16(acc_bytes(p.inst.hist.n_bins));
    unsigned char *l_grid = l_tab + tab_bytes(PREC, p.inst.n_tab);
    zero_lds_acc(acc);
    if (PREC == 0) stage_table64(p.inst, reinterpret_cast<double2 *>(l_tab));
    else stage_table32(p.inst, reinterpret_cast<float4 *>(l_tab), (float)p.run.dN);
    if (BIAS == kBiasMlp) stage_grid<PREC>(p.inst, l_grid);
    if (BIAS == kBiasMlpExact && PREC == 0) stage_mlp64(p.inst.mlp_params, reinterpret_cast<double *>(l_grid));
    if (BIAS == kBiasMlpMatrix) stage_mlp32(p.inst.mlp_params, reinterpret_cast<float *>(l_grid));
    __syncthreads();
    const RetireTo rt = retire_to(p, acc);
    const ReplayTo rp{nullptr, nullptr, nullptr};
    if (PREC == 0)
        lanes_fp64<BIAS, TAB, ALLPOS, kGradNone, POT>(p.inst, p.run, reinterpret_cast<const double2 *>(l_tab),
                                                  reinterpret_cast<const double2 *>(l_grid), rt, rp, p.cursor,
                                                  p.n_traj, p.traj_offset);
    else
        lanes_fp32<BIAS, TAB, ALLPOS, kGradNone>(p.inst, p.run, reinterpret_cast<const float4 *>(l_tab),
                                             reinterpret_cast<const float4 *>(l_grid), rt, rp, p.cursor, p.n_traj,
                                             p.traj_offset);
    __syncthreads();
    flush_lds_acc(acc, p.inst.acc);
}

// One block of paired waves (see Feed): trajectories traj_offset + first .. of instance I, one per lane of
// the block's first half of waves, of n_traj in all; the second half forms their normals.
template <int PREC, int BIAS, int TAB, bool ALLPOS, int POT>
__device__ __forceinline__ void pair_block(const Inst &I, const RunArgs &R, unsigned char *smem, uint32_t *flags,
                                           double *d_N, double *d_lnw, uint32_t *d_steps, uint64_t n_traj,
                                           uint64_t traj_offset, uint64_t first)
{
    const LdsAcc acc = lds_acc(smem, I.hist.n_bins);
    unsigned char *l_tab = smem + align16(acc_bytes(I.hist.n_bins));
    unsigned char *l_feed = l_tab + tab_bytes(PREC, I.n_tab);
    zero_lds_acc(acc);
    if (PREC == 0) stage_table64(I, reinterpret_cast<double2 *>(l_tab));
    else stage_table32(I, reinterpret_cast<float4 *>(l_tab), (float)R.dN);
    __syncthreads();
    const RetireTo rt{d_N, d_lnw, d_steps, acc.cnt, acc.sum, acc.nb, I.hist};
    const ReplayTo rp{nullptr, nullptr, nullptr};
    const int wave = (int)(__builtin_amdgcn_readfirstlane(threadIdx.x) / 64), pairs = (int)(blockDim.x / 128);
    const int pair = wave < pairs ? wave : wave - pairs;
    const Feed feed{l_feed + (size_t)pair * kFeedBytes, flags, pair, pairs, first + (uint64_t)pair * 64};
    if (wave < pairs) {
        if (PREC == 0)
            lanes_fp64<BIAS, TAB, ALLPOS, kGradNone, POT, true>(I, R, reinterpret_cast<const double2 *>(l_tab), nullptr,
                                                            rt, rp, nullptr, n_traj, traj_offset, feed);
        else
            lanes_fp32<BIAS, TAB, ALLPOS, kGradNone, true>(I, R, reinterpret_cast<const float4 *>(l_tab), nullptr, rt, rp,
                                                       nullptr, n_traj, traj_offset, feed);
    } else {
        if (PREC == 0)
            feed_fp64<1>(I, R, reinterpret_cast<const double2 *>(l_tab) + staged_nodes(I), traj_offset, feed);
        else feed_fp32<1>(I, R, traj_offset, feed);
    }
    __syncthreads();
    flush_lds_acc(acc, I.acc);
}

// A run on paired waves.  The grid covers the trajectories; p.cursor is not used.
template <int PREC, int BIAS, int TAB, bool ALLPOS, int POT = kPotPiecewiseLinear>
__global__ void __launch_bounds__(64 * 2 * kFeedMaxPairs) em_pair_kernel(EmParams p)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint32_t flags[2 * kFeedMaxPairs];
    pair_block<PREC, BIAS, TAB, ALLPOS, POT>(p.inst, p.run, smem, flags, p.d_N, p.d_lnw, p.d_steps, p.n_traj,
                                             p.traj_offset, (uint64_t)blockIdx.x * (blockDim.x / 2));
}

// A batch on paired waves: block b runs the slice items[b] of its instance, at most one trajectory per
// lane of its integrating waves.
template <int PREC, int BIAS, bool ALLPOS>
__global__ void __launch_bounds__(64 * 2 * kFeedMaxPairs) batch_pair_kernel(const Inst *insts, const WorkItem *items,
                                                                            RunArgs run)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint32_t flags[2 * kFeedMaxPairs];
    const WorkItem W = items[blockIdx.x];
    const Inst I = insts[W.inst];
    pair_block<PREC, BIAS, 1, ALLPOS, kPotPiecewiseLinear>(I, run, smem, flags, nullptr, nullptr, nullptr, W.count,
                                                           W.begin, 0);
}

// 2D noise, FP64 or FP32 state: a persistent grid over one instance.
template <int PREC, int BIAS, bool ALLPOS, bool TIME>
__global__ void __launch_bounds__(1024) FPT_EM_OCCUPANCY em2d_kernel(EmParams p)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const LdsAcc acc = lds_acc(smem, p.inst.hist.n_bins);
    unsigned char *l_tab = smem + align16(acc_bytes(p.inst.hist.n_bins));
    zero_lds_acc(acc);
    if (PREC == 0) stage_table64_2d(p.inst, reinterpret_cast<double2 *>(l_tab));
    else stage_table32_2d(p.inst, reinterpret_cast<float4 *>(l_tab), (float)p.run.dN);
    __syncthreads();
    const RetireTo rt = retire_to(p, acc);
    if (PREC == 0)
        lanes_fp64_2d<BIAS, ALLPOS, TIME>(p.inst, p.run, reinterpret_cast<const double2 *>(l_tab), rt, p.cursor,
                                          p.n_traj, p.traj_offset);
    else
        lanes_fp32_2d<BIAS, ALLPOS, TIME>(p.inst, p.run, reinterpret_cast<const float4 *>(l_tab), rt, p.cursor,
                                          p.n_traj, p.traj_offset);
    __syncthreads();
    flush_lds_acc(acc, p.inst.acc);
}

// A 2D-noise run on paired waves: pair_block with the 2D lanes and twice the buffer.
template <int PREC, int BIAS, bool ALLPOS, bool TIME>
__global__ void __launch_bounds__(64 * 2 * kFeedMaxPairs) em2d_pair_kernel(EmParams p)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint32_t flags[2 * kFeedMaxPairs];
    const LdsAcc acc = lds_acc(smem, p.inst.hist.n_bins);
    unsigned char *l_tab = smem + align16(acc_bytes(p.inst.hist.n_bins));
    unsigned char *l_feed = l_tab + tab2d_bytes(PREC, p.inst.n_tab);
    zero_lds_acc(acc);
    if (PREC == 0) stage_table64_2d(p.inst, reinterpret_cast<double2 *>(l_tab));
    else stage_table32_2d(p.inst, reinterpret_cast<float4 *>(l_tab), (float)p.run.dN);
    __syncthreads();
    const RetireTo rt = retire_to(p, acc);
    const int wave = (int)(__builtin_amdgcn_readfirstlane(threadIdx.x) / 64), pairs = (int)(blockDim.x / 128);
    const int pair = wave < pairs ? wave : wave - pairs;
    const Feed feed{l_feed + (size_t)pair * 2 * kFeedBytes, flags, pair, pairs,
                    (uint64_t)blockIdx.x * (blockDim.x / 2) + (uint64_t)pair * 64};
    if (wave < pairs) {
        if (PREC == 0)
            lanes_fp64_2d<BIAS, ALLPOS, TIME, true>(p.inst, p.run, reinterpret_cast<const double2 *>(l_tab), rt, nullptr,
                                                    p.n_traj, p.traj_offset, feed);
        else
            lanes_fp32_2d<BIAS, ALLPOS, TIME, true>(p.inst, p.run, reinterpret_cast<const float4 *>(l_tab), rt, nullptr,
                                                    p.n_traj, p.traj_offset, feed);
    } else {
        if (PREC == 0)
            feed_fp64<2>(p.inst, p.run, reinterpret_cast<const double2 *>(l_tab) + 3 * staged_nodes(p.inst),
                         p.traj_offset, feed);
        else feed_fp32<2>(p.inst, p.run, p.traj_offset, feed);
    }
    __syncthreads();
    flush_lds_acc(acc, p.inst.acc);
}

// Replay kernel: the listed trajectories with the tabulated control, scattering
// gradient factors onto the grid nodes (LDS, then global atomics).
template <int PREC, bool ALLPOS>
__global__ void __launch_bounds__(1024) FPT_EM_OCCUPANCY replay_kernel(ReplayParams p)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const Inst &I = p.inst;
    unsigned char *l_tab = smem;
    unsigned char *l_grid = l_tab + tab_bytes(PREC, I.n_tab);
    double *l_G = reinterpret_cast<double *>(l_grid + cell_bytes(PREC, grid_cells(I)));
    const int n_nodes = I.g_n0 * I.g_n1;
    const uint64_t n_tail = *p.n_tail;
    if (n_tail == 0) return;
    for (int i = threadIdx.x; i < n_nodes; i += blockDim.x) l_G[i] = 0.0;
    if (PREC == 0) stage_table64(I, reinterpret_cast<double2 *>(l_tab));
    else stage_table32(I, reinterpret_cast<float4 *>(l_tab), (float)p.run.dN);
    stage_grid<PREC>(I, l_grid);
    __syncthreads();
    RetireTo rt{};
    const ReplayTo rp{p.tail, l_G, p.mismatch};
    // The list's length is known on the device alone, so the grid is a full one; where the list does not
    // fill it, each block's first ceil(waves/blocks) waves share it (as run_shape does for fpt_run).
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x) / 64;
    if (wave >= ((n_tail + 63) / 64 + gridDim.x - 1) / gridDim.x) {
        // nothing to replay here
    } else if (PREC == 0)
        lanes_fp64<kBiasMlp, 1, ALLPOS, kGradReplay>(I, p.run, reinterpret_cast<const double2 *>(l_tab),
                                                 reinterpret_cast<const double2 *>(l_grid), rt, rp, p.cursor, n_tail,
                                                 0);
    else
        lanes_fp32<kBiasMlp, 1, ALLPOS, kGradReplay>(I, p.run, reinterpret_cast<const float4 *>(l_tab),
                                                 reinterpret_cast<const float4 *>(l_grid), rt, rp, p.cursor, n_tail,
                                                 0);
    __syncthreads();
    for (int i = threadIdx.x; i < n_nodes; i += blockDim.x)
        if (l_G[i] != 0.0) unsafeAtomicAdd(&p.d_G[i], l_G[i]);
}

// Recording run: em_kernel's tabulated control, with each path's gradient sums per visited cell kept.
// PAIRED: on paired waves, as em_pair_kernel (a training step on 5000 trajectories 20.4 -> 18.4 ms, on
// 100,000 25.3 -> 21.6; the integrating wave, some 440 cycles a step with its cell's sums, is the longer side).
template <int PREC, int TAB, bool ALLPOS, bool PAIRED>
__global__ void __launch_bounds__(1024) FPT_EM_OCCUPANCY em_record_kernel(EmParams p, RecordPool rec)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const LdsAcc acc = lds_acc(smem, p.inst.hist.n_bins);
    unsigned char *l_tab = smem + align16(acc_bytes(p.inst.hist.n_bins));
    unsigned char *l_grid = l_tab + tab_bytes(PREC, p.inst.n_tab);
    zero_lds_acc(acc);
    if (PREC == 0) stage_table64(p.inst, reinterpret_cast<double2 *>(l_tab));
    else stage_table32(p.inst, reinterpret_cast<float4 *>(l_tab), (float)p.run.dN);
    stage_grid<PREC>(p.inst, l_grid);
    __syncthreads();
    const RetireTo rt = retire_to(p, acc);
    const ReplayTo rp{nullptr, nullptr, nullptr, rec};
    if (PAIRED) {
        __shared__ uint32_t flags[2 * kFeedMaxPairs];
        unsigned char *l_feed = l_grid + cell_bytes(PREC, grid_cells(p.inst));
        const int wave = (int)(__builtin_amdgcn_readfirstlane(threadIdx.x) / 64), pairs = (int)(blockDim.x / 128);
        const int pair = wave < pairs ? wave : wave - pairs;
        const Feed feed{l_feed + (size_t)pair * kFeedBytes, flags, pair, pairs,
                        (uint64_t)blockIdx.x * (blockDim.x / 2) + (uint64_t)pair * 64};
        if (wave >= pairs) {
            if (PREC == 0)
                feed_fp64<1>(p.inst, p.run, reinterpret_cast<const double2 *>(l_tab) + staged_nodes(p.inst),
                             p.traj_offset, feed);
            else feed_fp32<1>(p.inst, p.run, p.traj_offset, feed);
        } else if (PREC == 0) {
            lanes_fp64<kBiasMlp, TAB, ALLPOS, kGradRecord, kPotPiecewiseLinear, true>(
                p.inst, p.run, reinterpret_cast<const double2 *>(l_tab), reinterpret_cast<const double2 *>(l_grid), rt,
                rp, nullptr, p.n_traj, p.traj_offset, feed);
        } else {
            lanes_fp32<kBiasMlp, TAB, ALLPOS, kGradRecord, true>(
                p.inst, p.run, reinterpret_cast<const float4 *>(l_tab), reinterpret_cast<const float4 *>(l_grid), rt, rp,
                nullptr, p.n_traj, p.traj_offset, feed);
        }
    } else if (PREC == 0)
        lanes_fp64<kBiasMlp, TAB, ALLPOS, kGradRecord>(p.inst, p.run, reinterpret_cast<const double2 *>(l_tab),
                                                       reinterpret_cast<const double2 *>(l_grid), rt, rp, p.cursor,
                                                       p.n_traj, p.traj_offset);
    else
        lanes_fp32<kBiasMlp, TAB, ALLPOS, kGradRecord>(p.inst, p.run, reinterpret_cast<const float4 *>(l_tab),
                                                       reinterpret_cast<const float4 *>(l_grid), rt, rp, p.cursor,
                                                       p.n_traj, p.traj_offset);
    __syncthreads();
    flush_lds_acc(acc, p.inst.acc);
}

// After a recording run: every path of the tail T (crossed with deltaN >= tail_lo) adds w^2 times its
// recorded sums to the node weights G, and w^2 and 1 to J_sum and n_tail_total; a path with more records
// than the pool has room for goes on the replay list instead.  A wave takes one path at a time, a lane
// one record; node weights are summed in LDS first.
template <typename T>
__global__ void __launch_bounds__(1024) tail_weigh_kernel(const double *d_N, const double *d_lnw, const uint32_t *d_steps,
                                                          uint64_t n, uint64_t traj_offset, double N_ref,
                                                          double tail_lo, RecordPool rec, int n0, int n1, double *d_G,
                                                          TailEntry *tail, unsigned long long *n_tail,
                                                          unsigned long long *n_tail_total, double *J_sum)
{
    extern __shared__ __align__(16) unsigned char smem[];
    double *l_G = reinterpret_cast<double *>(smem);
    for (int i = threadIdx.x; i < n0 * n1; i += blockDim.x) l_G[i] = 0.0;
    __syncthreads();
    const ReplayTo rp{nullptr, l_G, nullptr};
    const int lane = (int)__lane_id(), waves = (int)(gridDim.x * (blockDim.x / 64));
    double j_sum = 0.0;
    unsigned long long count = 0;
    for (uint64_t i = blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64; i < n; i += waves) {
        if ((d_steps[i] & (kFlagCensored | kFlagEndedEarly)) != 0u || !(d_N[i] - N_ref >= tail_lo)) continue;
        const double ww = exp(2.0 * d_lnw[i]);
        j_sum += ww;
        ++count;
        const uint32_t k = rec.count[i];
        if (k > rec.cap) {
            if (lane == 0) tail[atomicAdd(n_tail, 1ull)] = TailEntry{traj_offset + i, ww};
            continue;
        }
        for (uint32_t r = lane; r < k; r += 64) {
            const uint64_t at = i * rec.cap + r;
            const T *q = static_cast<const T *>(rec.sums) + 4 * at;
            T v[4] = {q[0], q[1], q[2], q[3]};
            grad_flush(rp, n1 - 1, (int)rec.cell[at], v, ww);
        }
    }
    if (lane == 0 && count != 0) {
        unsafeAtomicAdd(J_sum, j_sum);
        atomicAdd(n_tail_total, count);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n0 * n1; i += blockDim.x)
        if (l_G[i] != 0.0) unsafeAtomicAdd(&d_G[i], l_G[i]);
}

// ---------------------------------------------------------------------------
// Batch kernel: a persistent grid over many instances.  Each instance has a
// trajectory cursor of its own (cursors[1 + i], over its whole range of the
// run).  The work list holds tickets, each sending a block to one instance
// (ordered so that the blocks spread over the instances in proportion to their
// estimated cost), then one entry per instance, longest estimated cost first.
// A block takes a ticket (cursors[0]) and skips it when its instance has no
// trajectory left; otherwise it stages that instance's table and histogram in
// LDS, and its waves claim the instance's trajectories from its global cursor
// until all are claimed, as in the single-instance kernel.  It then flushes the
// histogram and takes the next ticket; once the tickets are used up it joins
// any instance that still has trajectories left.  A block leaves an instance
// only when the instance has no trajectory left, so its lanes drain once per
// instance it works on, not once per ticket.  Every selection either finds an
// instance with trajectories left or ends the block's loop, and an instance
// found empty is never selected again: the loop ends.  The run parameters are
// read from device memory so that a captured graph can be replayed with a new
// seed or time step.
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool has_left(const WorkItem &W, unsigned long long *cursors)
{
    return __hip_atomic_load(&cursors[1 + W.inst], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < W.count;
}

template <int PREC, int BIAS, bool ALLPOS>
__global__ void __launch_bounds__(1024) FPT_EM_OCCUPANCY batch_kernel(const Inst *insts, const WorkItem *items,
                                                                      const BatchRun *brun,
                                                                      unsigned long long *cursors, int max_bins)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ long long s_sel;
    const RunArgs R = brun->run;
    const uint64_t n_items = brun->n_items, n_inst = brun->n_inst;
    uint64_t scan = 0;     // thread 0: the next per-instance entry to look at once the tickets are used up
    for (;;) {
        if (threadIdx.x == 0) {
            long long sel = -1;
            for (;;) {
                const uint64_t t = atomicAdd(&cursors[0], 1ull);
                if (t >= n_items) break;
                if (has_left(items[t], cursors)) {
                    sel = (long long)t;
                    break;
                }
            }
            for (; sel < 0 && scan < n_inst; ++scan)
                if (has_left(items[n_items + scan], cursors)) sel = (long long)(n_items + scan);
            s_sel = sel;
        }
        __syncthreads();
        const long long sel = s_sel;
        if (sel < 0) break;
        const WorkItem W = items[sel];
        const Inst I = insts[W.inst];
        const LdsAcc acc = lds_acc(smem, I.hist.n_bins);
        unsigned char *l_tab = smem + align16(acc_bytes(max_bins));
        zero_lds_acc(acc);
        if (PREC == 0) stage_table64(I, reinterpret_cast<double2 *>(l_tab));
        else stage_table32(I, reinterpret_cast<float4 *>(l_tab), (float)R.dN);
        __syncthreads();
        RetireTo rt;
        rt.d_N = nullptr;
        rt.d_lnw = nullptr;
        rt.d_steps = nullptr;
        rt.cnt = acc.cnt;
        rt.sum = acc.sum;
        rt.nb = acc.nb;
        rt.hist = I.hist;
        const ReplayTo rp{nullptr, nullptr, nullptr};
        if (PREC == 0)
            lanes_fp64<BIAS, 1, ALLPOS, kGradNone>(I, R, reinterpret_cast<const double2 *>(l_tab), nullptr, rt, rp,
                                                  &cursors[1 + W.inst], W.count, W.begin);
        else
            lanes_fp32<BIAS, 1, ALLPOS, kGradNone>(I, R, reinterpret_cast<const float4 *>(l_tab), nullptr, rt, rp,
                                                  &cursors[1 + W.inst], W.count, W.begin);
        __syncthreads();
        flush_lds_acc(acc, I.acc);
        __syncthreads();
    }
}

__global__ void zero_words_kernel(unsigned long long *ptr, size_t n)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        ptr[i] = 0ull;
}

template <int PREC, int BIAS, int TAB, bool ALLPOS, int POT = kPotPiecewiseLinear>
const void *pptr() { return reinterpret_cast<const void *>(&em_pair_kernel<PREC, BIAS, TAB, ALLPOS, POT>); }
template <int PREC, int BIAS, int TAB, bool ALLPOS, int POT = kPotPiecewiseLinear>
const void *kptr() { return reinterpret_cast<const void *>(&em_kernel<PREC, BIAS, TAB, ALLPOS, POT>); }
template <int PREC, int BIAS, bool ALLPOS>
const void *bptr() { return reinterpret_cast<const void *>(&batch_kernel<PREC, BIAS, ALLPOS>); }

// (none for a learned control on a time table, which fpt_create refuses)
template <int PREC, int BIAS>
struct KTab {
    template <bool ALLPOS>
    static const void *on_time()
    {
        if constexpr (BIAS == kBiasNone || BIAS == kBiasConst) return kptr<PREC, BIAS, 2, ALLPOS>();
        else return nullptr;
    }
    const void *p[3][2] = {{kptr<PREC, BIAS, 0, false>(), kptr<PREC, BIAS, 0, true>()},
                           {kptr<PREC, BIAS, 1, false>(), kptr<PREC, BIAS, 1, true>()},
                           {on_time<false>(), on_time<true>()}};
};

}  // namespace

size_t em_lds_bytes(int n_bins, int n_tab, int precision, int n_cells, int bias_kind)
{
    // the exact network stages its parameters (FP64), its second layer's (matrix cores) or nothing instead of the
    // tabulated cells
    const size_t bias = bias_kind == kBiasMlpMatrix  ? kMlpLdsBytes32
                        : bias_kind == kBiasMlpExact ? (precision == 0 ? kMlpLdsBytes64 : 0)
                                                     : cell_bytes(precision, n_cells);
    return align16(acc_bytes(n_bins)) + tab_bytes(precision, n_tab) + bias;
}

size_t replay_lds_bytes(int n_tab, int precision, int n_cells, int n_nodes)
{
    return tab_bytes(precision, n_tab) + cell_bytes(precision, n_cells) + (size_t)n_nodes * 8;
}

const void *em_kernel_ptr(int precision, int bias_kind, int tab_mode, bool all_pos, int pot_kind)
{
    const int tm = tab_mode < 0 ? 0 : tab_mode > 2 ? 2 : tab_mode;
    if (pot_kind == kPotGaussianBump) {
        // FP64, bias none or constant (fpt_create rejects the rest)
        constexpr int B = kPotGaussianBump;
        static const void *const tb[2][3][2] = {
            {{kptr<0, kBiasNone, 0, false, B>(), kptr<0, kBiasNone, 0, true, B>()},
             {kptr<0, kBiasNone, 1, false, B>(), kptr<0, kBiasNone, 1, true, B>()},
             {kptr<0, kBiasNone, 2, false, B>(), kptr<0, kBiasNone, 2, true, B>()}},
            {{kptr<0, kBiasConst, 0, false, B>(), kptr<0, kBiasConst, 0, true, B>()},
             {kptr<0, kBiasConst, 1, false, B>(), kptr<0, kBiasConst, 1, true, B>()},
             {kptr<0, kBiasConst, 2, false, B>(), kptr<0, kBiasConst, 2, true, B>()}}};
        return tb[bias_kind == kBiasConst ? 1 : 0][tm][all_pos ? 1 : 0];
    }
    static const KTab<0, kBiasNone> f0n;
    static const KTab<0, kBiasConst> f0c;
    static const KTab<0, kBiasMlp> f0m;
    static const KTab<0, kBiasMlpExact> f0x;
    static const KTab<1, kBiasNone> f1n;
    static const KTab<1, kBiasConst> f1c;
    static const KTab<1, kBiasMlp> f1m;
    static const KTab<1, kBiasMlpExact> f1x;
    static const KTab<1, kBiasMlpMatrix> f1m32;
    const void *const(*t)[2];
    if (precision == 0)
        t = bias_kind == kBiasNone ? f0n.p : bias_kind == kBiasConst ? f0c.p : bias_kind == kBiasMlp ? f0m.p : f0x.p;
    else
        t = bias_kind == kBiasNone ? f1n.p : bias_kind == kBiasConst ? f1c.p : bias_kind == kBiasMlp ? f1m.p
            : bias_kind == kBiasMlpExact ? f1x.p : f1m32.p;
    return t[tm][all_pos ? 1 : 0];
}

template <int PREC, int BIAS, int POT>
struct PTab {
    const void *p[3][2] = {{pptr<PREC, BIAS, 0, false, POT>(), pptr<PREC, BIAS, 0, true, POT>()},
                           {pptr<PREC, BIAS, 1, false, POT>(), pptr<PREC, BIAS, 1, true, POT>()},
                           {pptr<PREC, BIAS, 2, false, POT>(), pptr<PREC, BIAS, 2, true, POT>()}};
};

const void *em_pair_kernel_ptr(int precision, int bias_kind, int tab_mode, bool all_pos, int pot_kind)
{
    static const PTab<0, kBiasNone, kPotGaussianBump> bn;
    static const PTab<0, kBiasConst, kPotGaussianBump> bc;
    static const PTab<0, kBiasNone, kPotPiecewiseLinear> dn;
    static const PTab<0, kBiasConst, kPotPiecewiseLinear> dc;
    static const PTab<1, kBiasNone, kPotPiecewiseLinear> fn;
    static const PTab<1, kBiasConst, kPotPiecewiseLinear> fc;
    if (bias_kind != kBiasNone && bias_kind != kBiasConst) return nullptr;
    const bool c = bias_kind == kBiasConst;
    const void *const(*t)[2] = pot_kind == kPotGaussianBump ? (c ? bc.p : bn.p)
                               : precision == 0             ? (c ? dc.p : dn.p)
                                                            : (c ? fc.p : fn.p);
    return t[tab_mode][all_pos ? 1 : 0];
}

hipError_t em_launch(const EmParams &p, int precision, int bias_kind, int grid, int block, hipStream_t stream)
{
    const size_t lds = em_lds_bytes(p.inst.hist.n_bins, p.inst.n_tab, precision, grid_cells(p.inst), bias_kind);
    const void *fn = em_kernel_ptr(precision, bias_kind, tab_mode(p.inst),
                                   p.inst.all_S_pos != 0, p.inst.pot_kind);
    EmParams pp = p;
    void *args[] = {&pp};
    return hipLaunchKernel(fn, dim3(grid), dim3(block), args, lds, stream);
}

size_t em2d_lds_bytes(int n_bins, int n_tab, int precision)
{
    return align16(acc_bytes(n_bins)) + tab2d_bytes(precision, n_tab);
}

template <int PREC, int BIAS>
struct K2Tab {
    const void *p[2][2] = {{reinterpret_cast<const void *>(&em2d_kernel<PREC, BIAS, false, false>),
                            reinterpret_cast<const void *>(&em2d_kernel<PREC, BIAS, false, true>)},
                           {reinterpret_cast<const void *>(&em2d_kernel<PREC, BIAS, true, false>),
                            reinterpret_cast<const void *>(&em2d_kernel<PREC, BIAS, true, true>)}};
};

const void *em2d_kernel_ptr(int precision, int bias_kind, bool all_pos, bool time_axis)
{
    static const K2Tab<0, kBiasNone> d_n;
    static const K2Tab<0, kBiasConst> d_c;
    static const K2Tab<1, kBiasNone> f_n;
    static const K2Tab<1, kBiasConst> f_c;
    const bool c = bias_kind != kBiasNone;
    const void *const(*t)[2] = precision == 0 ? (c ? d_c.p : d_n.p) : (c ? f_c.p : f_n.p);
    return t[all_pos ? 1 : 0][time_axis ? 1 : 0];
}

// nullptr for the FP32 state on a time table: its group of 16 steps holds 32 normals beside a record per step,
// and with the group's start saved it spills; 1000 trajectories (slow roll -> ultra-slow roll, 2048 time nodes)
// took 35.8 ms on paired waves and take 25.2 unpaired, with a constant bias 57.1 and 29.6 (65,536: 36.6 and 26.7, 82.9
// and 31.2).
template <int PREC, int BIAS>
struct P2Tab {
    template <bool ALLPOS>
    static const void *on_time()
    {
        if constexpr (PREC == 0) return reinterpret_cast<const void *>(&em2d_pair_kernel<PREC, BIAS, ALLPOS, true>);
        else return nullptr;
    }
    const void *p[2][2] = {{reinterpret_cast<const void *>(&em2d_pair_kernel<PREC, BIAS, false, false>), on_time<false>()},
                           {reinterpret_cast<const void *>(&em2d_pair_kernel<PREC, BIAS, true, false>), on_time<true>()}};
};

const void *em2d_pair_kernel_ptr(int precision, int bias_kind, bool all_pos, bool time_axis)
{
    static const P2Tab<0, kBiasNone> d_n;
    static const P2Tab<0, kBiasConst> d_c;
    static const P2Tab<1, kBiasNone> f_n;
    static const P2Tab<1, kBiasConst> f_c;
    const bool c = bias_kind != kBiasNone;
    const void *const(*t)[2] = precision == 0 ? (c ? d_c.p : d_n.p) : (c ? f_c.p : f_n.p);
    return t[all_pos ? 1 : 0][time_axis ? 1 : 0];
}

hipError_t em2d_launch(const EmParams &p, int precision, int grid, int block, hipStream_t stream)
{
    const size_t lds = em2d_lds_bytes(p.inst.hist.n_bins, p.inst.n_tab, precision);
    const void *fn = em2d_kernel_ptr(precision, p.inst.bias_kind, p.inst.all_S_pos != 0, tab_mode(p.inst) == 2);
    EmParams pp = p;
    void *args[] = {&pp};
    return hipLaunchKernel(fn, dim3(grid), dim3(block), args, lds, stream);
}

const void *replay_kernel_ptr(int precision, bool all_pos)
{
    static const void *const t[2][2] = {
        {reinterpret_cast<const void *>(&replay_kernel<0, false>), reinterpret_cast<const void *>(&replay_kernel<0, true>)},
        {reinterpret_cast<const void *>(&replay_kernel<1, false>), reinterpret_cast<const void *>(&replay_kernel<1, true>)}};
    return t[precision ? 1 : 0][all_pos ? 1 : 0];
}

hipError_t replay_launch(const ReplayParams &p, int precision, int grid, int block, hipStream_t stream)
{
    const size_t lds = replay_lds_bytes(p.inst.n_tab, precision, grid_cells(p.inst), p.inst.g_n0 * p.inst.g_n1);
    const void *fn = replay_kernel_ptr(precision, p.inst.all_S_pos != 0);
    ReplayParams pp = p;
    void *args[] = {&pp};
    return hipLaunchKernel(fn, dim3(grid), dim3(block), args, lds, stream);
}

template <int PREC, bool PAIRED>
const void *rptr(int tab_mode, bool all_pos)
{
    static const void *const t[2][2] = {{reinterpret_cast<const void *>(&em_record_kernel<PREC, 0, false, PAIRED>),
                                         reinterpret_cast<const void *>(&em_record_kernel<PREC, 0, true, PAIRED>)},
                                        {reinterpret_cast<const void *>(&em_record_kernel<PREC, 1, false, PAIRED>),
                                         reinterpret_cast<const void *>(&em_record_kernel<PREC, 1, true, PAIRED>)}};
    return t[tab_mode ? 1 : 0][all_pos ? 1 : 0];
}

const void *em_record_kernel_ptr(int precision, int tab_mode, bool all_pos, bool paired)
{
    if (paired) return precision == 0 ? rptr<0, true>(tab_mode, all_pos) : rptr<1, true>(tab_mode, all_pos);
    return precision == 0 ? rptr<0, false>(tab_mode, all_pos) : rptr<1, false>(tab_mode, all_pos);
}

hipError_t em_record_launch(const EmParams &p, const RecordPool &rec, int precision, int grid, int block, int pairs,
                            hipStream_t stream)
{
    EmParams pp = p;
    RecordPool rr = rec;
    void *args[] = {&pp, &rr};
    return hipLaunchKernel(em_record_kernel_ptr(precision, tab_mode(p.inst), p.inst.all_S_pos != 0, pairs > 0),
                           dim3(grid), dim3(block), args,
                           em_lds_bytes(p.inst.hist.n_bins, p.inst.n_tab, precision, grid_cells(p.inst)) +
                               pairs * kFeedBytes,
                           stream);
}

hipError_t tail_weigh(const double *d_N, const double *d_lnw, const uint32_t *d_steps, uint64_t n,
                      uint64_t traj_offset, double N_ref, double tail_lo, const RecordPool &rec, int precision, int n0,
                      int n1, double *d_G, TailEntry *tail, unsigned long long *n_tail,
                      unsigned long long *n_tail_total, double *J_sum, int cu_count, hipStream_t stream)
{
    const uint64_t most = (n + 15) / 16;
    const dim3 grid((unsigned)(most < (uint64_t)cu_count ? most : (uint64_t)cu_count)), block(1024);
    const size_t lds = (size_t)n0 * n1 * sizeof(double);
    if (precision == 0)
        hipLaunchKernelGGL(tail_weigh_kernel<double>, grid, block, lds, stream, d_N, d_lnw, d_steps, n, traj_offset,
                           N_ref, tail_lo, rec, n0, n1, d_G, tail, n_tail, n_tail_total, J_sum);
    else
        hipLaunchKernelGGL(tail_weigh_kernel<float>, grid, block, lds, stream, d_N, d_lnw, d_steps, n, traj_offset,
                           N_ref, tail_lo, rec, n0, n1, d_G, tail, n_tail, n_tail_total, J_sum);
    return hipGetLastError();
}

const void *batch_kernel_ptr(int precision, int bias_kind, bool all_pos)
{
    static const void *const t[2][2][2] = {
        {{bptr<0, kBiasNone, false>(), bptr<0, kBiasNone, true>()},
         {bptr<0, kBiasConst, false>(), bptr<0, kBiasConst, true>()}},
        {{bptr<1, kBiasNone, false>(), bptr<1, kBiasNone, true>()},
         {bptr<1, kBiasConst, false>(), bptr<1, kBiasConst, true>()}}};
    return t[precision ? 1 : 0][bias_kind == kBiasNone ? 0 : 1][all_pos ? 1 : 0];
}

template <int PREC, int BIAS, bool ALLPOS>
const void *bpptr() { return reinterpret_cast<const void *>(&batch_pair_kernel<PREC, BIAS, ALLPOS>); }

hipError_t batch_pair_launch(int precision, int bias_kind, bool all_pos, const Inst *insts, const WorkItem *items,
                             const RunArgs &run, int max_bins, int max_tab, int grid, int pairs, hipStream_t stream)
{
    static const void *const t[2][2][2] = {
        {{bpptr<0, kBiasNone, false>(), bpptr<0, kBiasNone, true>()},
         {bpptr<0, kBiasConst, false>(), bpptr<0, kBiasConst, true>()}},
        {{bpptr<1, kBiasNone, false>(), bpptr<1, kBiasNone, true>()},
         {bpptr<1, kBiasConst, false>(), bpptr<1, kBiasConst, true>()}}};
    const void *fn = t[precision ? 1 : 0][bias_kind == kBiasNone ? 0 : 1][all_pos ? 1 : 0];
    RunArgs r = run;
    void *args[] = {&insts, &items, &r};
    return hipLaunchKernel(fn, dim3(grid), dim3(128 * pairs), args,
                           em_lds_bytes(max_bins, max_tab, precision, 0) + pairs * kFeedBytes, stream);
}

hipError_t batch_launch(int precision, int bias_kind, bool all_pos, const Inst *insts, const WorkItem *items,
                        const BatchRun *run, unsigned long long *cursors, int max_bins, int max_tab, int grid,
                        int block, hipStream_t stream)
{
    const size_t lds = em_lds_bytes(max_bins, max_tab, precision, 0);
    const void *fn = batch_kernel_ptr(precision, bias_kind, all_pos);
    void *args[] = {&insts, &items, &run, &cursors, &max_bins};
    return hipLaunchKernel(fn, dim3(grid), dim3(block), args, lds, stream);
}

hipError_t zero_words(unsigned long long *ptr, size_t n, hipStream_t stream)
{
    const int block = 256;
    int grid = (int)((n + block - 1) / block);
    if (grid < 1) grid = 1;
    if (grid > 1024) grid = 1024;
    hipLaunchKernelGGL(zero_words_kernel, dim3(grid), dim3(block), 0, stream, ptr, n);
    return hipGetLastError();
}

}  // namespace fpt
