// rng.hpp -- device random numbers of the sampler.
//
// Philox4x32-10 (Salmon, Moraes, Dror & Shaw, "Parallel random numbers: as
// easy as 1, 2, 3", SC'11): a counter-based generator, so every draw is a pure
// function of (key, counter) and needs no state in memory.  Key = the chain's
// 64-bit seed; counter = (site or attempt, sweep, instance, tag).
//
// Normals: Box & Muller (1958), cosine branch.  Gamma: Marsaglia & Tsang
// (2000), "A simple method for generating gamma variables", without the
// squeeze test (the squeeze accepts a subset of the full test, so leaving it
// out changes no decision).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gmrf {

struct Words4 {
    uint32_t w0, w1, w2, w3;
};

// a ^ b ^ c in one instruction (truth table 0x96 of gfx950's three-input
// logic operation; the compiler emits two).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// Ten Philox rounds.  Each round multiplies two counter words by the Philox
// multipliers, mixes the high halves with the other two words and the key,
// and advances the key by the Weyl increments.
__device__ __forceinline__ Words4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2,
                                               uint32_t c3, uint32_t k0, uint32_t k1)
{
    constexpr uint32_t kMulA = 0xD2511F53u, kMulB = 0xCD9E8D57u;
    constexpr uint32_t kIncA = 0x9E3779B9u, kIncB = 0xBB67AE85u;
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t pa = (uint64_t)kMulA * c0;
        const uint64_t pb = (uint64_t)kMulB * c2;
        const uint32_t a_hi = (uint32_t)(pa >> 32), a_lo = (uint32_t)pa;
        const uint32_t b_hi = (uint32_t)(pb >> 32), b_lo = (uint32_t)pb;
        c0 = xor3(b_hi, c1, k0);
        c1 = b_lo;
        c2 = xor3(a_hi, c3, k1);
        c3 = a_lo;
        k0 += kIncA;
        k1 += kIncB;
    }
    return Words4{c0, c1, c2, c3};
}

__device__ __forceinline__ Words4 draw_words(uint64_t seed, uint32_t c0, uint32_t c1,
                                             uint32_t c2, uint32_t c3)
{
    return philox4x32_10(c0, c1, c2, c3, (uint32_t)seed, (uint32_t)(seed >> 32));
}

// (0,1) uniform from the top 52 bits of a word pair: (m + 1/2) 2^-52, never 0
// or 1.  The bits of m under the exponent of 1 are 1 + m 2^-52; subtracting
// 1 - 2^-53 leaves (2m + 1) 2^-53, which a double holds, so the subtraction
// is exact.  Three instructions against the conversion's ten.
__host__ __device__ __forceinline__ double open_uniform_f64(uint32_t hi, uint32_t lo)
{
    const uint64_t m = ((uint64_t)hi << 20) | (uint64_t)(lo >> 12);
    return __builtin_bit_cast(double, m | 0x3FF0000000000000ull) - 0x1.fffffffffffffp-1;
}

// f / d for d of order 1 (no scaling, no special values): the hardware
// reciprocal, one Newton step, and the quotient corrected by its exact
// remainder, which leaves it within a rounding of the divider's result.
// Measured on gfx950: 37 cycles per wavefront against 63 for the general
// divide.
__host__ __device__ __forceinline__ double quotient_f64(double f, double d)
{
#ifdef __HIP_DEVICE_COMPILE__
    double r = __builtin_amdgcn_rcp(d);
    r = fma(r, fma(-d, r, 1.0), r);
    const double s = f * r;
    return fma(fma(-d, s, f), r, s);
#else
    return f / d;
#endif
}

// sqrt(a) for a well inside the normal range (the Box-Muller radius: a in
// [2^-52, 80]): the hardware reciprocal square root, one coupled
// Newton (Goldschmidt) step for sqrt(a) and 1 / (2 sqrt(a)), and the exact
// residual a - g^2.  45 cycles per wavefront against 86 for the library's,
// which first scales its argument.
__host__ __device__ __forceinline__ double sqrt_f64(double a)
{
#ifdef __HIP_DEVICE_COMPILE__
    const double y = __builtin_amdgcn_rsq(a);
    double g = a * y, h = 0.5 * y;
    const double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    return fma(fma(-g, g, a), h, g);
#else
    return sqrt(a);
#endif
}

// Natural logarithm of an open uniform u in (0, 1) (u >= 2^-53), from the
// reduction u = m 2^k with m in [sqrt(1/2), sqrt(2)) and
//     log u = k log 2 + 2 atanh(s),   s = (m - 1) / (m + 1),   |s| < 0.1716.
// 2 atanh(s) = 2 s + 2 s s^2 p(s^2), p = 1/3 + s^2/5 + ...: its degree-6
// minimax polynomial on s^2 <= 0.02945 (Remez exchange, s^2 p within 1.9e-18
// with the coefficients rounded to doubles).  The reduction is done on the
// high word (the offset, mask and shift of musl's log1p), m - 1 is exact and
// log 2 is split into a head with trailing zero bits (k times it is exact)
// and a tail, so the result is within a few ulps of the correctly rounded
// logarithm.  About 30 instructions against ~100 for the general
// double-double library log, which dominates the Polya-Gamma sampler and the
// FP64 Box-Muller draw otherwise.
constexpr double kLn2Hi = 0x1.62e42fefa3800p-1;   // log 2 to 43 bits
constexpr double kLn2Lo = 0x1.ef35793c76730p-45;  // log 2 - kLn2Hi
__host__ __device__ inline double log_open_unit(double u)
{
    // exponent split at 0x3fe6a09e, the high word of sqrt(1/2)
    const uint64_t b = __builtin_bit_cast(uint64_t, u);
    const uint32_t e = (uint32_t)(b >> 32) + (0x3ff00000u - 0x3fe6a09eu);
    const int k = (int)(e >> 20) - 0x3ff;
    const uint32_t hi = (e & 0x000fffffu) + 0x3fe6a09eu;
    const double m = __builtin_bit_cast(double, ((uint64_t)hi << 32) | (uint32_t)b);
    const double f = m - 1.0;               // exact (m within a factor 2 of 1)
    const double s = quotient_f64(f, m + 1.0);
    const double s2 = s * s;
    double p = 0x1.2f0634870fe0ap-4;
    p = fma(p, s2, 0x1.39a1a6f733f8bp-4);
    p = fma(p, s2, 0x1.74663fa2250b8p-4);
    p = fma(p, s2, 0x1.c71c52060803ep-4);
    p = fma(p, s2, 0x1.24924941f4fb5p-3);
    p = fma(p, s2, 0x1.999999997fd77p-3);
    p = fma(p, s2, 0x1.5555555555592p-2);
    const double two_s = s + s;
    const double kd = (double)k;
    // k log2_hi + (2 s + (k log2_lo + 2 s s^2 p)), small terms first
    return fma(kd, kLn2Hi, two_s + fma(kd, kLn2Lo, two_s * s2 * p));
}

// cos(2 pi v) for v in [0, 1/4]: with w = 2 pi v <= pi/2,
//     cos w = 1 - w^2 (1/2 + w^2 q(w^2)),
// q the degree-6 minimax polynomial on w^2 <= pi^2/4 (Remez exchange, w^4 q
// within 1.4e-17 with the coefficients rounded to doubles).  Within a few 1e-16 of the exact value in absolute terms,
// which is what the Box-Muller product needs.
constexpr double kTwoPi = 6.283185307179586476925;
__host__ __device__ __forceinline__ double cos_2pi_quarter(double v)
{
    const double w = kTwoPi * v;
    const double w2 = w * w;
    double p = -0x1.9fc8d3aef65b1p-45;
    p = fma(p, w2, 0x1.93573fa111a71p-37);
    p = fma(p, w2, -0x1.1eecfaec8b6a0p-29);
    p = fma(p, w2, 0x1.27e4f9f33e23ep-22);
    p = fma(p, w2, -0x1.a01a019ba7401p-16);
    p = fma(p, w2, 0x1.6c16c16c10218p-10);
    p = fma(p, w2, -0x1.55555555554ddp-5);
    p = fma(p, w2, 0.5);
    return fma(-p, w2, 1.0);
}

// cos(2 pi u) for u in [0, 1], folded by the symmetries of the cosine:
// cos(2 pi u) = cos(2 pi (1 - u)) into v in [0, 1/2] and
// cos(2 pi v) = -cos(2 pi (1/2 - v)) into v in [0, 1/4] (both subtractions
// exact).
__host__ __device__ inline double cos_2pi_unit(double u)
{
    double v = u > 0.5 ? 1.0 - u : u;
    const bool neg = v > 0.25;
    if (neg)
        v = 0.5 - v;
    const double p = cos_2pi_quarter(v);
    return neg ? -p : p;
}

// sin(2 pi u) for u in [0, 1] as cos(2 pi (u - 1/4)), the argument moved
// back into [0, 1] by one period below u = 1/4.  For multiples of 2^-53 (the
// open uniforms) both shifts are exact: u - 1/4 lies in [0, 3/4] and u + 3/4
// in [3/4, 1), and every multiple of 2^-53 there is a double, so the error is
// cos_2pi_unit's.
__host__ __device__ inline double sin_2pi_unit(double u)
{
    return cos_2pi_unit(u < 0.25 ? u + 0.75 : u - 0.25);
}

// cos_2pi_unit(open_uniform_f64(hi, lo)), bit for bit, with both folds done on
// the words: 1 - (m + 1/2) 2^-52 = ((2^52 - 1 - m) + 1/2) 2^-52 is the
// complement of m, and 1/2 - v the complement of its low 51 bits, so each
// fold is an exclusive or with a sign mask (no FP64 compare or select).
__host__ __device__ __forceinline__ double cos_2pi_words(uint32_t hi, uint32_t lo)
{
    const uint32_t f1 = (uint32_t)((int32_t)hi >> 31);           // u > 1/2
    hi ^= f1;
    lo ^= f1;
    const uint32_t f2 = (uint32_t)((int32_t)(hi << 1) >> 31);    // v > 1/4
    hi ^= f2 >> 1;
    lo ^= f2;
    const double p = cos_2pi_quarter(open_uniform_f64(hi, lo));
    return __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, p) ^
                                          ((uint64_t)(f2 & 0x80000000u) << 32));
}

// sin_2pi_unit of the words' uniform: u - 1/4 modulo 1 is the high word less
// 2^30 modulo 2^32.
__host__ __device__ __forceinline__ double sin_2pi_words(uint32_t hi, uint32_t lo)
{
    return cos_2pi_words(hi - 0x40000000u, lo);
}

// FP64 standard normal of one Philox block.  log u1 and cos(2 pi u2) come
// from log_open_unit and cos_2pi_words: the library values up to a few ulps
// (no double-double logarithm, no general range reduction), with much
// lighter instruction sequences.  The FP64 sweeps are bound by the issue of
// this arithmetic: with the uniforms, folds, quotient, square root and
// polynomials above, against the library forms and Taylor series before
// them, a sweep takes 49.8 instead of 54.4 us (2048 x 2048, 8 neighbours),
// 8.0 instead of 10.1 us (64 x 64, 4 neighbours) and 8.1 instead of 9.6 us
// (50 x 50), a binomial iteration 169 instead of 183 us.
__device__ __forceinline__ double normal_f64(const Words4 &w)
{
    return sqrt_f64(-2.0 * log_open_unit(open_uniform_f64(w.w0, w.w1))) *
           cos_2pi_words(w.w2, w.w3);
}

// FP32 standard normal of the same block: the same two uniforms carried to
// FP32 precision (u1 keeps its relative precision down to 2^-56 so the tail
// tracks the FP64 draw), then Box-Muller on the hardware transcendental
// units: log2, square root, and the cosine whose argument is in revolutions,
// so cos(2 pi u2) is a single instruction.
__device__ __forceinline__ float normal_f32(const Words4 &w)
{
    const float u1 = fmaf((float)w.w0, 0x1p-32f, fmaf((float)(w.w1 >> 8), 0x1p-56f, 0x1p-57f));
    const float u2 = (float)w.w2 * 0x1p-32f;
    constexpr float kMinus2Ln2 = -1.38629436111989061883f;   // -2 ln 2
    return __builtin_amdgcn_sqrtf(kMinus2Ln2 * __builtin_amdgcn_logf(u1)) *
           __builtin_amdgcn_cosf(u2);
}

// One branch of a block's Box-Muller pair (the paired contract: the cosine
// branch for the lower-ranked site of a pair, the sine branch for its
// partner).
__device__ __forceinline__ double normal_branch_f64(const Words4 &w, bool sine)
{
    return sqrt_f64(-2.0 * log_open_unit(open_uniform_f64(w.w0, w.w1))) *
           cos_2pi_words(sine ? w.w2 - 0x40000000u : w.w2, w.w3);
}

__device__ __forceinline__ float normal_branch_f32(const Words4 &w, bool sine)
{
    const float u1 = fmaf((float)w.w0, 0x1p-32f, fmaf((float)(w.w1 >> 8), 0x1p-56f, 0x1p-57f));
    const float u2 = (float)w.w2 * 0x1p-32f;
    constexpr float kMinus2Ln2 = -1.38629436111989061883f;   // -2 ln 2
    const float r = __builtin_amdgcn_sqrtf(kMinus2Ln2 * __builtin_amdgcn_logf(u1));
    return r * (sine ? __builtin_amdgcn_sinf(u2) : __builtin_amdgcn_cosf(u2));
}

template <typename Real> __device__ __forceinline__ Real site_normal(const Words4 &w);
template <> __device__ __forceinline__ double site_normal<double>(const Words4 &w)
{
    return normal_f64(w);
}
template <> __device__ __forceinline__ float site_normal<float>(const Words4 &w)
{
    return normal_f32(w);
}

template <typename Real>
__device__ __forceinline__ Real site_normal_branch(const Words4 &w, bool sine)
{
    if constexpr (sizeof(Real) == 8)
        return normal_branch_f64(w, sine);
    else
        return normal_branch_f32(w, sine);
}

constexpr int kGammaMaxAttempts = 64;

// Marsaglia-Tsang constants of a shape >= 1: d = shape - 1/3, c = 1/sqrt(9 d)
// (the shapes depend only on n and the priors, so they are computed once per
// chain on the host, with the same operations).
struct GammaShape {
    double d, c;
};

// Gamma(shape, rate) for the hyperparameter draw after sweep `sweep`.
// Attempt k takes its normal from counter (2k, sweep, instance, tag) and its
// uniform from counter (2k + 1, ...).  Returns false when every attempt was
// rejected (the caller flags a numeric error).
__device__ inline bool gamma_draw(GammaShape g, double rate, uint64_t seed, uint32_t sweep,
                                  uint32_t instance, uint32_t tag, double *out)
{
    const double d = g.d, c = g.c;
    for (int k = 0; k < kGammaMaxAttempts; ++k) {
        const double z = normal_f64(draw_words(seed, (uint32_t)(2 * k), sweep, instance, tag));
        const double cz = c * z;
        if (cz <= -1.0)
            continue;
        const double L = 3.0 * log1p(cz);        // log of v = (1 + c z)^3
        const double v = exp(L);
        const Words4 wu = draw_words(seed, (uint32_t)(2 * k + 1), sweep, instance, tag);
        const double u = open_uniform_f64(wu.w0, wu.w1);
        // accept iff log u < z^2/2 + d - d v + d log v, with 1 - v + log v
        // evaluated as L - expm1(L) to avoid cancellation at large d
        if (log(u) < 0.5 * z * z + d * (L - expm1(L))) {
            *out = d * v / rate;
            return true;
        }
    }
    return false;
}

// ---------------------------------------------------------------------------
// Polya-Gamma variates (Polson, Scott & Windle 2013, Sec. 4, after Devroye
// 2009).  PG(1, c) = J*(1, |c|/2) / 4; J*(1, z) is drawn by rejection from
// an envelope of two pieces split at t = 0.64 -- a truncated exponential on
// (t, inf) and a truncated inverse Gaussian on (0, t) -- with the
// alternating-series test of the J*(1) density.  PG(m, c) for an integer m is
// the sum of m independent PG(1, c) terms.
// ---------------------------------------------------------------------------
constexpr double kPi = 3.141592653589793;
constexpr double kPgT = 0.64;
constexpr float kLn2f = 0.693147180559945309f;
constexpr float kLog2ef = 1.442695040888963407f;
constexpr float kPi2f = 9.869604401089358619f;      // pi^2
constexpr unsigned kPgMaxUniforms = 2048;   // uniforms available to one PG(1, c) draw
constexpr int kPgMaxTerms = 200;            // series terms per acceptance test

// Uniform stream of term j of one site's PG draw: uniform u is half (u & 1) of
// the Philox block at counter (site, sweep, instance, 2^31 | j << 10 | u >> 1).
struct PgStream {
    uint64_t seed;
    uint32_t site, sweep, instance, j;
    uint32_t used;
    bool exhausted;
    Words4 blk{};               // the block of the last even-numbered uniform

    // Uniform `used`: an even one computes its block and keeps it for the
    // odd one that follows (one Philox evaluation per two uniforms).
    __device__ double next()
    {
        const uint32_t u = used;
        if (u >= kPgMaxUniforms) {
            exhausted = true;
            return 0.5;
        }
        used = u + 1;
        if (u & 1u)
            return open_uniform_f64(blk.w2, blk.w3);
        blk = draw_words(seed, site, sweep, instance, 0x80000000u | (j << 10) | (u >> 1));
        return open_uniform_f64(blk.w0, blk.w1);
    }
};

__device__ inline double std_normal_cdf(double x) { return 0.5 * erfc(-x / sqrt(2.0)); }

// Terms of the alternating series of the J*(1) density at x, in order.
// Term n is pi (n + 1/2) c E^((2n+1)^2) with, right of t (x > t), c = 1 and
// E = exp(-pi^2 x / 8), and left of t, c = (2 / (pi x))^(3/2) and
// E = exp(-1 / (2 x)).  The powers come from one exp by the recurrence
// E^((2n+1)^2) = E^((2n-1)^2) * E^(8n), so each term after the first costs
// two multiplications; the values equal the per-term exponentials up to a
// few ulps.
struct PgSeries {
    double c, e, e8, ratio, power;
    int n;

    __device__ explicit PgSeries(double x)
    {
        if (x > kPgT) {
            c = 1.0;
            e = exp(-0.125 * kPi * kPi * x);
        } else {
            const double r = 2.0 / (kPi * x);
            c = r * sqrt(r);
            e = exp(-0.5 / x);
        }
        const double e2 = e * e, e4 = e2 * e2;
        e8 = e4 * e4;
        ratio = 1.0;
        power = e;
        n = 0;
    }
    // the current term, then advance to the next one
    __device__ double next()
    {
        const double v = kPi * ((double)n + 0.5) * c * power;
        ratio *= e8;                 // E^(8 (n + 1))
        power *= ratio;              // E^((2n + 3)^2)
        ++n;
        return v;
    }
};

// The acceptance of a pair of exponentials in the search of pg_left: E1^2 <=
// 2 E2 / t for E1 = -log u1, E2 = -log u2.  First from single-precision
// logarithms (hardware log2): their error is below 1e-6 (1 + e) for every e,
// so a difference beyond 1e-3 (1 + both sides) decides it as the
// double-precision test would; only closer calls take the double logarithms.
// The same decisions, so the same draws, with far fewer double logarithms.
__device__ __forceinline__ bool pg_pair_ok(double u1, double u2)
{
    const float a1 = -kLn2f * __builtin_amdgcn_logf((float)u1);
    const float a2 = -kLn2f * __builtin_amdgcn_logf((float)u2);
    const float lhs = a1 * a1, rhs = 2.0f * a2 / (float)kPgT;
    const float guard = 1e-3f * (1.0f + lhs + rhs);
    if (lhs - rhs > guard)
        return false;
    if (rhs - lhs > guard)
        return true;
    const double e1 = -log_open_unit(u1);
    return !(e1 * e1 > 2.0 * -log_open_unit(u2) / kPgT);
}

// The left piece's value for an accepted E1 = -log u1.
__device__ __forceinline__ double pg_left_value(double u1)
{
    const double d = 1.0 - kPgT * log_open_unit(u1);
    return quotient_f64(kPgT, d * d);
}

// u <= exp(w), w = -z^2 x / 2 in (-0.79, 0]: first against the
// single-precision exponential (relative error below 1e-6), the double one
// only within 1e-4 of it.
__device__ __forceinline__ bool pg_left_keep(double z, double x, double u)
{
    const double w = -0.5 * z * z * x;
    const double ef = (double)__builtin_amdgcn_exp2f((float)w * kLog2ef);
    if (u < ef * (1.0 - 1e-4))
        return true;
    if (u > ef * (1.0 + 1e-4))
        return false;
    return u <= exp(w);
}

// pg_left_keep where only u in (lo, hi) is known: 1 kept, 0 not, -1 undecided.
__device__ __forceinline__ int pg_left_keep_between(double z, double x, double lo, double hi)
{
    const double w = -0.5 * z * z * x;
    const double ef = (double)__builtin_amdgcn_exp2f((float)w * kLog2ef);
    return hi <= ef * (1.0 - 1e-4) ? 1 : lo >= ef * (1.0 + 1e-4) ? 0 : -1;
}

// The first test of the series, Y = u a0 <= a0 - a1, is u <= 1 - 3 E^8 (a1 /
// a0 = 3 E^8 for both forms of the terms), with 3 E^8 below 0.006 here.  From
// the single-precision exponential (error below 1e-8 absolute at these
// values) a u more than 1e-5 below it is accepted as the double-precision
// series would; other u need the series.
__device__ __forceinline__ bool pg_series_clear(double x, double u)
{
    const float xf = (float)x;
    const float w = x > kPgT ? -kPi2f * xf : -4.0f * __builtin_amdgcn_rcpf(xf);
    const float q = 3.0f * __builtin_amdgcn_exp2f(w * kLog2ef);
    return u < 1.0 - (double)q - 1e-5;
}

// One draw of IG(mu, 1) from its three uniforms (Michael, Schucany & Haas).
__device__ __forceinline__ double pg_steep_value(double mu, double u1, double u2, double u3)
{
    const double nrm = sqrt_f64(-2.0 * log_open_unit(u1)) * cos_2pi_unit(u2);
    const double y = nrm * nrm;
    const double my = mu * y;
    const double x = mu + 0.5 * mu * my - 0.5 * mu * sqrt(4.0 * my + my * my);
    return u3 > mu / (mu + x) ? mu * mu / x : x;
}

// IG(1/z, 1) restricted to (0, t).  z < 1/t: the z = 0 law on (0, t) from a
// normal tail beyond 1/sqrt(t) (1/X = (1 + t E1)^2 / t, E1^2 <= 2 E2 / t),
// kept with probability exp(-z^2 X / 2).  Otherwise: Michael, Schucany &
// Haas's transformation, repeated until X < t.
__device__ inline double pg_left(double z, PgStream &s)
{
    const double t = kPgT;
    if (z < 1.0 / t) {
        for (;;) {
            double u1;
            for (;;) {
                u1 = s.next();
                const double u2 = s.next();
                if (pg_pair_ok(u1, u2) || s.exhausted)
                    break;
            }
            const double x = pg_left_value(u1);
            if (pg_left_keep(z, x, s.next()) || s.exhausted)
                return x;
        }
    }
    const double mu = 1.0 / z;
    for (;;) {
        const double u1 = s.next();
        const double u2 = s.next();
        const double x = pg_steep_value(mu, u1, u2, s.next());
        if (x < t || s.exhausted)
            return x;
    }
}

// Envelope of PG(1, c) for one tilt: z = |c| / 2, rate K of the right piece
// and the probability p / (p + q) of drawing from it.
struct PgEnvelope {
    double z, K, right;
};

__device__ inline PgEnvelope pg_envelope(double c)
{
    const double t = kPgT;
    PgEnvelope e;
    e.z = 0.5 * fabs(c);
    e.K = kPi * kPi / 8.0 + 0.5 * e.z * e.z;
    const double p = kPi / (2.0 * e.K) * exp(-e.K * t);
    double q;
    if (e.z == 0.0) {
        q = 2.0 * erfc(1.0 / sqrt(2.0 * t));
    } else {
        const double a = std_normal_cdf((t * e.z - 1.0) / sqrt(t));
        const double b = e.z < 700.0 ? exp(e.z) * std_normal_cdf(-(t * e.z + 1.0) / sqrt(t)) : 0.0;
        q = 2.0 * (exp(-e.z) * a + b);
    }
    e.right = p / (p + q);
    return e;
}

// The right piece's value from its uniform.
__device__ __forceinline__ double pg_right_value(double K, double u)
{
    return kPgT - quotient_f64(log_open_unit(u), K);
}

// PG(1, c) from the stream of term j; false when the stream ran out.  used:
// 0, or the uniforms that a draw of the left piece has taken when it is to go
// on with its search from the next one.
__device__ inline bool pg1_draw(const PgEnvelope &e, uint64_t seed, uint32_t site, uint32_t sweep,
                                uint32_t instance, uint32_t j, uint32_t used, double *out)
{
    PgStream s{seed, site, sweep, instance, j, used, false, Words4{}};
    if (used & 1u)
        s.blk = draw_words(seed, site, sweep, instance, 0x80000000u | (j << 10) | (used >> 1));
    for (bool resume = used > 0;; resume = false) {
        double x;
        if (!resume && s.next() < e.right)
            x = pg_right_value(e.K, s.next());
        else
            x = pg_left(e.z, s);
        const double u = s.next();
        if (s.exhausted)
            return false;
        if (pg_series_clear(x, u)) {
            *out = 0.25 * x;
            return true;
        }
        PgSeries terms(x);
        double S = terms.next();
        const double Y = u * S;
        for (int n = 1; n <= kPgMaxTerms; ++n) {
            if (n & 1) {
                S -= terms.next();
                if (Y <= S) {
                    *out = 0.25 * x;
                    return true;
                }
            } else {
                S += terms.next();
                if (Y > S)
                    break;
            }
        }
    }
}

} // namespace gmrf
