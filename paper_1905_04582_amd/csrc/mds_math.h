// mds_math.h -- device special functions of the truncated-normal MDS model.
//
// For t = delta/sigma >= 0 every pair needs ln Phi(t) (Eq. 2) and the ratio
// phi(t)/Phi(t) (Eq. 9).  Both are built branch-free from one exponential:
//     e = exp(-t^2/2),  z = t/sqrt 2,  erfcx(z) ~ P(z)/Q(z),
//     q = Phi(-t) = e erfcx(z) / 2 = a / (2Q)   with a = e P,
//     ln Phi(t) = log1p(-q) = -2 s A(s^2),  s = q/(2-q) = a / (4Q - a),
//     phi(t)/Phi(t) = e / (sqrt(2 pi) (1-q)) = 4 e Q / (sqrt(2 pi) (4Q - 2a)),
// where A(v) = atanh(sqrt v)/sqrt v.  s <= 1/3 because q <= 1/2, so A is a
// short polynomial on [0, 1/9], and log1p keeps full relative accuracy as
// q -> 0.  The two divisions share one reciprocal of (4Q - a)(4Q - 2a).
// Coefficients come from gen_coeffs.py (mds_coeffs.h).  Every lane runs the
// same instructions whatever t is: no branches, no lane divergence.  The FP64
// sweep and the held-out density use shorter forms of the same precision on
// their range of t (further down).
//
// The general helpers at the end also cover t < 0 (never reached by the
// sweeps, where delta >= 0 and sigma > 0) through the log-erfc form
//     ln Phi(t) = -t^2/2 + ln(erfcx(-t/sqrt 2)/2),
//     phi(t)/Phi(t) = sqrt(2/pi) / erfcx(-t/sqrt 2),
// which neither underflows nor cancels however far t goes below 0.
#pragma once

#include <hip/hip_runtime.h>

#include "mds_coeffs.h"

namespace mds {

constexpr double kInvSqrt2 = 0.70710678118654752440;
constexpr double kInvSqrt2Pi = 0.39894228040143267794;  // 1/sqrt(2 pi)
constexpr double kSqrt2OverPi = 0.79788456080286535588;  // sqrt(2/pi)

template <typename T, int N>
__device__ __forceinline__ T horner(const T (&c)[N], T x)
{
    T acc = c[N - 1];
#pragma unroll
    for (int k = N - 2; k >= 0; --k) acc = fma(acc, x, c[k]);
    return acc;
}

// acc * x + c with c in a scalar register: one VOP3 v_fma_f64.  (The
// compiler otherwise prefers the two-operand v_fmac_f64, whose addend must be
// a vector register, and copies every coefficient into one first.)
__device__ __forceinline__ double fma_sc(double acc, double x, double c)
{
    double r;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(acc), "v"(x), "s"(c));
    return r;
}

// The FP64 coefficient tables in one constant-memory object, so that one
// scalar base address reaches every coefficient by an immediate offset.
struct CoefTables64 {
    double exp[sizeof(kExpC64) / sizeof(double)];
    double erfcx_p[sizeof(kErfcxP64) / sizeof(double)];
    double erfcx_q[sizeof(kErfcxQ64) / sizeof(double)];
    double atanh[sizeof(kAtanhA64) / sizeof(double)];
    double near_p[sizeof(kNearP64) / sizeof(double)];
    double near_q[sizeof(kNearQ64) / sizeof(double)];
    double exp2[sizeof(kExp2C64) / sizeof(double)];
};

constexpr CoefTables64 make_tables64()
{
    CoefTables64 t{};
    for (size_t k = 0; k < sizeof(kExpC64) / sizeof(double); ++k) t.exp[k] = kExpC64[k];
    for (size_t k = 0; k < sizeof(kErfcxP64) / sizeof(double); ++k) t.erfcx_p[k] = kErfcxP64[k];
    for (size_t k = 0; k < sizeof(kErfcxQ64) / sizeof(double); ++k) t.erfcx_q[k] = kErfcxQ64[k];
    for (size_t k = 0; k < sizeof(kAtanhA64) / sizeof(double); ++k) t.atanh[k] = kAtanhA64[k];
    for (size_t k = 0; k < sizeof(kNearP64) / sizeof(double); ++k) t.near_p[k] = kNearP64[k];
    for (size_t k = 0; k < sizeof(kNearQ64) / sizeof(double); ++k) t.near_q[k] = kNearQ64[k];
    for (size_t k = 0; k < sizeof(kExp2C64) / sizeof(double); ++k) t.exp2[k] = kExp2C64[k];
    return t;
}

static __constant__ CoefTables64 kTab64 = make_tables64();

typedef const __attribute__((address_space(4))) double* const_f64_ptr;
typedef const __attribute__((address_space(4))) CoefTables64* tab64_ptr;

// The tables' address, hidden from the optimiser by an empty asm: the
// coefficients are then fetched by uniform scalar loads (s_load) instead of
// being folded into immediates, which a 64-bit VALU operand cannot encode.
// A caller that evaluates the special functions in a loop takes the address
// once and passes it in.
__device__ __forceinline__ tab64_ptr tab64()
{
    tab64_ptr p = (tab64_ptr)&kTab64;
    asm volatile("" : "+s"(p));
    return p;
}

// Horner's rule over a table of N coefficients in constant memory.
template <int N>
__device__ __forceinline__ double horner_tab(const_f64_ptr c, double x)
{
    double acc = fma_sc(c[N - 1], x, c[N - 2]);
#pragma unroll
    for (int k = N - 3; k >= 0; --k) acc = fma_sc(acc, x, c[k]);
    return acc;
}

// Horner's rule for two arguments at once: each coefficient is loaded once
// and feeds both chains (two independent dependency chains interleave).
template <int N>
__device__ __forceinline__ void horner2_tab(const_f64_ptr c, double x1, double x2, double& r1,
                                            double& r2)
{
    double a1 = fma_sc(c[N - 1], x1, c[N - 2]);
    double a2 = fma_sc(c[N - 1], x2, c[N - 2]);
#pragma unroll
    for (int k = N - 3; k >= 0; --k) {
        a1 = fma_sc(a1, x1, c[k]);
        a2 = fma_sc(a2, x2, c[k]);
    }
    r1 = a1;
    r2 = a2;
}

// ---------------------------------------------------------------- FP64 --

// 1/d for finite d > 0 (not subnormal): hardware estimate + 2 Newton steps
__device__ __forceinline__ double rcp_f64(double d)
{
    double r = __builtin_amdgcn_rcp(d);
    double e = fma(-d, r, 1.0);
    r = fma(r, e, r);
    e = fma(-d, r, 1.0);
    return fma(r, e, r);
}

// 1/sqrt(x) for finite x >= DBL_MIN: hardware estimate r (relative error
// below 2^-24 on gfx950), then one correction of third order: with
// e = 1 - x r^2, 1/sqrt(x) = r (1 + e/2 + 3/8 e^2 + 5/16 e^3 + ...), and
// the first omitted term is below 2^-70 of the result, so the final fma's
// rounding sets the error (a Newton step only squares it: two would be
// needed).  Five operations after the estimate.
__device__ __forceinline__ double rsqrt_f64(double x)
{
    const double r = __builtin_amdgcn_rsq(x);
    const double e = fma(-(x * r), r, 1.0);
    return fma(r, e * fma(0.375, e, 0.5), r);
}

constexpr int kExpN = sizeof(kExpC64) / sizeof(double);
constexpr int kErfcxPN = sizeof(kErfcxP64) / sizeof(double);
constexpr int kErfcxQN = sizeof(kErfcxQ64) / sizeof(double);
constexpr int kAtanhN = sizeof(kAtanhA64) / sizeof(double);

// exp(-t^2/2) for t >= 0; 0 once the value leaves the FP64 range
__device__ __forceinline__ double exp_neg_half_sq(double t, tab64_ptr tb)
{
    const double x = fmax(-0.5 * (t * t), -760.0);
    const double k = rint(x * kLog2e);
    double r = fma(k, -kLn2Head, x);
    r = fma(k, -kLn2Tail, r);
    return ldexp(horner_tab<kExpN>(tb->exp, r), (int)k);
}

// ln Phi(t) and phi(t)/Phi(t) for t >= 0 (the sweep's domain)
__device__ __forceinline__ void trunc_terms_f64(double t, double& lnphi, double& mills)
{
    const tab64_ptr tb = tab64();
    const double e = exp_neg_half_sq(t, tb);
    // beyond the fitted range e == 0, so any finite positive erfcx will do
    const double z = fmin(t * kInvSqrt2, kErfcxZmax64 + 1.0);
    const double P = horner_tab<kErfcxPN>(tb->erfcx_p, z);
    const double Q = horner_tab<kErfcxQN>(tb->erfcx_q, z);
    const double a = e * P;               // 2 q Q
    const double d1 = fma(4.0, Q, -a);    // 4Q - a   = 2Q (2 - q)
    const double d2 = d1 - a;             // 4Q - 2a  = 4Q (1 - q)
    const double rr = rcp_f64(d1 * d2);
    const double s = a * d2 * rr;         // q / (2 - q)
    lnphi = -2.0 * s * horner_tab<kAtanhN>(tb->atanh, s * s);
    mills = (4.0 * kInvSqrt2Pi) * (e * Q) * (d1 * rr);
}

// The sweep's truncation terms.  Its sums need sum ln Phi(t) and m =
// phi(t)/Phi(t) of each near pair (t below the sweep's skip point), and the
// first only as a sum: it is -ln of the product G of the pairs' 1/Phi, so a
// pair costs a multiplication instead of a logarithm.  With e = exp(-t^2/2),
// 1 - Phi = e P/Q (fitted in relative error, as the form above) and x = e P,
//     u = 1/Phi - 1 = x / (Q - x),   sigma m = (sigma/sqrt(2 pi)) e (1 + u),
// from one reciprocal.  The product is carried as E = G - 1, E' = E + u + E u,
// and closed by ln(1 + E), so that a sum of small terms keeps its relative
// precision (at t = 8 a term is 6e-16, which a factor 1/Phi would round away).
// Against the form above (84 instructions a pair) this is 52, in one form for
// every near t, with 32 coefficients instead of 44.

// what the near terms take from sigma, formed once per wave
struct NearConst64 {
    double inv_s;  // 1/sigma
    double c2;     // -log2(e) / (2 sigma^2): log2 of exp(-t^2/2) over delta^2
    double kappa;  // sigma / sqrt(2 pi)
};
__device__ __forceinline__ NearConst64 near_const(double sigma, double inv_s)
{
    return {inv_s, -0.5 * kLog2e * inv_s * inv_s, sigma * kInvSqrt2Pi};
}

constexpr int kNearPN = sizeof(kNearP64) / sizeof(double);
constexpr int kNearQN = sizeof(kNearQ64) / sizeof(double);
constexpr int kExp2N = sizeof(kExp2C64) / sizeof(double);

// exp(-t^2/2) of a near pair from s2 = delta^2: 2^y, y = c2 s2 = k + f, with k
// read from the low word of y + 1.5 2^52 and added to the exponent field.  For
// a pair that is not near the result is meaningless (the caller drops it).
__device__ __forceinline__ double near_scale(double p, double shifted)
{
    const int k = __double2loint(shifted);
    return __hiloint2double(__double2hiint(p) + (int)((unsigned)k << 20), __double2loint(p));
}

// Two pairs, sharing every coefficient load: s2 = delta^2, dl = delta; `na`,
// `nb`: whether the pair is near (one that is not gets u = m = 0).
// u = 1/Phi(t) - 1, m = sigma phi(t)/Phi(t).
__device__ __forceinline__ void near_terms2_f64(double s2a, double s2b, double dla, double dlb,
                                                bool na, bool nb, const NearConst64& k,
                                                tab64_ptr tb, double& ua, double& ub, double& ma,
                                                double& mb)
{
    constexpr double kMagic = 6755399441055744.0;  // 1.5 * 2^52
    const double ha = fma(s2a, k.c2, kMagic), hb = fma(s2b, k.c2, kMagic);
    const double fa = fma(s2a, k.c2, -(ha - kMagic)), fb = fma(s2b, k.c2, -(hb - kMagic));
    double pa, pb;
    horner2_tab<kExp2N - 1>(tb->exp2 + 1, fa, fb, pa, pb);
    pa = fma(pa, fa, 1.0);
    pb = fma(pb, fb, 1.0);
    const double ea = na ? near_scale(pa, ha) : 0.0;
    const double eb = nb ? near_scale(pb, hb) : 0.0;
    // (the bound keeps P and Q finite for pairs that are not near)
    const double ta = fmin(dla * k.inv_s, 10.0), tb2 = fmin(dlb * k.inv_s, 10.0);
    double Pa, Pb, Qa, Qb;
    horner2_tab<kNearPN>(tb->near_p, ta, tb2, Pa, Pb);
    horner2_tab<kNearQN - 1>(tb->near_q + 1, ta, tb2, Qa, Qb);
    Qa = fma(Qa, ta, 1.0);
    Qb = fma(Qb, tb2, 1.0);
    const double xa = ea * Pa, xb = eb * Pb;
    const double da = Qa - xa, db = Qb - xb;
    // x/d: the hardware reciprocal r (relative error v below 2^-22), then the
    // quotient by 1 + v + v^2
    const double ra = __builtin_amdgcn_rcp(da), rb = __builtin_amdgcn_rcp(db);
    const double va = fma(-da, ra, 1.0), vb = fma(-db, rb, 1.0);
    const double qa = xa * ra, qb = xb * rb;
    ua = fma(qa, fma(va, va, va), qa);
    ub = fma(qb, fma(vb, vb, vb), qb);
    const double ka = ea * k.kappa, kb = eb * k.kappa;
    ma = fma(ka, ua, ka);
    mb = fma(kb, ub, kb);
}

// E = G - 1 of a product G = (1 + E) with two more factors 1 + u
__device__ __forceinline__ double extend_product(double E, double ua, double ub)
{
    const double u = fma(ua, ub, ua + ub);
    return fma(E, u, E + u);
}

// -ln Phi(t) of two pairs in the same terms, 0 for a pair with near = false:
// q = e P/Q, -ln Phi = 2 atanh(s) with s = q/(2 - q) = e P/(2Q - e P).  The
// exponent is taken from t itself: sigma may be as small as a double holds.
__device__ __forceinline__ void neg_ln_phi2_f64(double ta, double tb2, bool na, bool nb,
                                                tab64_ptr tb, double& la, double& lb)
{
    constexpr double kMagic = 6755399441055744.0;  // 1.5 * 2^52
    constexpr double kC2 = -0.5 * kLog2e;
    const double t2a = ta * ta, t2b = tb2 * tb2;
    const double ha = fma(t2a, kC2, kMagic), hb = fma(t2b, kC2, kMagic);
    const double fa = fma(t2a, kC2, -(ha - kMagic)), fb = fma(t2b, kC2, -(hb - kMagic));
    double pa, pb;
    horner2_tab<kExp2N - 1>(tb->exp2 + 1, fa, fb, pa, pb);
    pa = fma(pa, fa, 1.0);
    pb = fma(pb, fb, 1.0);
    const double ea = na ? near_scale(pa, ha) : 0.0;
    const double eb = nb ? near_scale(pb, hb) : 0.0;
    const double za = fmin(ta, 10.0), zb = fmin(tb2, 10.0);
    double Pa, Pb, Qa, Qb;
    horner2_tab<kNearPN>(tb->near_p, za, zb, Pa, Pb);
    horner2_tab<kNearQN - 1>(tb->near_q + 1, za, zb, Qa, Qb);
    Qa = fma(Qa, za, 1.0);
    Qb = fma(Qb, zb, 1.0);
    const double xa = ea * Pa, xb = eb * Pb;
    const double da = fma(2.0, Qa, -xa), db = fma(2.0, Qb, -xb);
    const double ra = __builtin_amdgcn_rcp(da), rb = __builtin_amdgcn_rcp(db);
    const double va = fma(-da, ra, 1.0), vb = fma(-db, rb, 1.0);
    const double ua = xa * ra, ub = xb * rb;
    const double sa = fma(ua, fma(va, va, va), ua), sb = fma(ub, fma(vb, vb, vb), ub);
    double Aa, Ab;
    horner2_tab<kAtanhN>(tb->atanh, sa * sa, sb * sb, Aa, Ab);
    la = 2.0 * sa * Aa;
    lb = 2.0 * sb * Ab;
}

// exp(x) for -700 <= x <= 0 (2^f and an exponent, as above; f takes the tail of
// log2(e) too, whose product with x grows to 9 units of the result), two at a time
__device__ __forceinline__ void exp2_neg_f64(double x1, double x2, tab64_ptr tb, double& e1,
                                             double& e2)
{
    constexpr double kMagic = 6755399441055744.0;
    const double h1 = fma(x1, kLog2e, kMagic), h2 = fma(x2, kLog2e, kMagic);
    const double f1 = fma(x1, kLog2eTail, fma(x1, kLog2e, -(h1 - kMagic)));
    const double f2 = fma(x2, kLog2eTail, fma(x2, kLog2e, -(h2 - kMagic)));
    double p1, p2;
    horner2_tab<kExp2N - 1>(tb->exp2 + 1, f1, f2, p1, p2);
    e1 = near_scale(fma(p1, f1, 1.0), h1);
    e2 = near_scale(fma(p2, f2, 1.0), h2);
}

// ln(1 + E), E >= 0, for the product 1 + E of up to 256 factors 1/Phi in
// [1, 2]: 1 + E = 2^n f, f in [sqrt(1/2), sqrt 2), ln f = 2 atanh((f - 1)/(f + 1)),
// the quotient below 0.172; where n = 0, f - 1 is E itself
__device__ __forceinline__ double log1p_product(double E, tab64_ptr tb)
{
    constexpr double kLn2 = 0.693147180559945309417;
    const double g = 1.0 + E;
    const double h = __builtin_amdgcn_frexp_mant(g);
    const bool low = h < kInvSqrt2;
    const int n = __builtin_amdgcn_frexp_exp(g) - (low ? 1 : 0);
    const double f = low ? 2.0 * h : h;
    const double d = f + 1.0;
    const double r = __builtin_amdgcn_rcp(d);
    const double v = fma(-d, r, 1.0);
    const double q = (n == 0 ? E : f - 1.0) * r;
    const double s = fma(q, fma(v, v, v), q);
    const double a = horner_tab<kAtanhN>(tb->atanh, s * s);
    return fma(2.0 * s, a, (double)n * kLn2);
}

// ---------------------------------------------------------------- FP32 --

// ln Phi(t) and phi(t)/Phi(t) for t >= 0 in FP32 arithmetic
__device__ __forceinline__ void trunc_terms_f32(float t, float& lnphi, float& mills)
{
    const float e = __builtin_amdgcn_exp2f(-0.5f * (t * t) * (float)kLog2e);
    const float z = fminf(t * (float)kInvSqrt2, kErfcxZmax32 + 1.0f);
    const float P = horner(kErfcxP32, z);
    const float Q = horner(kErfcxQ32, z);
    const float a = e * P;
    const float d1 = fmaf(4.0f, Q, -a);
    const float d2 = d1 - a;
    const float rr = __builtin_amdgcn_rcpf(d1 * d2);
    const float s = a * d2 * rr;
    lnphi = -2.0f * s * horner(kAtanhA32, s * s);
    mills = (float)(4.0 * kInvSqrt2Pi) * (e * Q) * (d1 * rr);
}

// The sweep's form of trunc_terms_f32, same roundings: h = -ln Phi(t)/2 (the
// factor -2 is exact and taken out of the sum), and a pair with ok = false
// gets h = m = 0 from e = 0 (z is bounded, so P and Q are finite).
__device__ __forceinline__ void near_terms_f32(float t, bool ok, float& h, float& mills)
{
    const float x = __builtin_amdgcn_exp2f((t * t) * (float)(-0.5 * kLog2e));
    const float e = ok ? x : 0.0f;
    const float z = fminf(t * (float)kInvSqrt2, kErfcxZmax32 + 1.0f);
    const float P = horner(kErfcxP32, z);
    const float Q = horner(kErfcxQ32, z);
    const float a = e * P;
    const float d1 = fmaf(4.0f, Q, -a);
    const float d2 = d1 - a;
    const float rr = __builtin_amdgcn_rcpf(d1 * d2);
    const float s = a * d2 * rr;
    h = s * horner(kAtanhA32, s * s);
    mills = (float)(4.0 * kInvSqrt2Pi) * (e * Q) * (d1 * rr);
}

// --------------------------------------------------- general helpers ----

// any real t
__device__ inline void log_phi_general_f64(double t, double& lnphi, double& mills)
{
    if (t >= 0.0) {
        trunc_terms_f64(t, lnphi, mills);
    } else {
        // log-erfc form of the lower tail
        const double z = -t * kInvSqrt2;
        const double ex = erfcx(z);
        lnphi = -0.5 * t * t + log(0.5 * ex);
        mills = kSqrt2OverPi / ex;
    }
}

// any real t: FP32 arithmetic, except the far lower tail t < -5, which is
// evaluated in FP64 by the log-erfc form and rounded once.
__device__ inline void log_phi_general_f32(float t, float& lnphi, float& mills)
{
    if (t >= 0.0f) {
        trunc_terms_f32(t, lnphi, mills);
    } else if (t >= -5.0f) {
        const float z = -t * (float)kInvSqrt2;
        const float ex = erfcxf(z);
        lnphi = -0.5f * t * t + logf(0.5f * ex);
        mills = (float)kSqrt2OverPi / ex;
    } else {
        double l, m;
        log_phi_general_f64((double)t, l, m);
        lnphi = (float)l;
        mills = (float)m;
    }
}

}  // namespace mds
