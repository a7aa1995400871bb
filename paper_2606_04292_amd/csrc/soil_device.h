// Device-side constitutive laws, sink and the pointwise Newton solve.
//
// theta(psi), theta'(psi), K(psi)/Ks follow Table tab:models (Haverkamp;
// van Genuchten - Mualem with m = 1 - 1/n and l = 1/2); psi >= 0 is saturated.
// The vGM forms are rearranged to avoid cancellation:
//   P = (alpha|psi|)^n = exp(n log(alpha|psi|)),  Se = exp(-m log1p(P)),
//   1 - Se^(1/m) = P / (1 + P), so the Mualem bracket is
//   1 - (P/(1+P))^m = -expm1(m (n log(alpha|psi|) - log1p(P))).
// Haverkamp uses Q = |u psi|^beta = exp(beta log|u psi|) and
//   theta' = u beta (theta - theta_r) (Q / (alpha + Q)) / |u psi|.
// The sweep and residual evaluate ln, ln(1+p) and exp with the short
// series below (a few ulp); the once-per-step K(psi) uses the library ones.
// Each law is a template specialisation so the sweep kernels carry no model
// switch; the generic entry points dispatch on Law::model.
#pragma once

#include "rs_internal.h"

namespace rs {

// 1/x from the hardware estimate refined by two Newton-Raphson steps
// (error of a few ulp; used where a correctly rounded quotient is not needed).
__device__ __forceinline__ double rcp_nr(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    double e = fma(-x, r, 1.0);
    r = fma(r, e, r);
    e = fma(-x, r, 1.0);
    return fma(r, e, r);
}

// 1/x from the hardware estimate (about 2^-24) refined by one Newton-Raphson
// step: within ~11 ulp, enough where the quotient only feeds a self-correcting
// iteration or a term already carrying that much rounding.
__device__ __forceinline__ double rcp_1nr(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    double e = fma(-x, r, 1.0);
    return fma(r, e, r);
}

// Natural logarithm of a positive normal double.  x = m 2^e with m in
// [sqrt(1/2), sqrt(2)), ln x = e ln2 + 2 atanh(s), s = (m-1)/(m+1), |s| <= 0.1716,
// and ln2 split Cody-Waite style so that e ln2_hi is exact.
constexpr double kLn2Hi = 6.93147180369123816490e-01;
constexpr double kLn2Lo = 1.90821492927058770002e-10;
constexpr double kInvLn2 = 1.44269504088896338700e+00;

// A value that every lane of the wave holds, in a scalar register pair (there is
// no scalar FP64 arithmetic: a product of kernel arguments lands in vector
// registers, two per value, for as long as it lives).
template <bool PER_LANE>
__device__ __forceinline__ double uniform_f64(double v)
{
    if (PER_LANE) return v;
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)b);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// p * r + c with the coefficient c in a scalar register pair (one VOP3 FMA;
// no vector moves to materialise the constant).
__device__ __forceinline__ double fma_sc(double p, double r, double c)
{
    double out;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(out) : "v"(p), "v"(r), "s"(c));
    return out;
}

// 2 atanh(s) = 2 s + 2 s^3 R(s^2), R the degree-7 polynomial of least relative
// error over |s| <= 0.1716 (Remez exchange: 8.2e-21).  Against 50-digit values at
// 40000 points 0.500 ulp at most and 0.183 on average, as the nine-term Taylor
// series it replaces (0.500, 0.184).
__device__ __forceinline__ double atanh2_series(double s)
{
    const double s2 = s * s;
    double p = 0.06625447453546243;
    p = fma_sc(p, s2, 0.0662508549448883);
    p = fma_sc(p, s2, 0.07693544063083087);
    p = fma_sc(p, s2, 0.0909088786714923);
    p = fma_sc(p, s2, 0.11111111322895023);
    p = fma_sc(p, s2, 0.1428571428454699);
    p = fma_sc(p, s2, 0.20000000000003107);
    p = fma_sc(p, s2, 0.3333333333333333);
    return fma(2.0 * s * s2, p, 2.0 * s);
}

__device__ __forceinline__ double rs_log(double x)
{
    int e = __builtin_amdgcn_frexp_exp(x);
    double m = __builtin_amdgcn_frexp_mant(x);      // [0.5, 1)
    if (m < 0.70710678118654752440) {
        m += m;
        e -= 1;
    }
    const double s = (m - 1.0) * rcp_1nr(m + 1.0);
    const double de = (double)e;
    return fma(de, kLn2Hi, fma(de, kLn2Lo, atanh2_series(s)));
}

// ln(1 + p) for p >= 0: the atanh series with s = p/(2+p) while p < sqrt(2)-1
// (no cancellation for small p), else ln of the rounded sum.
__device__ __forceinline__ double rs_log1p(double p)
{
    if (p < 0.41421356237309504880) return atanh2_series(p * rcp_1nr(2.0 + p));
    return rs_log(1.0 + p);
}

// e^y: y = n ln2 + r (Cody-Waite, |r| <= ln2/2), e^r = 1 + r + r^2/2 + r^3 q(r)
// with q the degree-9 polynomial of least error (Remez exchange: 5.4e-20 in e^r),
// scaled by 2^n (overflows to inf, underflows to 0 past the double range).
// Against 50-digit values at 40000 points 0.605 ulp at most and 0.186 on
// average, as the Taylor series to r^13/13! it replaces.
__device__ __forceinline__ double rs_exp(double y)
{
    const double n = rint(y * kInvLn2);
    double r = fma(-n, kLn2Hi, y);
    r = fma(-n, kLn2Lo, r);
    double p = 2.0925702139195154e-09;
    p = fma_sc(p, r, 2.5112179532238123e-08);
    p = fma_sc(p, r, 2.755723860719594e-07);
    p = fma_sc(p, r, 2.755723443702197e-06);
    p = fma_sc(p, r, 2.48015873651743e-05);
    p = fma_sc(p, r, 0.00019841269896820335);
    p = fma_sc(p, r, 0.0013888888888865139);
    p = fma_sc(p, r, 0.008333333333316859);
    p = fma_sc(p, r, 0.0416666666666667);
    p = fma_sc(p, r, 0.16666666666666682);
    p = fma(p, r, 0.5);
    p = fma(p, r, 1.0);
    p = fma(p, r, 1.0);
    return __builtin_amdgcn_ldexp(p, (int)n);
}

// (1 + u)^e - 1 by the binomial series to u^7 (c[k - 1] = binom(e, k)), for
// |u| < 2^-8: for -1 <= e <= 7, |binom(e, k)| <= |e| for k >= 8, so the terms left
// out sum to at most |e| |u|^8 / (1 - |u|) < 2^-63 |e|.
__device__ __forceinline__ double pow1p_m1_series(double u, const double *c)
{
    double p = c[6];
    p = fma(p, u, c[5]);
    p = fma(p, u, c[4]);
    p = fma(p, u, c[3]);
    p = fma(p, u, c[2]);
    p = fma(p, u, c[1]);
    p = fma(p, u, c[0]);
    return p * u;
}

// Power terms of the last law evaluation at a node.
struct PowState {
    bool ok;       // the last iterate was unsaturated (Haverkamp, vGM)
    double h;      // its magnitude: unit |x| (Haverkamp), |x| (vGM)
    double ih;     // 1 / h
    double q;      // Haverkamp: Q = (unit |x|)^beta; vGM: P = (alpha |x|)^n
    double se;     // vGM: Se = (1 + P)^-m
    double ix1p;   // vGM: 1 / (1 + P)
};

// The state behind a magnitude and the vGM power terms that were kept (h = 0:
// none).
__device__ __forceinline__ PowState pow_kept(double h, double q, double se)
{
    const double X = 1.0 + q, w = rcp_1nr(X * h);
    return PowState{h > 0.0, h, X * w, q, se, h * w};
}

__device__ __forceinline__ PowState pow_none()
{
    return PowState{false, 0.0, 0.0, 0.0, 1.0, 0.0};
}

// The law at x < 0 within the visits of one node: theta - theta_r = L.c_th s and
// theta' = L.c_dth ds.  The power terms of the Haverkamp and vGM laws scale from
// the last iterate's: Q(x) = Q(x') (1 + u)^beta and P(x) = P(x') (1 + u)^n with
// u = x / x' - 1, then Se(x) = Se(x') (1 + v)^-m with v = (P(x) - P(x')) / (1 + P(x'));
// each factor is taken by the binomial series while its u or v is below
// L.series_u (2^-8; 0 for exponents outside [-1, 7]) in magnitude, else the
// powers are evaluated afresh.  A scaled power adds one rounding to the last
// one's error (the argument u carries |u| times its own), far below the few ulp
// times the exponent of a fresh evaluation.  NR2: two Newton-Raphson steps in
// the reciprocal that enters theta, for values that enter a defect.
template <int MODEL, bool NR2 = false>
__device__ __forceinline__ void law_unsat(const Law &L, double x, PowState &p, double &s,
                                          double &ds)
{
    if (MODEL == kLinear) {
        s = x;
        ds = 1.0;
    } else if (MODEL == kGardner) {
        s = rs_exp(L.gd_alpha * L.unit * x);
        ds = s;
    } else if (MODEL == kHaverkamp) {
        const double hu = -L.unit * x;
        const double u = (hu - p.h) * p.ih;
        double Q;
        if (p.ok && fabs(u) < L.series_u) Q = fma(p.q, pow1p_m1_series(u, L.bin1), p.q);
        else Q = rs_exp(L.hk_beta * rs_log(hu));
        // one reciprocal serves 1/(alpha + Q) = hu w and 1/hu = (alpha + Q) w
        const double den = L.hk_alpha + Q;
        const double w = NR2 ? rcp_nr(hu * den) : rcp_1nr(hu * den);
        s = hu * w;
        ds = Q * (s * w);
        p.q = Q;
        p.h = hu;
        p.ih = den * w;
        p.ok = true;
    } else {
        const double h = -x;
        const double u = (h - p.h) * p.ih;
        double P = 0.0;
        bool fresh = true;
        if (p.ok && fabs(u) < L.series_u) {
            const double dP = p.q * pow1p_m1_series(u, L.bin1);
            const double v = dP * p.ix1p;
            P = p.q + dP;
            if (fabs(v) < L.series_u) {
                s = fma(p.se, pow1p_m1_series(v, L.bin2), p.se);
                fresh = false;
            }
        }
        if (fresh) {
            P = rs_exp(L.vg_n * rs_log(L.vg_alpha * h));
            s = rs_exp(-L.vg_m * rs_log1p(P));
        }
        const double X = 1.0 + P;
        const double w = rcp_1nr(X * h);
        ds = P * (s * w);
        p.q = P;
        p.se = s;
        p.h = h;
        p.ih = X * w;
        p.ix1p = h * w;
        p.ok = true;
    }
}

template <int MODEL>
__device__ __forceinline__ double theta_only_t(const Law &L, double x)
{
    if (MODEL == kLinear) return L.tr + L.lin_c * x;
    if (!(x < 0.0)) return L.ts;
    if (MODEL == kGardner) return L.tr + L.dT * rs_exp(L.gd_alpha * L.unit * x);
    if (MODEL == kHaverkamp) {
        double hu = -L.unit * x;
        double Q = rs_exp(L.hk_beta * rs_log(hu));
        double den = L.hk_alpha + Q;
        double w = rcp_nr(hu * den);
        return L.tr + L.hk_alpha * L.dT * (hu * w);
    }
    double P = rs_exp(L.vg_n * rs_log(-L.vg_alpha * x));
    return L.tr + L.dT * rs_exp(-L.vg_m * rs_log1p(P));
}

__device__ __forceinline__ double theta_only(const Law &L, double x)
{
    switch (L.model) {
    case kGardner: return theta_only_t<kGardner>(L, x);
    case kHaverkamp: return theta_only_t<kHaverkamp>(L, x);
    case kVgm: return theta_only_t<kVgm>(L, x);
    default: return theta_only_t<kLinear>(L, x);
    }
}

// K(psi) / Ks.
__device__ __forceinline__ double krel(const Law &L, double x)
{
    if (L.model == kLinear || !(x < 0.0)) return 1.0;
    if (L.model == kGardner) return exp(L.gd_alpha * L.unit * x);
    if (L.model == kHaverkamp) {
        double hu = -L.unit * x;
        return L.hk_A / (L.hk_A + exp(L.hk_gamma * log(hu)));
    }
    double lg = log(-L.vg_alpha * x);
    double P = exp(L.vg_n * lg);
    double l1 = log1p(P);
    double Se = exp(-L.vg_m * l1);
    double br = -expm1(L.vg_m * (L.vg_n * lg - l1));
    return sqrt(Se) * br * br;
}

// Feddes stress factor a(psi) and its segment slope (half-open segments).
__device__ __forceinline__ void feddes(const Law &L, double x, double &a, double &da)
{
    if (x < L.h4) { a = 0.0; da = 0.0; }
    else if (x < L.h3) { da = 1.0 / (L.h3 - L.h4); a = (x - L.h4) * da; }
    else if (x < L.h2) { a = 1.0; da = 0.0; }
    else if (x < L.h1) { da = -1.0 / (L.h1 - L.h2); a = (L.h1 - x) / (L.h1 - L.h2); }
    else { a = 0.0; da = 0.0; }
}

// law_unsat where every active lane of the wave is unsaturated and within the
// series' range of its last evaluation; false (and nothing done) otherwise.
template <int MODEL>
__device__ __forceinline__ bool law_scaled(const Law &L, double x, PowState &p, double &s,
                                           double &ds)
{
    const double h = MODEL == kHaverkamp ? -L.unit * x : -x;
    const double u = (h - p.h) * p.ih;
    const double dq = p.q * pow1p_m1_series(u, L.bin1);
    bool good = p.ok & (x < 0.0) & (fabs(u) < L.series_u);
    const double v = dq * p.ix1p;
    if (MODEL == kVgm) good = good & (fabs(v) < L.series_u);
    if (__builtin_amdgcn_ballot_w64(!good) != 0) return false;
    p.q += dq;
    p.h = h;
    if (MODEL == kHaverkamp) {
        const double den = L.hk_alpha + p.q;
        const double w = rcp_1nr(h * den);
        s = h * w;
        ds = p.q * (s * w);
        p.ih = den * w;
    } else {
        s = fma(p.se, pow1p_m1_series(v, L.bin2), p.se);
        const double X = 1.0 + p.q;
        const double w = rcp_1nr(X * h);
        ds = p.q * (s * w);
        p.se = s;
        p.ih = X * w;
        p.ix1p = h * w;
    }
    return true;
}

// Pointwise equation of the NGS update (eq. point-update with the BDF
// coefficient a and sink beta * a_F):  a theta(x) + beta a_F(x) + c x = f.
// NEWTON (or L.newton when NEWTON == 0) safeguarded Newton steps from x0: the
// root stays inside [lo, hi] (initially [(f - a theta_s - beta)/c,
// (f - a theta_r)/c] widened by 1e-12 of the ends' magnitudes, so that the
// root of a saturated cell -- the lower end, F being linear there -- lies
// strictly inside; narrowed by the sign of F at each iterate); a step that does
// not land strictly inside, or a non-positive F', becomes a bisection, unless
// the step leaves the iterate unchanged.  A Newton step (not a bisection) that
// moves x by at most L.newton_tol |x_new| ends the solve for that cell: the
// steps left out would move it by about that step squared times F''/2F'.
// ic = rcp_nr(c) (unused by the linear law); ps: the power terms of the node's
// last evaluation (pow_none() if there is none), left at those of the solve's
// last one.  A wave issues one instruction every 6 to 7 cycles whatever its
// kind, so the loop is written for few of them: F as v + (c x - (f - a theta_r))
// with v = a (theta - theta_r), uniform factors of the law formed once, selects
// instead of branches, the bisection only where some lane needs it.
// PER_LANE: the law differs between lanes (layered media).  KEPT: ps usually
// holds the node's last evaluation.
template <int MODEL, bool SINK, int NEWTON, bool PER_LANE = false, bool KEPT = false>
__device__ __forceinline__ double local_solve_ic(const Law &L, double a, double beta, double c,
                                                 double ic, double f, double x0, PowState &ps)
{
    const double ath = uniform_f64<PER_LANE>(a * L.c_th), adth = uniform_f64<PER_LANE>(a * L.c_dth);
    const double as = uniform_f64<PER_LANE>(a * L.dT);
    const double fr = f - a * L.tr;
    double lo, hi;
    if (MODEL == kLinear) {
        lo = -INFINITY;
        hi = INFINITY;
    } else {
        lo = (f - a * L.ts - beta) * ic;
        hi = fr * ic;
        const double pad = 1e-12 * (fabs(lo) + fabs(hi));
        lo -= pad;
        hi += pad;
    }
    double x = x0;
    bool done = false;
    // three copies of the iteration pay for the Haverkamp law (257^3 sweep 89.8 ->
    // 88.1 us); of the longer vGM law with a sink they spill scalar registers
    // (root box, a step: 13.3 -> 14.1 ms)
    const int iters = NEWTON > 0 ? NEWTON : L.newton;
#pragma clang loop unroll_count(NEWTON == 3 && MODEL == kHaverkamp ? 3 : 1)
    for (int k = 0; k < iters; ++k) {
        double v = 0.0, dF = 0.0, s, ds;
        bool scaled = false;
        if constexpr (KEPT && (MODEL == kHaverkamp || MODEL == kVgm)) {
            // the whole wave unsaturated and close to its last evaluations: the
            // powers scale without a branch per lane
            if (law_scaled<MODEL>(L, x, ps, s, ds)) {
                v = ath * s;
                dF = fma(adth, ds, c);
                scaled = true;
            }
        }
        if (!scaled) {
            v = as;   // saturated: theta_s, theta' = 0
            dF = c;
            if (MODEL == kLinear || x < 0.0) {
                law_unsat<MODEL>(L, x, ps, s, ds);
                v = ath * s;
                dF = fma(adth, ds, c);
            } else {
                ps.ok = false;
            }
        }
        double F = v + fma(c, x, -fr);
        if (SINK) {
            double fa, dfa;
            feddes(L, x, fa, dfa);
            F += beta * fa;
            dF += beta * dfa;
        }
        // x becomes an end of the bracket by the sign of F
        const bool pos = F > 0.0, neg = F < 0.0;
        hi = (pos & !(hi <= x)) ? x : hi;
        lo = (neg & !(lo >= x)) ? x : lo;
        double xn = fma(-F, rcp_1nr(dF), x);
        const bool bisect = !(dF > 0.0) | ((xn != x) & !((xn > lo) & (xn < hi)));
        // (at a root, or where F is not a number, the value stays)
        if (__builtin_amdgcn_ballot_w64(bisect) != 0 && bisect) xn = (pos | neg) ? 0.5 * (lo + hi) : x;
        const bool small = !bisect & (fabs(xn - x) <= L.newton_tol * fabs(xn));
        // lanes whose solve has ended keep their value while the rest of the
        // wave iterates; the wave leaves once every lane has ended
        x = done ? x : xn;
        done = done | small;
        if (__builtin_amdgcn_ballot_w64(!done) == 0) break;
    }
    return x;
}

template <int MODEL, bool SINK, int NEWTON>
__device__ __forceinline__ double local_solve_t(const Law &L, double a, double beta, double c,
                                                double f, double x0)
{
    PowState ps = pow_none();
    return local_solve_ic<MODEL, SINK, NEWTON>(L, a, beta, c,
                                               MODEL == kLinear ? 0.0 : rcp_nr(c), f, x0, ps);
}

// The pointwise solve with the law of one soil picked at run time (layered
// media): the same iteration as local_solve_t for that soil's model.
template <bool SINK, int NEWTON>
__device__ __forceinline__ double local_solve_soil_ic(const Law &Ls, double a, double beta,
                                                      double c, double ic, double f, double x0,
                                                      PowState &ps)
{
    switch (Ls.model) {
    case kGardner: return local_solve_ic<kGardner, SINK, NEWTON, true>(Ls, a, beta, c, ic, f, x0, ps);
    case kHaverkamp: return local_solve_ic<kHaverkamp, SINK, NEWTON, true>(Ls, a, beta, c, ic, f, x0, ps);
    case kVgm: return local_solve_ic<kVgm, SINK, NEWTON, true>(Ls, a, beta, c, ic, f, x0, ps);
    default: return local_solve_ic<kLinear, SINK, NEWTON, true>(Ls, a, beta, c, ic, f, x0, ps);
    }
}

template <bool SINK, int NEWTON>
__device__ __forceinline__ double local_solve_soil(const Law &Ls, double a, double beta, double c,
                                                   double f, double x0)
{
    PowState ps = pow_none();
    return local_solve_soil_ic<SINK, NEWTON>(Ls, a, beta, c, rcp_nr(c), f, x0, ps);
}

// theta at x for a defect, from the power terms of the node's last evaluation.
template <int MODEL>
__device__ __forceinline__ double theta_defect(const Law &L, double x, PowState &ps)
{
    if constexpr (MODEL == kMulti) {
        switch (L.model) {
        case kHaverkamp: return theta_defect<kHaverkamp>(L, x, ps);
        case kVgm: return theta_defect<kVgm>(L, x, ps);
        default: return theta_only(L, x);
        }
    } else if constexpr (MODEL == kHaverkamp || MODEL == kVgm) {
        if (!(x < 0.0)) {
            ps.ok = false;
            return L.ts;
        }
        double s, ds;
        law_unsat<MODEL, true>(L, x, ps, s, ds);
        return L.tr + L.c_th * s;
    } else {
        return theta_only_t<MODEL>(L, x);
    }
}

// Node kinds from indices (no node-type array): Dirichlet if on a Dirichlet
// face or on the patch; value = patch value, else the highest-numbered
// Dirichlet face holding the node (*from_state: that face takes its values
// from the state psi^n).
__device__ __forceinline__ bool dirichlet_at(const Geo &g, int i, int j, int k, double *val,
                                             bool *from_state = nullptr)
{
    const int c[3] = {i, j, k};
    bool dir = false;
    double v = 0.0;
    int face = -1;
    // every array below is indexed by constants only (the loops unroll), so
    // the level's descriptor stays in scalar registers
#pragma unroll
    for (int l = 0; l < 3; ++l) {
        if (l >= g.dim) break;
        if (c[l] == 0 && g.bc[2 * l] == kBcDirichlet) { dir = true; v = g.bcval[2 * l]; face = 2 * l; }
        if (c[l] == g.n[l] - 1 && g.bc[2 * l + 1] == kBcDirichlet) {
            dir = true;
            v = g.bcval[2 * l + 1];
            face = 2 * l + 1;
        }
    }
    if (g.pface >= 0) {
        const int ax = g.pax;
        if ((ax == 0 ? i : (ax == 1 ? j : k)) == g.pat) {
            // the tangential axes in increasing order: (1, 2), (0, 2) or (0, 1)
            const int t0 = ax == 0 ? j : i;
            const int t1 = ax == 2 ? j : k;
            bool in = t0 >= g.plo[0] && t0 <= g.phi[0];
            if (g.dim == 3) in = in && t1 >= g.plo[1] && t1 <= g.phi[1];
            if (in) { dir = true; v = g.pval; face = -1; }
        }
    }
    if (val) *val = v;
    if (from_state) *from_state = face >= 0 && ((g.state_mask >> face) & 1);
    return dir;
}

// dirichlet_at's test (without the value) on a level of DIM axes, every
// descriptor field read unconditionally, so that the reads issue together
// instead of one scalar-load round trip per branch.
template <int DIM>
__device__ __forceinline__ bool dirichlet_t(const Geo &g, int i, int j, int k)
{
    const int c[3] = {i, j, k};
    bool dir = false;
#pragma unroll
    for (int l = 0; l < DIM; ++l)
        dir = dir | ((c[l] == 0) & (g.bc[2 * l] == kBcDirichlet)) |
              ((c[l] == g.n[l] - 1) & (g.bc[2 * l + 1] == kBcDirichlet));
    const int ax = g.pax;
    const int cp = ax == 0 ? i : (ax == 1 ? j : k);
    const int t0 = ax == 0 ? j : i;
    const int t1 = ax == 2 ? j : k;
    bool in = (g.pface >= 0) & (cp == g.pat) & (t0 >= g.plo[0]) & (t0 <= g.phi[0]);
    if (DIM == 3) in = in & (t1 >= g.plo[1]) & (t1 <= g.phi[1]);
    return dir | in;
}

// Division of a 32-bit index by a run-time constant d (Granlund-Montgomery):
// with l = ceil(log2 d) and p = 31 + l, m = ceil(2^p / d) satisfies
// m d - 2^p = e < d <= 2^l, so t m / 2^p = t/d + t e / (d 2^p) < t/d + 1/d for
// t < 2^31 and floor(t m / 2^p) = floor(t / d).  d = 1 is carried as m = 0.
struct FastDiv {
    unsigned m;   // ceil(2^p / d), or 0 for d = 1
    unsigned s;   // p - 32
};

inline FastDiv make_fastdiv(unsigned d)
{
    FastDiv f;
    if (d <= 1) {
        f.m = 0;
        f.s = 0;
        return f;
    }
    unsigned l = 0;
    while ((1ull << l) < d) ++l;
    const unsigned long long p = 31ull + l;
    f.m = (unsigned)(((1ull << p) + d - 1) / d);
    f.s = (unsigned)(p - 32);
    return f;
}

// floor(t / d) for t < 2^31 (grids are limited to 2^31 nodes).
__device__ __forceinline__ unsigned udiv(unsigned t, const FastDiv &f)
{
    return f.m ? (__umulhi(t, f.m) >> f.s) : t;
}

}  // namespace rs
