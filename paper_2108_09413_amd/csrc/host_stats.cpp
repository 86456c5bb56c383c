// Host-side decisions of the certification procedure (Alg. 1) and the
// prediction procedure (Alg. 2): Clopper-Pearson lower bound, standard normal
// quantile, two-sided binomial test.  float64 results computed in long double.
#include <cmath>
#include <cstdint>

#include "isr.h"

namespace {

typedef long double ld;

// The functions below come in long double for the results and in double for the first steps of the iterations.
template <class F> struct Limits;
template <> struct Limits<double> { static constexpr double tiny = 1e-290, eps = 1e-15; };
template <> struct Limits<ld> { static constexpr ld tiny = 1e-4000L, eps = 1e-20L; };

// Continued fraction of the regularised incomplete beta function (modified
// Lentz evaluation); valid and fast for x < (a+1)/(a+b+2).
template <class F>
F beta_cf(F a, F b, F x) {
    const F tiny = Limits<F>::tiny, eps = Limits<F>::eps;
    F c = 1, d = 1 - (a + b) * x / (a + 1);
    if (std::fabs(d) < tiny) d = tiny;
    d = 1 / d;
    F h = d;
    for (int m = 1; m < 200000; ++m) {
        F m2 = 2 * (F)m;
        F num = m * (b - m) * x / ((a + m2 - 1) * (a + m2));
        d = 1 + num * d; if (std::fabs(d) < tiny) d = tiny;
        c = 1 + num / c; if (std::fabs(c) < tiny) c = tiny;
        d = 1 / d;
        h *= d * c;
        num = -(a + m) * (a + b + m) * x / ((a + m2) * (a + m2 + 1));
        d = 1 + num * d; if (std::fabs(d) < tiny) d = tiny;
        c = 1 + num / c; if (std::fabs(c) < tiny) c = tiny;
        d = 1 / d;
        F del = d * c;
        h *= del;
        if (std::fabs(del - 1) < eps) break;
    }
    return h;
}

ld log_beta_fn(ld a, ld b) { return lgammal(a) + lgammal(b) - lgammal(a + b); }

// I_x(a, b), a, b > 0, 0 <= x <= 1, with log B(a, b) at hand; *density, if asked for, is that of Beta(a, b) at x.
template <class F>
F inc_beta(F a, F b, F x, F log_beta, F *density = nullptr) {
    if (density) *density = 0;
    if (x <= 0) return 0;
    if (x >= 1) return 1;
    const F pre = std::exp(a * std::log(x) + b * std::log1p(-x) - log_beta);
    if (density) *density = pre / (x * (1 - x));
    if (x < (a + 1) / (a + b + 2)) return pre * beta_cf(a, b, x) / a;
    return 1 - pre * beta_cf(b, a, 1 - x) / b;
}

// Upper tail of the standard normal.
template <class F> F norm_sf(F x) { return (F)0.5L * std::erfc(x * (F)0.70710678118654752440084436210484903928L); }

// x with upper tail q <= 1/2, to 4.5e-4: Abramowitz and Stegun, Handbook of Mathematical Functions, 26.2.23.
double rough_normal_quantile(double q) {
    const double t = std::sqrt(-2.0 * std::log(q));
    return t - (2.515517 + t * (0.802853 + t * 0.010328)) / (1.0 + t * (1.432788 + t * (0.189269 + t * 0.001308)));
}

// One safeguarded Newton phase of isr_cp_lower.  Convergence is quadratic: behind a step the next is about its square times
// half the logarithmic slope of the density (not less than over the law's width, for the slope is 0 at the mode).  A
// step whose next would be `accept` p or less is the last.
template <class F>
F cp_newton(F a, F b, F target, F log_beta, F p, F accept) {
    F lo = 0, hi = 1;
    for (int it = 0; it < 300; ++it) {
        F dens;
        const F f = inc_beta(a, b, p, log_beta, &dens) - target;
        if (f > 0) hi = p; else lo = p;
        const bool newton = dens > 0 && std::isfinite((double)(f / dens));
        F next = newton ? p - f / dens : (lo + hi) / 2;
        const F slope = std::fabs((a - 1) / p - (b - 1) / (1 - p)) / 2 + std::sqrt((a + b) / (p * (1 - p))), step = next - p;
        if (newton && step * step * slope <= accept * p) return next;
        if (!(next > lo && next < hi)) next = (lo + hi) / 2;
        p = next;
        if (hi - lo <= (F)1e-19L * hi) break;
    }
    return p;
}

// The same for isr_normal_quantile, on the log of the tail q; lq = log q.
template <class F>
F quantile_newton(F lq, F x, F accept) {
    F lo = 0, hi = 40;
    for (int it = 0; it < 200; ++it) {
        const F sf = norm_sf(x);
        const F g = std::log(sf) - lq;              // decreasing in x
        if (g > 0) lo = x; else hi = x;
        const F dens = (F)0.39894228040143267793994605993438L * std::exp(-x * x / 2);
        F next = x + g * sf / dens;
        if (std::fabs(next - x) <= accept * std::fabs(x)) return next;
        if (!(next > lo && next < hi)) next = (lo + hi) / 2;
        x = next;
        if (hi - lo <= (F)1e-19L * hi) break;
    }
    return x;
}

}  // namespace

extern "C" int isr_cp_lower(uint32_t k, uint32_t n, double alpha, double *p_lower) {
    if (!p_lower || n == 0 || k > n || !(alpha > 0.0 && alpha < 1.0)) return ISR_ERR_ARG;
    if (k == 0) { *p_lower = 0.0; return ISR_OK; }
    if (k == n) { *p_lower = (double)expl(logl((ld)alpha) / (ld)n); return ISR_OK; }
    // Root in p of P[Bin(n, p) >= k] = I_p(k, n-k+1) = alpha: safeguarded Newton from the normal approximation with the
    // score interval, in double first (most of the steps at a fraction of their cost), then in long double until the next
    // step would be far below the last place of p.
    const ld a = k, b = (ld)n - k + 1.0L, log_beta = log_beta_fn(a, b);
    const double ph = (double)k / n, z = rough_normal_quantile(alpha < 0.5 ? alpha : 0.5), zz = z * z / n;
    double p0 = (ph + zz / 2 - z * std::sqrt(ph * (1 - ph) / n + zz / (4.0 * n))) / (1 + zz);
    if (!(p0 > 0.0 && p0 < 1.0)) p0 = ph * 0.5;
    p0 = cp_newton<double>((double)a, (double)b, alpha, (double)log_beta, p0, 1e-11);
    const ld p = cp_newton<ld>(a, b, alpha, log_beta, p0 > 0.0 && p0 < 1.0 ? (ld)p0 : ph * 0.5L, 1e-18L);
    *p_lower = (double)p;
    return ISR_OK;
}

extern "C" int isr_normal_quantile(double p, double *z) {
    if (!z || !(p > 0.0 && p < 1.0)) return ISR_ERR_ARG;
    if (p == 0.5) { *z = 0.0; return ISR_OK; }
    // Solve the upper-tail equation on the side where the tail is <= 1/2.
    const bool upper = p > 0.5;
    const ld q = upper ? (ld)1.0 - (ld)p : (ld)p;  // exact in long double
    const ld lq = logl(q);
    // double first, then long double; the convergence is quadratic: behind a step of 1e-12 x the next would be below the last
    // place of x
    double x0 = rough_normal_quantile((double)q);
    if (!(x0 > 0.0)) x0 = (0.5 - (double)q) * 2.5066282746310005024;
    if ((double)q > 1e-290) x0 = quantile_newton<double>((double)lq, x0, 1e-8);
    const ld x = quantile_newton<ld>(lq, x0, 1e-12L);
    *z = (double)(upper ? x : -x);
    return ISR_OK;
}

extern "C" int isr_binom_pvalue(uint32_t n_a, uint32_t n_b, double *pvalue) {
    if (!pvalue) return ISR_ERR_ARG;
    if (n_a == 0) { *pvalue = 1.0; return ISR_OK; }
    // P[Bin(m, 1/2) >= n_a], m = n_a + n_b: n_b + 1 terms C(m, j) 2^-m, j = 0 .. n_b; where there are many, the incomplete
    // beta function I_{1/2}(n_a, n_b + 1)
    ld tail;
    if (n_b <= 100 && n_a <= 16000) {
        ld term = ldexpl(1.0L, -(int)(n_a + n_b));
        tail = term;
        for (uint32_t j = 1; j <= n_b; ++j) {
            term = term * (ld)(n_a + n_b - j + 1) / (ld)j;
            tail += term;
        }
    } else {
        const ld a = n_a, b = (ld)n_b + 1.0L;
        tail = inc_beta(a, b, 0.5L, log_beta_fn(a, b));
    }
    ld pv = 2.0L * tail;
    *pvalue = (double)(pv > 1.0L ? 1.0L : pv);
    return ISR_OK;
}

static uint32_t lowest_argmax(const uint32_t *c, uint32_t n) {
    uint32_t best = 0;
    for (uint32_t i = 1; i < n; ++i) if (c[i] > c[best]) best = i;
    return best;
}

extern "C" int isr_decide_certify(const uint32_t *counts0, const uint32_t *counts1, uint32_t classes,
                                  double sigma, uint32_t n, double alpha, isr_result *out) {
    if (!counts0 || !counts1 || !out || classes == 0 || !(sigma > 0.0)) return ISR_ERR_ARG;
    uint32_t ca = lowest_argmax(counts0, classes);
    uint32_t k = counts1[ca];
    double pl = 0.0;
    int rc = isr_cp_lower(k, n, alpha, &pl);
    if (rc != ISR_OK) return rc;
    out->n_top = k;
    out->n_second = 0;
    out->p_lower = pl;
    out->radius_int = 0;
    out->radius_sq_int = 0;
    if (pl > 0.5) {
        double z = 0.0;
        rc = isr_normal_quantile(pl, &z);
        if (rc != ISR_OK) return rc;
        out->cls = (int32_t)ca;
        out->radius = sigma * z;
        // integer-only tail (Thm 3.2, proof steps 2-3): quantile of the discrete law by table lookup
        if (sigma >= 1.0 && sigma <= 1024.0 && sigma == std::floor(sigma)) {
            rc = isr_discrete_quantile((uint32_t)sigma, pl, &out->radius_int, &out->radius_sq_int);
            if (rc != ISR_OK) return rc;
        }
    } else {
        out->cls = ISR_ABSTAIN;
        out->radius = 0.0;
    }
    return ISR_OK;
}

extern "C" int isr_decide_predict(const uint32_t *counts, uint32_t classes, double alpha, isr_result *out) {
    if (!counts || !out || classes == 0 || !(alpha > 0.0 && alpha < 1.0)) return ISR_ERR_ARG;
    uint32_t ca = lowest_argmax(counts, classes);
    uint32_t nb = 0;
    for (uint32_t i = 0; i < classes; ++i) if (i != ca && counts[i] > nb) nb = counts[i];
    double pv = 1.0;
    int rc = isr_binom_pvalue(counts[ca], nb, &pv);
    if (rc != ISR_OK) return rc;
    out->radius_int = 0;
    out->radius_sq_int = 0;
    out->n_top = counts[ca];
    out->n_second = nb;
    out->p_lower = pv;
    out->radius = 0.0;
    out->cls = pv <= alpha ? (int32_t)ca : ISR_ABSTAIN;
    return ISR_OK;
}

extern "C" int isr_certified_metrics(const isr_result *results, const int32_t *labels, uint32_t count, const double *radii,
                                     uint32_t n_radii, double *cp_out, double *ca_out) {
    if (!results || count == 0 || (n_radii && (!radii || !ca_out || !labels))) return ISR_ERR_ARG;
    uint32_t certified = 0;
    for (uint32_t i = 0; i < count; ++i) certified += results[i].cls != ISR_ABSTAIN;
    if (cp_out) *cp_out = (double)certified / (double)count;
    for (uint32_t j = 0; j < n_radii; ++j) {
        uint32_t hit = 0;
        for (uint32_t i = 0; i < count; ++i)
            hit += results[i].cls != ISR_ABSTAIN && results[i].cls == labels[i] && results[i].radius >= radii[j];
        ca_out[j] = certified ? (double)hit / (double)certified : 0.0;
    }
    return ISR_OK;
}
