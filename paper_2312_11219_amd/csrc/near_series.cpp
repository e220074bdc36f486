// Chebyshev coefficients of the near field's frequency dependence (near_moments.hip), in extended
// precision from the values at Chebyshev nodes, rounded once.
#include <algorithm>
#include <array>
#include <cmath>
#include <numeric>

#include "host.h"

namespace gaca {

namespace {

using ld = long double;
struct Cx {
    ld re, im;
};
Cx mul(Cx a, Cx b) { return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }
Cx div(Cx a, Cx b) {
    const ld d = b.re * b.re + b.im * b.im;
    return {(a.re * b.re + a.im * b.im) / d, (a.im * b.re - a.re * b.im) / d};
}
Cx expm(Cx t) {   // e^{-t}
    const ld m = expl(-t.re);
    return {m * cosl(t.im), -m * sinl(t.im)};
}

// Chebyshev coefficients of e^{-z x} on [-1, 1]: I_0(z), then 2 (-1)^k I_k(z).  Modified Bessel functions by
// Miller's backward recurrence I_{k-1} = I_{k+1} + (2 k / z) I_k, normalised by the generating function;
// near 0, where the recurrence overflows, by their power series
void exp_coefficients(Cx z, int K, Cx *a) {
    const ld z2 = z.re * z.re + z.im * z.im;
    if (z2 < 0.25L) {
        const Cx q{0.25L * (z.re * z.re - z.im * z.im), 0.5L * z.re * z.im};   // z^2 / 4
        Cx lead{1, 0};   // (-z / 2)^k / k!
        for (int k = 0; k < K; ++k) {
            Cx s{1, 0};
            for (int m = 12; m > 0; --m) {
                const Cx t = mul(s, q);
                s = {1 + t.re / (m * (ld)(k + m)), t.im / (m * (ld)(k + m))};
            }
            const Cx t = mul(lead, s);
            a[k] = {(k ? 2 : 1) * t.re, (k ? 2 : 1) * t.im};
            lead = mul(lead, {-0.5L * z.re / (k + 1), -0.5L * z.im / (k + 1)});
        }
        return;
    }
    // sum I_0 + 2 sum I_k = e^z; in the left half plane the alternating one, e^{-z}
    const bool left = z.re < 0;
    const Cx iz{2 * z.re / z2, -2 * z.im / z2};
    Cx up{0, 0}, cur{1e-300L, 0}, sum{0, 0};
    for (int k = K + 24; k >= 0; --k) {
        const ld sg = k % 2 ? -1 : 1, w = (k ? 2 : 1) * (left ? sg : 1);
        sum = {sum.re + w * cur.re, sum.im + w * cur.im};
        if (k < K) a[k] = {(k ? 2 : 1) * sg * cur.re, (k ? 2 : 1) * sg * cur.im};
        const Cx t = mul(iz, cur), down{up.re + k * t.re, up.im + k * t.im};
        up = cur;
        cur = down;
    }
    const Cx f = div(left ? expm(z) : expm({-z.re, -z.im}), sum);
    for (int k = 0; k < K; ++k) a[k] = mul(a[k], f);
}

// J_n = int_0^1 u^n e^{-t u} du, n = 0, 1, 2: power series up to |t| = 2 (2^k / k! below 1e-19 from k = 26),
// J_n = (n J_{n-1} - e^{-t}) / t above
void radial(Cx t, Cx (&J)[3]) {
    constexpr int NT = 28;
    static const auto inv = [] {
        std::array<ld, NT + 3> v{};
        for (int k = 1; k < NT + 3; ++k) v[k] = 1.0L / k;
        return v;
    }();
    if (t.re * t.re + t.im * t.im <= 4) {
        Cx term{1, 0};
        J[0] = J[1] = J[2] = {0, 0};
        for (int k = 0; k < NT; ++k) {
            for (int n = 0; n < 3; ++n) J[n] = {J[n].re + term.re * inv[k + n + 1], J[n].im + term.im * inv[k + n + 1]};
            term = mul(term, {-t.re * inv[k + 1], -t.im * inv[k + 1]});
        }
        return;
    }
    const Cx e = expm(t);
    J[0] = div({1 - e.re, -e.im}, t);
    J[1] = div({J[0].re - e.re, J[0].im - e.im}, t);
    J[2] = div({2 * J[1].re - e.re, 2 * J[1].im - e.im}, t);
}

// 2 |I_K(z)| < 2e-17 at the bounds
int terms(double z) { return z <= 1.1 ? 16 : z <= 2.2 ? 20 : z <= 3.7 ? 24 : 30; }

}  // namespace

void SeriesTables::build(double band_max, double reach, double rc_max, const double *re, const double *im, int n) {
    S = NearSeries{};
    rest = true;
    double lo = INFINITY, hi = -INFINITY, top = 0.0, R = 0.0;
    for (int l = 0; l < n; ++l) {
        lo = std::min(lo, re[l]);
        hi = std::max(hi, re[l]);
        top = std::max(top, std::hypot(re[l], im[l]));
    }
    for (int l = 0; l < n; ++l) R = std::max(R, std::hypot(re[l] - 0.5 * (lo + hi), im[l]));
    // the pairs covered: a margin for the device's rounding of a span; e^{-s r_c} and the weights
    // e^{-c (r - r_c)} stay far from the ends of the range of doubles
    S.half = R > 0.0 ? std::min(1.001 * reach, kNearSeriesMax / R) : 1.001 * reach;
    S.rmax = top > 0.0 ? 600.0 / top : INFINITY;
    if (!(S.half > 0.0) || !std::isfinite(S.half) || !std::isfinite(top)) return;
    S.nband = std::max(1, (int)std::ceil(0.5 * (hi - lo) * S.half / band_max));
    // A band costs its points' exponentials and sums, about two frequencies' worth of a point: with fewer than
    // eight frequencies, or four a band, the points are visited at every frequency.  At four a band, near
    // field of all pairs of 768 triangles, every point at every frequency -> moments: single layer 0.52 -> 0.29 ms
    // (three bands), 0.69 -> 0.48 (five); Galerkin 9.7 -> 5.9, 13.7 -> 9.5; P1 2.3 -> 0.5, 3.4 -> 0.9
    if (n < 8 || n < 4 * S.nband || S.nband > kNearBands) return;
    rest = 1.001 * reach > S.half * (1.0 + 1e-12) || !(1.001 * rc_max <= S.rmax);
    std::vector<int> band(n, 0);
    double zmax = 0.0;
    for (int b = 0; b < S.nband; ++b) S.c[b] = lo + (hi - lo) * (b + 0.5) / S.nband;
    for (int l = 0; l < n; ++l) {
        if (hi > lo) band[l] = std::min(S.nband - 1, (int)((re[l] - lo) / (hi - lo) * S.nband));
        zmax = std::max(zmax, std::hypot(re[l] - S.c[band[l]], im[l]) * S.half);
        S.first[band[l] + 1]++;
    }
    for (int b = 0; b < S.nband; ++b) S.first[b + 1] += S.first[b];
    S.K = terms(zmax);
    order.resize(n);
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return band[a] < band[b]; });
    coef.resize((size_t)n * S.K);
    Cx a[32];
    for (int p = 0; p < n; ++p) {
        const int l = order[p];
        exp_coefficients({((ld)re[l] - S.c[band[l]]) * S.half, (ld)im[l] * S.half}, S.K, a);
        for (int k = 0; k < S.K; ++k) coef[(size_t)p * S.K + k] = make_double2((double)a[k].re, (double)a[k].im);
    }
}

// phi(s rho) on 0 <= rho <= S.half from the values at Chebyshev nodes, four more than terms; the three
// kinds share them
void SeriesTables::build_touching(double reach, const double *re, const double *im, int n, SeriesTables (&T)[3]) {
    double lo = INFINITY, top = 0.0;
    for (int l = 0; l < n; ++l) {
        lo = std::min(lo, re[l]);
        top = std::max(top, std::hypot(re[l], im[l]));
    }
    NearSeries S{};
    S.half = top > 0.0 ? std::min(1.001 * reach, 2.0 * kNearSeriesMax / top) : 1.001 * reach;
    S.rmax = INFINITY;
    S.nband = 1;
    S.first[1] = n;
    for (auto &t : T) {
        t.S = NearSeries{};
        t.rest = true;
    }
    // in the left half plane the integrals grow, and their series would lose digits
    if (n < 8 || lo < 0.0 || !(S.half > 0.0) || !std::isfinite(S.half) || !std::isfinite(top)) return;
    const int K = S.K = terms(0.5 * top * S.half);
    const int N = K + 4;           // even
    std::vector<ld> turn(4 * N);   // cos(pi m / (2 N))
    for (int m = 0; m < 4 * N; ++m) turn[m] = cosl(m * (acosl(-1.0L) / (2 * N)));
    for (auto &t : T) {
        t.S = S;
        t.rest = 1.001 * reach > S.half * (1.0 + 1e-12);
        t.order.resize(n);
        std::iota(t.order.begin(), t.order.end(), 0);
        t.coef.resize((size_t)n * K);
    }
    std::vector<Cx> f(3 * N);   // edge u - u^2, vertex u^2, coincident (1 - u)^2
    for (int l = 0; l < n; ++l) {
        for (int i = 0; i < N; ++i) {
            const ld x = 0.5L * (turn[2 * i + 1] + 1) * S.half;
            Cx J[3];
            radial({re[l] * x, im[l] * x}, J);
            f[i] = {J[1].re - J[2].re, J[1].im - J[2].im};
            f[N + i] = J[2];
            f[2 * N + i] = {(J[0].re - J[1].re) - f[i].re, (J[0].im - J[1].im) - f[i].im};
        }
        for (int c = 0; c < 3; ++c) {
            // T_k(-x) = (-1)^k T_k(x): sums and differences of opposite nodes
            for (int i = 0; i < N / 2; ++i) {
                Cx &u = f[c * N + i], &v = f[c * N + N - 1 - i];
                const Cx s{u.re + v.re, u.im + v.im}, d{u.re - v.re, u.im - v.im};
                u = s;
                v = d;
            }
            for (int k = 0; k < K; ++k) {
                ld a = 0, b = 0;
                for (int i = 0; i < N / 2; ++i) {
                    const ld w = turn[k * (2 * i + 1) % (4 * N)];
                    const Cx &v = f[c * N + (k % 2 ? N - 1 - i : i)];
                    a += w * v.re;
                    b += w * v.im;
                }
                const ld w = (k ? 2.0L : 1.0L) / N;
                T[c].coef[(size_t)l * K + k] = make_double2((double)(w * a), (double)(w * b));
            }
        }
    }
}

}  // namespace gaca
