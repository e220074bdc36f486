// Near field of every frequency from moments of the quadrature points.
//
// An entry is sum_q w_q k(r_q) e^{-s r_q} over the points of its rule.  With the frequencies in the
// disc |s - c| <= R (c real) and the distances in r_c +- delta, R delta <= 6, the sum is a power
// series in (s - c) / R,
//   e^{-s r_c} sum_m (-(s - c) / R)^m M_m,   M_m = sum_q w_q k(r_q) e^{-c (r_q - r_c)} tau_q^m / m!,
//   tau_q = R (r_q - r_c),
// cut after K terms where the rest is below the rounding of the sum (R delta up to 2: 24 terms,
// 2^24 / 24! = 3e-17; 3.5: 32, 1e-18; 6: 44, 6e-21).  The points are visited once, with one real exponential each, instead of once
// per frequency with e^x, sin and cos; a frequency then costs K complex steps.  The double layer's
// factor 1 + s r = (1 + s r_c) + s (r - r_c) takes the derivative of the series along:
//   sum_q (r_q - r_c) ... = P'(u) / R,  u = -(s - c) / R.
// Touching and coincident Galerkin pairs carry exact radial integrals of e^{-s rho u},
//   phi2: u^2,  phie: u - u^2,  psi: (1 - u)^2,   0 <= u <= 1;
// with J_n(x) = int u^n e^{-x u} du their moments are combinations of
// S_m^p = sum_q w_q tau_q^m / m! J_{m+p}(c rho_q), p = 0, 1, 2, and J_n = (x J_{n+1} + e^{-x}) / (n + 1) gives
//   S_m^p = ((c / R) (m + 1) S_{m+1}^p + B_m) / (m + p + 1)
// from the moments B_m = sum_q w_q e^{-c rho_q} tau_q^m / m!, tau = R rho (max(|c|, R) rho <= 6: all
// sums are of one sign and the start from 0 at m = K is below the rounding).
//
// What bounds it: the moments' multiply-adds (FP64 VALU, two per moment and point) where a rule has
// many points, the writes of the entries and the steps per frequency where it has few.  G lanes
// share a pair, first its points, then its frequencies.  Near field of a build, every point at every
// frequency -> moments: Galerkin P0 (3072-triangle L-shape, L = 96) 82 -> 5.6 ms; P1 double layer
// (4802-vertex sphere, L = 128) 49 -> 10 ms; collocation (9408-triangle sphere, L = 128) 17.5 ->
// 9.1 ms, of which the writes of its 18 GB take 4.  Pairs beyond the bound (few elements per
// wavelength) are left to the kernels that visit the points at every frequency.
#include <hip/hip_runtime.h>

#include "device_util.h"
#include "entries_dev.h"
#include "galerkin_dev.h"
#include "kernels.h"
#include "near_series_dev.h"

namespace gaca {

namespace {

template <int K>
struct InvFact {
    double v[K];
    constexpr InvFact() : v{} {
        double f = 1.0;
        for (int k = 0; k < K; ++k) {
            if (k > 0) f /= k;
            v[k] = f;
        }
    }
};

// sum over G adjacent lanes (a power of two up to 16), in every one of them
template <int G>
__device__ __forceinline__ double group_sum(double v) {
    if (G > 1) v += dpp_d<0xB1>(v);
    if (G > 2) v += dpp_d<0x4E>(v);
    if (G > 4) v += dpp_d<0x141>(v);
    if (G > 8) v += dpp_d<0x140>(v);
    return v;
}

template <int K>
struct Moments {
    double m[K];
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int k = 0; k < K; ++k) m[k] = 0.0;
    }
    __device__ __forceinline__ void add(double tau, double w) {
        double t = w;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            m[k] += t;
            t *= tau;
        }
    }
    // the lanes' sums together, over k!
    template <int G>
    __device__ __forceinline__ void finish() {
        constexpr InvFact<K> F;
#pragma unroll
        for (int k = 0; k < K; ++k) m[k] = group_sum<G>(m[k]) * F.v[k];
    }
    // B_m -> S_m^2 (WHAT 0), S_m^1 - S_m^2 (1), S_m^0 - 2 S_m^1 + S_m^2 (2)
    template <int WHAT>
    __device__ __forceinline__ void radial(double cr) {
        double s0 = 0.0, s1 = 0.0, s2 = 0.0;
#pragma unroll
        for (int k = K - 1; k >= 0; --k) {
            const double b = m[k], a = cr * (k + 1);
            s2 = fma(a, s2, b) * (1.0 / (k + 3));
            if (WHAT > 0) s1 = fma(a, s1, b) * (1.0 / (k + 2));
            if (WHAT > 1) s0 = fma(a, s0, b) * (1.0 / (k + 1));
            m[k] = WHAT == 0 ? s2 : WHAT == 1 ? s1 - s2 : (s0 - s1) - (s1 - s2);
        }
    }
    // P(u) (and P'(u))
    template <bool D>
    __device__ __forceinline__ void eval(double ur, double ui, double2 &P, double2 &dP) const {
        double pr = m[K - 1], pi = 0.0, dr = 0.0, di = 0.0;
#pragma unroll
        for (int k = K - 2; k >= 0; --k) {
            if (D) {
                const double nr = fma(ur, dr, fma(-ui, di, pr));
                di = fma(ur, di, fma(ui, dr, pi));
                dr = nr;
            }
            const double nr = fma(ur, pr, fma(-ui, pi, m[k]));
            pi = fma(ur, pi, ui * pr);
            pr = nr;
        }
        P = make_double2(pr, pi);
        dP = make_double2(dr, di);
    }
};

template <int KERNEL, int K>
__device__ __forceinline__ void add_point(Moments<K> &M, const NearSeries &S, double rc, double r, double ir, double w) {
    const double dr = r - rc;
    M.add(S.R * dr, w * kInvFourPi * (KERNEL == 0 ? ir : ir * ir * ir) * fm::exp(-S.c * dr));
}

// points sub, sub + G, ... of the collapsed n x n rule on (a, b, c) seen from x; lam < 0, or the
// barycentric coordinate that weighs them
template <int KERNEL, int K, int G>
__device__ __forceinline__ void add_collapsed(Moments<K> &M, const NearSeries &S, double rc, const double *x,
                                              const double *a, const double *b, const double *c, int n,
                                              const double *gt, double wscale, int sub, int lam = -1) {
    const double e1x = b[0] - a[0], e1y = b[1] - a[1], e1z = b[2] - a[2];
    const double e2x = c[0] - b[0], e2y = c[1] - b[1], e2z = c[2] - b[2];
    const double nx = e1y * e2z - e1z * e2y, ny = e1z * e2x - e1x * e2z, nz = e1x * e2y - e1y * e2x;
    const double ws = sqrt(nx * nx + ny * ny + nz * nz) * wscale;
    for (int p = sub; p < n * n; p += G) {
        const int iu = p / n, iv = p - iu * n;
        const double u = gt[2 * iu], uv = u * gt[2 * iv];
        double w = gt[2 * iu + 1] * gt[2 * iv + 1] * u * ws, ir;
        if (lam >= 0) w *= lam == 0 ? 1.0 - u : (lam == 1 ? u - uv : uv);
        const double r = dist3_inv(x[0], x[1], x[2], a[0] + u * e1x + uv * e2x, a[1] + u * e1y + uv * e2y,
                                   a[2] + u * e1z + uv * e2z, ir);
        add_point<KERNEL, K>(M, S, rc, r, ir, w);
    }
}

// w / (4 pi rho) at the end of the radial integral along d
template <int K>
__device__ __forceinline__ void add_radial(Moments<K> &M, const NearSeries &S, const double *d, double w) {
    const double rho = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
    M.add(S.R * rho, w / (kFourPi * rho) * fm::exp(-S.c * rho));
}

template <int TIER, int K, int G>
__device__ __forceinline__ void gal_moments(Moments<K> &M, const GeoDev &g, const QuadDev &q, const NearSeries &S,
                                            double rc, int64_t i, int64_t j, int sub) {
    const double aj[3] = {g.ax[j], g.ay[j], g.az[j]}, bj[3] = {g.bx[j], g.by[j], g.bz[j]},
                 cj[3] = {g.cx[j], g.cy[j], g.cz[j]};
    const double ai[3] = {g.ax[i], g.ay[i], g.az[i]}, bi[3] = {g.bx[i], g.by[i], g.bz[i]},
                 ci[3] = {g.cx[i], g.cy[i], g.cz[i]};
    if constexpr (TIER == GT_FAR36) {
        const int64_t T = g.M;
        for (int p = sub; p < 36; p += G) {
            const int pi = p / 6, pj = p - 6 * pi;
            double ir;
            const double r = dist3_inv(g.q6x[pi * T + i], g.q6y[pi * T + i], g.q6z[pi * T + i], g.q6x[pj * T + j],
                                       g.q6y[pj * T + j], g.q6z[pj * T + j], ir);
            add_point<0, K>(M, S, rc, r, ir, g.q6w[pi * T + i] * g.q6w[pj * T + j]);
        }
    } else if constexpr (TIER == GT_MID || TIER == GT_NEAR) {
        const int no = TIER == GT_MID ? q.n4 : q.ng;
        const double *go = TIER == GT_MID ? q.g4 : q.gg;
        const double e1x = bi[0] - ai[0], e1y = bi[1] - ai[1], e1z = bi[2] - ai[2];
        const double e2x = ci[0] - bi[0], e2y = ci[1] - bi[1], e2z = ci[2] - bi[2];
        const double nx = e1y * e2z - e1z * e2y, ny = e1z * e2x - e1x * e2z, nz = e1x * e2y - e1y * e2x;
        const double ws = sqrt(nx * nx + ny * ny + nz * nz);
        // an item: an outer point (MID), an outer point and one of its three sub-triangles (NEAR)
        const int parts = TIER == GT_MID ? 1 : 3;
        for (int it = sub; it < no * no * parts; it += G) {
            const int o = it / parts, s = it - o * parts, iu = o / no, iv = o - iu * no;
            const double u = go[2 * iu], uv = u * go[2 * iv], wx = go[2 * iu + 1] * go[2 * iv + 1] * u * ws;
            const double x[3] = {ai[0] + u * e1x + uv * e2x, ai[1] + u * e1y + uv * e2y, ai[2] + u * e1z + uv * e2z};
            if constexpr (TIER == GT_MID) {
                add_collapsed<0, K, 1>(M, S, rc, x, aj, bj, cj, q.n4, q.g4, wx, 0);
            } else {
                double p[3];
                closest_on_triangle(x, aj, bj, cj, p);
                const double *V1 = s == 0 ? bj : (s == 1 ? cj : aj), *V2 = s == 0 ? cj : (s == 1 ? aj : bj);
                const double p1[3] = {V1[0], V1[1], V1[2]}, p2[3] = {V2[0], V2[1], V2[2]};
                add_collapsed<0, K, 1>(M, S, rc, x, p, p1, p2, q.ng, q.gg, wx, 0);
            }
        }
    } else if constexpr (TIER == GT_COINC) {
        // in-plane frame at the first vertex, gradients of the barycentric coordinates, sectors
        // between the edge directions (the frame of gal_coincident)
        double ux = bj[0] - aj[0], uy = bj[1] - aj[1], uz = bj[2] - aj[2];
        const double lu = sqrt(ux * ux + uy * uy + uz * uz);
        ux /= lu; uy /= lu; uz /= lu;
        const double wx = cj[0] - aj[0], wy = cj[1] - aj[1], wz = cj[2] - aj[2];
        const double wu = wx * ux + wy * uy + wz * uz;
        const double vx = wx - wu * ux, vy = wy - wu * uy, vz = wz - wu * uz;
        const double lv = sqrt(vx * vx + vy * vy + vz * vz);
        const double Px[3] = {0.0, lu, wu}, Py[3] = {0.0, 0.0, lv}, A2 = lu * lv;
        double Gx[3], Gy[3], th[6];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int k1 = (k + 1) % 3, k2 = (k + 2) % 3;
            Gx[k] = (Py[k1] - Py[k2]) / A2;
            Gy[k] = (Px[k2] - Px[k1]) / A2;
            double t = atan2(Py[k1] - Py[k], Px[k1] - Px[k]);
            if (t < 0.0) t += 2.0 * M_PI;
            th[2 * k] = t;
            double t2 = t + M_PI;
            if (t2 >= 2.0 * M_PI) t2 -= 2.0 * M_PI;
            th[2 * k + 1] = t2;
        }
#pragma unroll
        for (int a = 0; a < 5; ++a)
#pragma unroll
            for (int b = 0; b < 5 - a; ++b) {
                const double lo = fmin(th[b], th[b + 1]), hi = fmax(th[b], th[b + 1]);
                th[b] = lo;
                th[b + 1] = hi;
            }
#pragma unroll
        for (int sct = 0; sct < 6; ++sct) {
            const double ta = th[sct], span = (sct == 5 ? th[0] + 2.0 * M_PI : th[(sct + 1) % 6]) - ta;
            if (span <= 0.0) continue;
            for (int p = sub; p < q.nth; p += G) {
                double sn, cs;
                sincos(ta + span * q.gth[2 * p], &sn, &cs);
                double gsum = 0.0;
#pragma unroll
                for (int k = 0; k < 3; ++k) gsum += fmax(0.0, Gx[k] * cs + Gy[k] * sn);
                const double R = 1.0 / gsum;
                // area / (4 pi) R psi(s R)
                M.add(S.R * R, 0.5 * A2 / kFourPi * span * q.gth[2 * p + 1] * R * fm::exp(-S.c * R));
            }
        }
    } else {
        // shared vertices (equal coordinates): positions in tau_i (ascending) and tau_j
        const double *Vi[3] = {ai, bi, ci}, *Vj[3] = {aj, bj, cj};
        int ns = 0, pi0 = 0, pj0 = 0, pi1 = 0, pj1 = 0;
#pragma unroll
        for (int va = 0; va < 3; ++va)
#pragma unroll
            for (int vb = 0; vb < 3; ++vb)
                if (Vi[va][0] == Vj[vb][0] && Vi[va][1] == Vj[vb][1] && Vi[va][2] == Vj[vb][2]) {
                    if (ns == 0) {
                        pi0 = va;
                        pj0 = vb;
                    } else {
                        pi1 = va;
                        pj1 = vb;
                    }
                    ++ns;
                }
        auto pick = [](const double *a, const double *b, const double *c, int k, int d) {
            return k == 0 ? a[d] : (k == 1 ? b[d] : c[d]);
        };
        const double sc = 4.0 * g.area[i] * g.area[j];
        const int n = q.ns;
        const double *t = q.gs;
        if constexpr (TIER == GT_EDGE) {
            double E[3], A[3], B[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const double P1 = pick(ai, bi, ci, pi1, k);
                E[k] = P1 - pick(ai, bi, ci, pi0, k);
                A[k] = pick(ai, bi, ci, 3 - pi0 - pi1, k) - P1;
                B[k] = pick(aj, bj, cj, 3 - pj0 - pj1, k) - P1;
            }
            for (int p = sub; p < n * n; p += G) {
                const int p2 = p / n, p3 = p - p2 * n;
                const double e2 = t[2 * p2], e3 = t[2 * p3], w = sc * t[2 * p2 + 1] * t[2 * p3 + 1];
                // coefficients of (E, A, B) in d for the five pieces
                const double c[5][3] = {{e2, e3, -(1.0 - e2)},
                                        {e2 * e3, 1.0, -e2 * (1.0 - e3)},
                                        {-e2, 1.0 - e2, -e2 * e3},
                                        {-e2 * e3, e2 * (1.0 - e3), -1.0},
                                        {-e2 * e3, 1.0 - e2 * e3, -e2}};
#pragma unroll
                for (int r = 0; r < 5; ++r) {
                    double d[3];
#pragma unroll
                    for (int k = 0; k < 3; ++k) d[k] = c[r][0] * E[k] + c[r][1] * A[k] + c[r][2] * B[k];
                    add_radial<K>(M, S, d, r == 0 ? w : w * e2);
                }
            }
        } else {
            double X1[3], X2[3], Y1[3], Y2[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const double a1 = pick(ai, bi, ci, (pi0 + 1) % 3, k), b1 = pick(aj, bj, cj, (pj0 + 1) % 3, k),
                             V = pick(ai, bi, ci, pi0, k);
                X1[k] = a1 - V;
                X2[k] = pick(ai, bi, ci, (pi0 + 2) % 3, k) - a1;
                Y1[k] = b1 - V;
                Y2[k] = pick(aj, bj, cj, (pj0 + 2) % 3, k) - b1;
            }
            for (int p = sub; p < n * n; p += G) {
                const int p1 = p / n, p2 = p - p1 * n;
                const double e1 = t[2 * p1], e2 = t[2 * p2], w12 = sc * t[2 * p1 + 1] * t[2 * p2 + 1] * e2;
                for (int p3 = 0; p3 < n; ++p3) {
                    const double e3 = t[2 * p3], w = w12 * t[2 * p3 + 1];
                    double d[3];
#pragma unroll
                    for (int k = 0; k < 3; ++k) d[k] = (X1[k] + e1 * X2[k]) - e2 * (Y1[k] + e3 * Y2[k]);
                    add_radial<K>(M, S, d, w);
#pragma unroll
                    for (int k = 0; k < 3; ++k) d[k] = e2 * (X1[k] + e3 * X2[k]) - (Y1[k] + e1 * Y2[k]);
                    add_radial<K>(M, S, d, w);
                }
            }
        }
    }
}

// the entry at the frequencies sub, sub + G, ... (KERNEL 1: with the factor 1 + s r)
template <int KERNEL, int K, int G>
__device__ __forceinline__ void write_entry(const Moments<K> &M, const NearSeries &S, const FreqDev &f, double rc,
                                            double num, int sub, int64_t base, int n, double2 *out64, float2 *out32) {
    const double iR = 1.0 / S.R;
    for (int l = sub; l < f.L_eval; l += G) {
        const double sr = f.re[l], si = f.im[l];
        double2 P, D;
        M.template eval<KERNEL == 1>((S.c - sr) * iR, -si * iR, P, D);
        if (KERNEL == 1) {
            // (1 + s r_c) P + s P' / R
            const double ar = fma(sr, rc, 1.0), ai = si * rc, br = sr * iR, bi = si * iR;
            const double pr = ar * P.x - ai * P.y + (br * D.x - bi * D.y);
            P.y = ar * P.y + ai * P.x + (br * D.y + bi * D.x);
            P.x = pr;
        }
        const double mag = num * fm::exp(-sr * rc);
        double sn, cs;
        fm::sincos(si * rc, &sn, &cs);
        const double er = mag * cs, ei = -mag * sn;
        const double vr = er * P.x - ei * P.y, vi = er * P.y + ei * P.x;
        const int64_t o = base + (int64_t)l * n, om = base + (int64_t)(f.L - 1 - l) * n;
        const bool mir = f.mirror && f.L - 1 - l != l;
        if (out64) {
            out64[o] = make_double2(vr, vi);
            if (mir) out64[om] = make_double2(vr, -vi);
        } else {
            out32[o] = make_float2((float)vr, (float)vi);
            if (mir) out32[om] = make_float2((float)vr, (float)-vi);
        }
    }
}

// CLS: Galerkin class (GAL), collocation tier, or the P1 double layer
enum { GAL = 0, COL = 1, P1 = 2 };
template <int WHAT, int KERNEL, int TIER, int K, int G>
__global__ void __launch_bounds__(256)
    near_series_kernel(GeoDev g, QuadDev q, FreqDev f, NearSeries S, const NearPair *__restrict__ pairs,
                       int64_t npairs, const NearBlockDev *__restrict__ blocks, double2 *out64, float2 *out32) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x, p = t / G;
    const int sub = (int)(t % G);
    if (p >= npairs) return;   // the G lanes of a pair together
    const NearPair pr = pairs[p];
    const NearBlockDev B = blocks[pr.blk];
    const int64_t i = B.r0 + pr.i, j = B.c0 + pr.j;
    double rc, num = 1.0;
    double z;
    if constexpr (WHAT == GAL) z = gal_span<TIER>(g, S, i, j, rc);
    else if constexpr (WHAT == COL) z = near_span(g, S, i, j, rc);
    else z = p1_span(g, S, i, j, rc);
    if (!(z <= kNearSeriesMax)) return;
    Moments<K> M;
    M.zero();
    if constexpr (WHAT == GAL) {
        gal_moments<TIER, K, G>(M, g, q, S, rc, i, j, sub);
    } else if constexpr (WHAT == COL) {
        const double x[3] = {g.xx[i], g.xy[i], g.xz[i]};
        const double a[3] = {g.ax[j], g.ay[j], g.az[j]}, b[3] = {g.bx[j], g.by[j], g.bz[j]},
                     c[3] = {g.cx[j], g.cy[j], g.cz[j]};
        if constexpr (TIER == TIER_FAR6) {
            const int64_t T = g.M;
            for (int k = sub; k < 6; k += G) {
                double ir;
                const double r = dist3_inv(x[0], x[1], x[2], g.q6x[k * T + j], g.q6y[k * T + j], g.q6z[k * T + j], ir);
                add_point<KERNEL, K>(M, S, rc, r, ir, g.q6w[k * T + j]);
            }
        } else if constexpr (TIER == TIER_SELF) {
            for (int e = 0; e < 3; ++e) {
                const double *p1 = e == 0 ? b : (e == 1 ? c : a), *p2 = e == 0 ? c : (e == 1 ? a : b);
                const double v1[3] = {p1[0], p1[1], p1[2]}, v2[3] = {p2[0], p2[1], p2[2]};
                add_collapsed<KERNEL, K, G>(M, S, rc, x, x, v1, v2, q.nd, q.gd, 1.0, sub);
            }
        } else {
            add_collapsed<KERNEL, K, G>(M, S, rc, x, a, b, c, TIER == TIER_MID4 ? q.n4 : q.n8,
                                        TIER == TIER_MID4 ? q.g4 : q.g8, 1.0, sub);
        }
        if (KERNEL == 1) num = g.nx[j] * x[0] + g.ny[j] * x[1] + g.nz[j] * x[2] - g.d[j];
    } else {
        const double x[3] = {g.xx[i], g.xy[i], g.xz[i]};
        const int32_t vid = g.dvid[i];
        for (int32_t e = g.pptr[j]; e < g.pptr[j + 1]; ++e) {
            const int64_t tr = g.ptri[e];
            if (p1_holds(g, tr, vid)) continue;
            const int loc = g.ploc[e];
            const double nt = g.nx[tr] * x[0] + g.ny[tr] * x[1] + g.nz[tr] * x[2] - g.d[tr];
            const double qd = dist3(x[0], x[1], x[2], g.tcx[tr], g.tcy[tr], g.tcz[tr]) / g.h[tr];
            if (qd >= 4.0) {
                const int64_t T = g.T;
                for (int k = sub; k < 6; k += G) {
                    double ir;
                    const double r =
                        dist3_inv(x[0], x[1], x[2], g.q6x[k * T + tr], g.q6y[k * T + tr], g.q6z[k * T + tr], ir);
                    add_point<1, K>(M, S, rc, r, ir, nt * g.q6wl[(int64_t)(loc * 6 + k) * T + tr]);
                }
            } else {
                const double a[3] = {g.ax[tr], g.ay[tr], g.az[tr]}, b[3] = {g.bx[tr], g.by[tr], g.bz[tr]},
                             c[3] = {g.cx[tr], g.cy[tr], g.cz[tr]};
                add_collapsed<1, K, G>(M, S, rc, x, a, b, c, qd >= 2.0 ? q.n4 : q.n8, qd >= 2.0 ? q.g4 : q.g8, nt, sub,
                                       loc);
            }
        }
    }
    M.template finish<G>();
    if constexpr (WHAT == GAL && TIER >= GT_EDGE)
        M.template radial<TIER == GT_VERTEX ? 0 : TIER == GT_EDGE ? 1 : 2>(S.c / S.R);
    const int64_t base = B.off + (int64_t)pr.i * f.L * B.n + pr.j;
    write_entry<KERNEL, K, G>(M, S, f, rc, num, sub, base, B.n, out64, out32);
}

template <int WHAT, int KERNEL, int TIER, int G>
void launch(const GeoDev &g, const QuadDev &q, const FreqDev &f, const NearSeries &S, const NearPair *pairs,
            int64_t npairs, const NearBlockDev *blocks, double2 *o64, float2 *o32, hipStream_t st) {
    const unsigned nb = (unsigned)((npairs * G + 255) / 256);
#define GACA_SERIES(K) \
    near_series_kernel<WHAT, KERNEL, TIER, K, G><<<nb, 256, 0, st>>>(g, q, f, S, pairs, npairs, blocks, o64, o32)
    if (S.K == 24) GACA_SERIES(24);
    else if (S.K == 32) GACA_SERIES(32);
    else GACA_SERIES(44);
#undef GACA_SERIES
}

}  // namespace

void launch_near_series_galerkin(int tier, const GeoDev &g, const QuadDev &q, const FreqDev &f, const NearSeries &S,
                                 const NearPair *pairs, int64_t npairs, const NearBlockDev *blocks, double2 *o64,
                                 float2 *o32, hipStream_t st) {
    if (npairs <= 0) return;
#define GACA_NEAR(T, G) launch<GAL, 0, T, G>(g, q, f, S, pairs, npairs, blocks, o64, o32, st)
    switch (tier) {
        case GT_FAR36: GACA_NEAR(GT_FAR36, 4); break;
        case GT_MID: GACA_NEAR(GT_MID, 4); break;
        case GT_NEAR: GACA_NEAR(GT_NEAR, 8); break;
        case GT_EDGE: GACA_NEAR(GT_EDGE, 16); break;
        case GT_VERTEX: GACA_NEAR(GT_VERTEX, 16); break;
        default: GACA_NEAR(GT_COINC, 16); break;
    }
#undef GACA_NEAR
}

void launch_near_series(int kernel, int tier, const GeoDev &g, const QuadDev &q, const FreqDev &f, const NearSeries &S,
                        const NearPair *pairs, int64_t npairs, const NearBlockDev *blocks, double2 *o64, float2 *o32,
                        hipStream_t st) {
    if (npairs <= 0) return;
#define GACA_NEAR(K, T, G) launch<COL, K, T, G>(g, q, f, S, pairs, npairs, blocks, o64, o32, st)
    if (kernel == 0) {
        switch (tier) {
            case TIER_FAR6: GACA_NEAR(0, TIER_FAR6, 1); break;
            case TIER_MID4: GACA_NEAR(0, TIER_MID4, 4); break;
            case TIER_NEAR8: GACA_NEAR(0, TIER_NEAR8, 8); break;
            default: GACA_NEAR(0, TIER_SELF, 16); break;
        }
    } else {
        switch (tier) {
            case TIER_FAR6: GACA_NEAR(1, TIER_FAR6, 1); break;
            case TIER_MID4: GACA_NEAR(1, TIER_MID4, 4); break;
            default: GACA_NEAR(1, TIER_NEAR8, 8); break;
        }
    }
#undef GACA_NEAR
}

void launch_near_series_p1(const GeoDev &g, const QuadDev &q, const FreqDev &f, const NearSeries &S,
                           const NearPair *pairs, int64_t npairs, const NearBlockDev *blocks, double2 *o64,
                           hipStream_t st) {
    if (npairs > 0) launch<P1, 1, 0, 8>(g, q, f, S, pairs, npairs, blocks, o64, nullptr, st);
}

}  // namespace gaca
