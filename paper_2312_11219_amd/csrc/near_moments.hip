// Near field of every frequency from moments of the quadrature points.
//
// An entry is sum_q w_q k(r_q) e^{-s r_q} over the points of its rule (double layer: with the factor
// 1 + s r_q).  With the distances in r_c +- delta, delta <= Delta (the class's largest), and the
// frequencies in bands of real parts about real centres c,
//   e^{-s r} = e^{-s r_c} e^{-c (r - r_c)} sum_k a_k(s) T_k(x),  x = (r - r_c) / Delta,
// the Chebyshev series of e^{-z x}, z = (s - c) Delta (a_k: modified Bessel functions of z), cut where
// the rest is below the rounding of the sum (near_series.cpp: 16 terms for |z| <= 1.1, 20 for 2.2, 24 for
// 3.7, 30 for 6.2).  The points are visited once per band, for
//   M_k = sum_q w_q k(r_q) e^{-c (r_q - r_c)} T_k(x_q)
// and, in the double layer, the same with another factor r_q; a frequency then costs one real times
// complex product a term.  Touching and coincident Galerkin pairs carry exact radial integrals phi(s rho),
// which fall off as powers only: the Chebyshev series of phi(s rho) on 0 <= rho <= Delta, one band, no
// exponential.
//
// Rounding: sum |a_k| is the few that it is for imaginary z, times up to e^{|Re z|}, so the bands keep
// |Re z| <= 1.25, and <= 2 for the 6-point rules of distant pairs (whose own rounding, of s r at every
// point, is larger).  s r_c is formed with its remainder, and the two parts of the double layer have
// positive weights.  Against 80-bit arithmetic on random pairs, R Delta up to 6 (R: radius of the
// frequencies), largest error of an entry relative to it, in brackets point by point: 6 points, far 4.2e-15
// (1.4e-14); 16 points 1.8e-15 (6.7e-15); 64 points, close 1.7e-15 (1.5e-15); touching pairs up to
// |s| rho = 12 5.5e-15 (5.5e-15).  One power series in s - c for all frequencies, whose terms
// exceed its sum by up to e^{2 R delta}, had 4e-13.
//
// What bounds it: the moments' multiply-adds (FP64 VALU, two or three per moment, point and band) where a
// rule has many points, the writes of the entries and the steps per frequency where it has few.  G lanes
// share a pair and band, first its points, then its frequencies.  Near field of a build beside the far
// field, every point at every frequency -> moments: Galerkin P0 (3072-triangle L-shape, L = 96) 82 -> 11 ms;
// P1 double layer (4802-vertex sphere, L = 128) 49 -> 8.1 ms; collocation (9408-triangle sphere, L = 128)
// 17.5 -> 10.8 ms, of which the writes of its 18 GB take 4.  (The power series took 6.1, 6.2 and 10.7.)
// Pairs beyond the bound (few elements per wavelength) are left to the kernels that visit the points at
// every frequency.
#include <hip/hip_runtime.h>

#include "device_util.h"
#include "entries_dev.h"
#include "galerkin_dev.h"
#include "kernels.h"
#include "near_series_dev.h"

namespace gaca {

namespace {

// sum over G adjacent lanes (a power of two up to 16), in every one of them
template <int G>
__device__ __forceinline__ double group_sum(double v) {
    if (G > 1) v += dpp_d<0xB1>(v);
    if (G > 2) v += dpp_d<0x4E>(v);
    if (G > 4) v += dpp_d<0x141>(v);
    if (G > 8) v += dpp_d<0x140>(v);
    return v;
}

// M_k and, with D, the same weighted by r
template <int K, bool D>
struct Moments {
    double m[K], n[D ? K : 1];
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            m[k] = 0.0;
            if (D) n[k] = 0.0;
        }
    }
    __device__ __forceinline__ void add(double x, double r, double w) {
        const double x2 = 2.0 * x;
        double t0 = w, t1 = w * x;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            m[k] += t0;
            if (D) n[k] = fma(r, t0, n[k]);
            const double t2 = fma(x2, t1, -t0);
            t0 = t1;
            t1 = t2;
        }
    }
    // the lanes' sums together
    template <int G>
    __device__ __forceinline__ void finish() {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            m[k] = group_sum<G>(m[k]);
            if (D) {
                n[k] = group_sum<G>(n[k]);
                asm volatile("" : "+v"(m[k]), "+v"(n[k]));   // one after the other (registers)
            }
        }
    }
    // sum_k a_k M_k (+ s sum_k a_k N_k), the terms at a[k step].  ONE: every lane of the wave takes this
    // frequency, and the table is read as constant memory, by scalar loads
    template <bool ONE>
    __device__ __forceinline__ double2 eval(const double2 *a, int step, double sr, double si) const {
        const auto *ac = (const __attribute__((address_space(4))) double *)a;
        double pr = 0.0, pi = 0.0, nr = 0.0, ni = 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const double cr = ONE ? ac[2 * k * step] : a[k * step].x, ci = ONE ? ac[2 * k * step + 1] : a[k * step].y;
            pr = fma(cr, m[k], pr);
            pi = fma(ci, m[k], pi);
            if (D) {
                nr = fma(cr, n[k], nr);
                ni = fma(ci, n[k], ni);
            }
            // six terms in flight: more cost registers, of which the double layer has none left.  (The single
            // layer runs with two waves per SIMD; with three it holds up the far field beside it: Galerkin
            // 3072-triangle build 28.1 ms for 27.1.)
            if (ONE && k % 6 == 5) __builtin_amdgcn_sched_barrier(0);
            if (D && !ONE && k % 6 == 5) asm volatile("" : "+v"(pr), "+v"(pi), "+v"(nr), "+v"(ni) : : "memory");
        }
        if (D) {
            pr += sr * nr - si * ni;
            pi += sr * ni + si * nr;
        }
        return make_double2(pr, pi);
    }
};

// the band's centre and the pair's middle distance; 1 / Delta (touching pairs: 2 / Delta)
struct Span {
    double c, rc, scale;
};

template <int K, bool D>
__device__ __forceinline__ void add_point(Moments<K, D> &M, const Span &S, double r, double ir, double w) {
    const double dr = r - S.rc;
    M.add(dr * S.scale, r, w * kInvFourPi * (D ? ir * ir * ir : ir) * fm::exp(-S.c * dr));
}

// points sub, sub + G, ... of the collapsed n x n rule on (a, b, c) seen from x; lam < 0, or the
// barycentric coordinate that weighs them
template <int G, int K, bool D>
__device__ __forceinline__ void add_collapsed(Moments<K, D> &M, const Span &S, const double *x, const double *a,
                                              const double *b, const double *c, int n, const double *gt,
                                              double wscale, int sub, int lam = -1) {
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
        add_point(M, S, r, ir, w);
    }
}

// w / (4 pi rho) at the end of the radial integral along d
template <int K>
__device__ __forceinline__ void add_radial(Moments<K, false> &M, const Span &S, const double *d, double w) {
    const double rho = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
    M.add(fma(rho, S.scale, -1.0), 0.0, w / (kFourPi * rho));
}

template <int TIER, int G, int K>
__device__ __forceinline__ void gal_moments(Moments<K, false> &M, const GeoDev &g, const QuadDev &q, const Span &S,
                                            int64_t i, int64_t j, int sub) {
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
            add_point(M, S, r, ir, g.q6w[pi * T + i] * g.q6w[pj * T + j]);
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
                add_collapsed<1>(M, S, x, aj, bj, cj, q.n4, q.g4, wx, 0);
            } else {
                double p[3];
                closest_on_triangle(x, aj, bj, cj, p);
                const double *V1 = s == 0 ? bj : (s == 1 ? cj : aj), *V2 = s == 0 ? cj : (s == 1 ? aj : bj);
                const double p1[3] = {V1[0], V1[1], V1[2]}, p2[3] = {V2[0], V2[1], V2[2]};
                add_collapsed<1>(M, S, x, p, p1, p2, q.ng, q.gg, wx, 0);
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
                M.add(fma(R, S.scale, -1.0), 0.0, 0.5 * A2 / kFourPi * span * q.gth[2 * p + 1] * R);
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
                    add_radial(M, S, d, r == 0 ? w : w * e2);
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
                    add_radial(M, S, d, w);
#pragma unroll
                    for (int k = 0; k < 3; ++k) d[k] = e2 * (X1[k] + e3 * X2[k]) - (Y1[k] + e1 * Y2[k]);
                    add_radial(M, S, d, w);
                }
            }
        }
    }
}

// the entry at the frequencies sub, sub + G, ... of band b (RADIAL: no factor e^{-s r_c})
template <bool RADIAL, int G, int K, bool D>
__device__ __forceinline__ void write_entry(const Moments<K, D> &M, const NearSeries &S, const FreqDev &f, int b,
                                            double rc, double num, int sub, int64_t base, int n, double2 *out64,
                                            float2 *out32) {
    for (int p = S.first[b] + sub; p < S.first[b + 1]; p += G) {
        const int l = S.order[p];
        const double sr = f.re[l], si = f.im[l];
        const double2 P = G == 1 ? M.template eval<true>(S.by_freq + (int64_t)p * K, 1, sr, si)
                                 : M.template eval<false>(S.by_term + p, f.L_eval, sr, si);
        double vr = P.x, vi = P.y;
        if (!RADIAL) {
            // e^{-s r_c}, the products with r_c corrected by what their rounding leaves
            const double hr = sr * rc, hi = si * rc;
            const double mag = fm::exp(-hr) * (1.0 - fma(sr, rc, -hr)), lo = fma(si, rc, -hi);
            double sn, cs;
            fm::sincos(hi, &sn, &cs);
            const double er = num * mag * fma(-sn, lo, cs), ei = -num * mag * fma(cs, lo, sn);
            vr = er * P.x - ei * P.y;
            vi = er * P.y + ei * P.x;
        }
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

// WHAT: Galerkin class (GAL), collocation tier, or the P1 double layer.  blockIdx.y: band
enum { GAL = 0, COL = 1, P1 = 2 };
template <int WHAT, int KERNEL, int TIER, int K, int G>
__global__ void __launch_bounds__(256, 2)
    near_series_kernel(GeoDev g, QuadDev q, FreqDev f, NearSeries S, const NearPair *__restrict__ pairs,
                       int64_t npairs, const NearBlockDev *__restrict__ blocks, double2 *out64, float2 *out32) {
    constexpr bool RADIAL = WHAT == GAL && TIER >= GT_EDGE;
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x, p = t / G;
    const int sub = (int)(t % G);
    if (p >= npairs) return;   // the G lanes of a pair together
    const NearPair pr = pairs[p];
    const NearBlockDev B = blocks[pr.blk];
    const int64_t i = B.r0 + pr.i, j = B.c0 + pr.j, base = B.off + (int64_t)pr.i * f.L * B.n + pr.j;
    double rc, half, num = 1.0;
    if constexpr (WHAT == GAL) gal_span<TIER>(g, i, j, rc, half);
    else if constexpr (WHAT == COL) near_span(g, i, j, rc, half);
    else p1_span(g, i, j, rc, half);
    if (!series_covers(S, rc, half)) return;
    const double x[3] = {g.xx[i], g.xy[i], g.xz[i]};
    if (WHAT == COL && KERNEL == 1) num = g.nx[j] * x[0] + g.ny[j] * x[1] + g.nz[j] * x[2] - g.d[j];
    const int b = blockIdx.y;
    const Span sp{S.c[b], rc, (RADIAL ? 2.0 : 1.0) / S.half};
    Moments<K, KERNEL == 1> M;
    M.zero();
    if constexpr (WHAT == GAL) {
        gal_moments<TIER, G>(M, g, q, sp, i, j, sub);
    } else if constexpr (WHAT == COL) {
        const double a[3] = {g.ax[j], g.ay[j], g.az[j]}, b3[3] = {g.bx[j], g.by[j], g.bz[j]},
                     c[3] = {g.cx[j], g.cy[j], g.cz[j]};
        if constexpr (TIER == TIER_FAR6) {
            const int64_t T = g.M;
            for (int k = sub; k < 6; k += G) {
                double ir;
                const double r = dist3_inv(x[0], x[1], x[2], g.q6x[k * T + j], g.q6y[k * T + j], g.q6z[k * T + j], ir);
                add_point(M, sp, r, ir, g.q6w[k * T + j]);
            }
        } else if constexpr (TIER == TIER_SELF) {
            for (int e = 0; e < 3; ++e) {
                const double *p1 = e == 0 ? b3 : (e == 1 ? c : a), *p2 = e == 0 ? c : (e == 1 ? a : b3);
                const double v1[3] = {p1[0], p1[1], p1[2]}, v2[3] = {p2[0], p2[1], p2[2]};
                add_collapsed<G>(M, sp, x, x, v1, v2, q.nd, q.gd, 1.0, sub);
            }
        } else {
            add_collapsed<G>(M, sp, x, a, b3, c, TIER == TIER_MID4 ? q.n4 : q.n8, TIER == TIER_MID4 ? q.g4 : q.g8,
                             1.0, sub);
        }
    } else {
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
                    add_point(M, sp, r, ir, nt * g.q6wl[(int64_t)(loc * 6 + k) * T + tr]);
                }
            } else {
                const double a[3] = {g.ax[tr], g.ay[tr], g.az[tr]}, b3[3] = {g.bx[tr], g.by[tr], g.bz[tr]},
                             c[3] = {g.cx[tr], g.cy[tr], g.cz[tr]};
                add_collapsed<G>(M, sp, x, a, b3, c, qd >= 2.0 ? q.n4 : q.n8, qd >= 2.0 ? q.g4 : q.g8, nt, sub, loc);
            }
        }
    }
    M.template finish<G>();
    write_entry<RADIAL, G>(M, S, f, b, rc, num, sub, base, B.n, out64, out32);
}

template <int WHAT, int KERNEL, int TIER, int G>
void launch(const GeoDev &g, const QuadDev &q, const FreqDev &f, const NearSeries &S, const NearPair *pairs,
            int64_t npairs, const NearBlockDev *blocks, double2 *o64, float2 *o32, hipStream_t st) {
    // a grid holds fewer than 2^32 threads: G lanes a pair for at most 2^27 pairs
    constexpr int64_t kPairs = (int64_t)1 << 27;
    static_assert(kPairs * 16 < ((int64_t)1 << 32) && G <= 16, "threads of a launch");
    for (; npairs > 0; pairs += kPairs, npairs -= kPairs) {
        const int64_t n = npairs < kPairs ? npairs : kPairs;
        const dim3 nb((unsigned)((n * G + 255) / 256), S.nband);
#define GACA_SERIES(K) \
    near_series_kernel<WHAT, KERNEL, TIER, K, G><<<nb, 256, 0, st>>>(g, q, f, S, pairs, n, blocks, o64, o32)
        if (S.K == 16) GACA_SERIES(16);
        else if (S.K == 20) GACA_SERIES(20);
        else if (S.K == 24) GACA_SERIES(24);
        else GACA_SERIES(30);
#undef GACA_SERIES
    }
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

void launch_near_series_p1(int tier, const GeoDev &g, const QuadDev &q, const FreqDev &f, const NearSeries &S,
                           const NearPair *pairs, int64_t npairs, const NearBlockDev *blocks, double2 *o64,
                           hipStream_t st) {
    if (npairs <= 0) return;
    // one lane where a pair has six points a triangle (the sums over lanes would cost more than the points)
    if (tier == 0) launch<P1, 1, 0, 1>(g, q, f, S, pairs, npairs, blocks, o64, nullptr, st);
    else launch<P1, 1, 0, 4>(g, q, f, S, pairs, npairs, blocks, o64, nullptr, st);
}

}  // namespace gaca
