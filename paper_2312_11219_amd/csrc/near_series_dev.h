// Which pairs of the near field the Chebyshev series in the distance covers (near_moments.hip): the
// kernels of both kinds decide by the same functions.
#pragma once

#include "entries_dev.h"
#include "galerkin_dev.h"
#include "kernels.h"

namespace gaca {

// r_c and delta of a pair of regular class from the distance of the centres and the radii
__device__ __forceinline__ void span_of(double d, double rad, double &rc, double &half) {
    const double lo = fmax(d - rad, 0.0);
    rc = 0.5 * (lo + d + rad);
    half = 0.5 * (d + rad - lo);
}

__device__ __forceinline__ double tri_radius(const GeoDev &g, int64_t t) {
    const double cx = g.xx[t], cy = g.xy[t], cz = g.xz[t];
    return fmax(fmax(dist3(g.ax[t], g.ay[t], g.az[t], cx, cy, cz), dist3(g.bx[t], g.by[t], g.bz[t], cx, cy, cz)),
                dist3(g.cx[t], g.cy[t], g.cz[t], cx, cy, cz));
}

// The series takes these pairs, the kernels that visit the points at every frequency the others.  Two
// kernels may round a span differently, so the latter (share = 1 - 1e-9) leave out only what is safely
// covered; what both write is the same entry.
__device__ __forceinline__ bool series_covers(const NearSeries &S, double rc, double half, double share = 1.0) {
    return S.K > 0 && half <= S.half * share && rc <= S.rmax * share;
}
constexpr double kSeriesSafe = 1.0 - 1e-9;

// touching pairs: the distances reach from 0 to half
template <int TIER>
__device__ __forceinline__ void gal_span(const GeoDev &g, int64_t i, int64_t j, double &rc, double &half) {
    if (TIER == GT_EDGE || TIER == GT_VERTEX || TIER == GT_COINC) {
        rc = 0.0;
        half = TIER == GT_COINC ? g.h[i] : g.h[i] + g.h[j];
    } else {
        span_of(dist3(g.xx[i], g.xy[i], g.xz[i], g.xx[j], g.xy[j], g.xz[j]), tri_radius(g, i) + tri_radius(g, j), rc,
                half);
    }
}

__device__ __forceinline__ void near_span(const GeoDev &g, int64_t i, int64_t j, double &rc, double &half) {
    span_of(i == j ? 0.0 : dist3(g.xx[i], g.xy[i], g.xz[i], g.xx[j], g.xy[j], g.xz[j]), tri_radius(g, j), rc, half);
}

// The distances to a patch reach up to that of its farthest vertex, and down to the vertex j's less
// the patch's longest edge at it.
__device__ __forceinline__ void p1_span(const GeoDev &g, int64_t i, int64_t j, double &rc, double &half) {
    const double x[3] = {g.xx[i], g.xy[i], g.xz[i]}, v[3] = {g.xx[j], g.xy[j], g.xz[j]};
    double rad2 = 0.0, top2 = 0.0;
    auto sq = [](const double *o, double px, double py, double pz) {
        return (px - o[0]) * (px - o[0]) + (py - o[1]) * (py - o[1]) + (pz - o[2]) * (pz - o[2]);
    };
    for (int32_t e = g.pptr[j]; e < g.pptr[j + 1]; ++e) {
        const int64_t t = g.ptri[e];
        rad2 = fmax(rad2, fmax(fmax(sq(v, g.ax[t], g.ay[t], g.az[t]), sq(v, g.bx[t], g.by[t], g.bz[t])),
                               sq(v, g.cx[t], g.cy[t], g.cz[t])));
        top2 = fmax(top2, fmax(fmax(sq(x, g.ax[t], g.ay[t], g.az[t]), sq(x, g.bx[t], g.by[t], g.bz[t])),
                               sq(x, g.cx[t], g.cy[t], g.cz[t])));
    }
    const double rad = sqrt(rad2), top = sqrt(top2);
    const double lo = fmax(dist3(x[0], x[1], x[2], v[0], v[1], v[2]) - rad, 0.0);
    rc = 0.5 * (lo + top);
    half = 0.5 * (top - lo);
}

}  // namespace gaca
