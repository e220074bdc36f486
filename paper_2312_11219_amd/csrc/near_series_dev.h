// Which pairs of the near field the power series in the frequency covers (near_moments.hip): the
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

// Two kernels may round a pair's bound differently: the series takes pairs up to kNearSeriesMax, the
// kernels that visit the points at every frequency leave out those safely below it.  What both
// write is the same entry.
constexpr double kSeriesSafe = kNearSeriesMax * (1.0 - 1e-9);

// Argument of the series' bound; the exponentials at r_c and over the span stay far from the ends
// of the range of doubles.
__device__ __forceinline__ double span_bound(const NearSeries &S, double rc, double half) {
    return fmax(S.R * half, (fabs(S.c) + S.R) * rc * (kNearSeriesMax / 600.0));
}

// the pair's span; returns the argument of the series' bound
template <int TIER>
__device__ __forceinline__ double gal_span(const GeoDev &g, const NearSeries &S, int64_t i, int64_t j, double &rc) {
    if (TIER == GT_EDGE || TIER == GT_VERTEX || TIER == GT_COINC) {
        rc = 0.0;
        return fmax(fabs(S.c), S.R) * (TIER == GT_COINC ? g.h[i] : g.h[i] + g.h[j]);
    }
    double half;
    span_of(dist3(g.xx[i], g.xy[i], g.xz[i], g.xx[j], g.xy[j], g.xz[j]), tri_radius(g, i) + tri_radius(g, j), rc, half);
    return span_bound(S, rc, half);
}

__device__ __forceinline__ double near_span(const GeoDev &g, const NearSeries &S, int64_t i, int64_t j, double &rc) {
    double half;
    span_of(i == j ? 0.0 : dist3(g.xx[i], g.xy[i], g.xz[i], g.xx[j], g.xy[j], g.xz[j]), tri_radius(g, j), rc, half);
    return span_bound(S, rc, half);
}

// The distances to a patch reach up to that of its farthest vertex, and down to the vertex j's less
// the patch's longest edge at it.
__device__ __forceinline__ double p1_span(const GeoDev &g, const NearSeries &S, int64_t i, int64_t j, double &rc) {
    const double x = g.xx[i], y = g.xy[i], z = g.xz[i], vx = g.xx[j], vy = g.xy[j], vz = g.xz[j];
    double rad = 0.0, top = 0.0;
    for (int32_t e = g.pptr[j]; e < g.pptr[j + 1]; ++e) {
        const int64_t t = g.ptri[e];
        rad = fmax(rad, fmax(fmax(dist3(vx, vy, vz, g.ax[t], g.ay[t], g.az[t]), dist3(vx, vy, vz, g.bx[t], g.by[t], g.bz[t])),
                             dist3(vx, vy, vz, g.cx[t], g.cy[t], g.cz[t])));
        top = fmax(top, fmax(fmax(dist3(x, y, z, g.ax[t], g.ay[t], g.az[t]), dist3(x, y, z, g.bx[t], g.by[t], g.bz[t])),
                             dist3(x, y, z, g.cx[t], g.cy[t], g.cz[t])));
    }
    const double lo = fmax(dist3(x, y, z, vx, vy, vz) - rad, 0.0);
    rc = 0.5 * (lo + top);
    return span_bound(S, rc, 0.5 * (top - lo));
}

}  // namespace gaca
