// Near field of the Galerkin P1 operators (hypersingular D, adjoint double layer K'), assembled by
// triangle pairs: the local integrals
//   M_ab = int int k(x, y) l_a(x) l_b(y),  a, b = 0, 1, 2,  S = int int k = sum_ab M_ab
// of every pair of triangles that a near entry needs are computed once, and an entry is then the
// sum over the pairs of its two patches.  (One thread per entry evaluated each pair for all nine
// vertex pairs that share it, with thousands of points in a row per thread where the triangles
// touch: 768-triangle cube, D, L = 8, 6 points a direction, 617 ms; 4.9 ms by pairs.)
//
// What bounds it: the kernel evaluations (FP64 VALU).  The rules and the classes are those of
// gp1_pair; the split follows the number of points of a class:
//   6 x 6 points       one lane per pair
//   collapsed (mid)    16 lanes per pair, each the inner rule of its outer points
//   disjoint, q < 2    one wave per pair over all points; closest points and weights of the outer
//                      points once per pair, through LDS
//   touching           one wave per pair over the n^4 points, all regions per point
// Every lane takes NF frequencies per point (the distance and the weights are shared).  Sums over
// lanes are in a fixed order.  The pair buffer (up to 512 MiB) holds a chunk of frequencies at a time, and
// on larger meshes a chunk of the rows ti, whose part of every entry is added in turn.
#include <hip/hip_runtime.h>

#include "device_util.h"
#include "entries_dev.h"
#include "galerkin_p1_dev.h"
#include "kernels.h"

namespace gaca {

namespace {

constexpr int NF = 2;   // frequencies per lane: 36 sums and the point data stay in registers

// distance, its inverse and the numerator of the kernel at x - y
template <int OP>
__device__ __forceinline__ void pair_point(const double *x, const double *y, const double *nx, double &r,
                                           double &ir, double &num) {
    const double dx = x[0] - y[0], dy = x[1] - y[1], dz = x[2] - y[2];
    const double d = dx * dx + dy * dy + dz * dz;
    double t = __builtin_amdgcn_rsq(d);
#pragma unroll
    for (int it = 0; it < 2; ++it) t = fma(0.5 * t, fma(-d * t, t, 1.0), t);
    ir = t;
    r = d * t;
    num = OP == 1 ? -(dx * nx[0] + dy * nx[1] + dz * nx[2]) : 1.0;
}

struct Local {   // M_ab of NF frequencies
    double r[NF][9], i[NF][9];
    __device__ void zero() {
#pragma unroll
        for (int k = 0; k < NF; ++k)
#pragma unroll
            for (int t = 0; t < 9; ++t) r[k][t] = i[k][t] = 0.0;
    }
};

// += w k(x, y) la_a lb_b
template <int OP>
__device__ __forceinline__ void add_point(const double *x, const double *la, const double *y, const double *lb,
                                          double w, const double *nx, const FreqDev &f, int l0, int nl, Local &M) {
    double r, ir, num;
    pair_point<OP>(x, y, nx, r, ir, num);
    double wl[9];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double wa = w * num * la[a];
#pragma unroll
        for (int b = 0; b < 3; ++b) wl[3 * a + b] = wa * lb[b];
    }
#pragma unroll
    for (int k = 0; k < NF; ++k)
        if (k < nl) {
            double gr, gi;
            gp1_kval<OP>(r, ir, f.re[l0 + k], f.im[l0 + k], gr, gi);
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                M.r[k][t] += wl[t] * gr;
                M.i[k][t] += wl[t] * gi;
            }
        }
}

// sums over the inner rule of one outer point: += w k(x, y) lb_b
template <int OP>
__device__ __forceinline__ void add_inner(const double *x, const double *y, const double *wb, const double *nx,
                                          const FreqDev &f, int l0, int nl, double (&sr)[NF][3], double (&si)[NF][3]) {
    double r, ir, num;
    pair_point<OP>(x, y, nx, r, ir, num);
#pragma unroll
    for (int k = 0; k < NF; ++k)
        if (k < nl) {
            double gr, gi;
            gp1_kval<OP>(r, ir, f.re[l0 + k], f.im[l0 + k], gr, gi);
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                sr[k][b] += wb[b] * num * gr;
                si[k][b] += wb[b] * num * gi;
            }
        }
}

__device__ __forceinline__ void fold_outer(const double *wa, double (&sr)[NF][3], double (&si)[NF][3], Local &M) {
#pragma unroll
    for (int k = 0; k < NF; ++k)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                M.r[k][3 * a + b] += wa[a] * sr[k][b];
                M.i[k][3 * a + b] += wa[a] * si[k][b];
            }
            sr[k][b] = si[k][b] = 0.0;
        }
}

// sum over 2^LG adjacent lanes (up to a row of 16, or the wave), in every one of them
template <int LG>
__device__ __forceinline__ double lanes_sum(double v) {
    if constexpr (LG == 6) return wave_sum(v);
    if constexpr (LG > 0) v += dpp_d<0xB1>(v);
    if constexpr (LG > 1) v += dpp_d<0x4E>(v);
    if constexpr (LG > 2) v += dpp_d<0x141>(v);
    if constexpr (LG > 3) v += dpp_d<0x140>(v);
    return v;
}

// The pair's slot [frequency of the chunk][10]: M_ab (original local vertices), then S
template <int LG>
__device__ __forceinline__ void store_local(Local &M, bool first, int nl, const int *pa, const int *pb, double2 *slot) {
#pragma unroll
    for (int k = 0; k < NF; ++k) {
        double sr = 0.0, si = 0.0;
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            M.r[k][t] = lanes_sum<LG>(M.r[k][t]);
            M.i[k][t] = lanes_sum<LG>(M.i[k][t]);
            sr += M.r[k][t];
            si += M.i[k][t];
        }
        if (first && k < nl) {
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int b = 0; b < 3; ++b)
                    slot[10 * k + 3 * pa[a] + pb[b]] = make_double2(M.r[k][3 * a + b], M.i[k][3 * a + b]);
            slot[10 * k + 9] = make_double2(sr, si);
        }
    }
}

// the dG/dn_x integrand of a coplanar pair is 0 (as gp1_pair)
__device__ __forceinline__ bool coplanar(const GP1Tri &Ti, const GP1Tri &Tj) {
    for (int c = 0; c < 3; ++c) {
        const double dd = (Tj.v[c][0] - Ti.v[0][0]) * Ti.n[0] + (Tj.v[c][1] - Ti.v[0][1]) * Ti.n[1] +
                          (Tj.v[c][2] - Ti.v[0][2]) * Ti.n[2];
        if (fabs(dd) > 1e-14 * Ti.h) return false;
    }
    return true;
}

struct PairArgs {
    GeoDev g;
    QuadDev q;
    FreqDev f;
    const int2 *pairs;       // (ti, tj) of every pair
    const int32_t *list;     // the pairs of the class
    int64_t cnt;
    int l0, nfc;             // chunk of frequencies [l0, l0 + nfc)
    int64_t p0;              // first pair of the buffer
    double2 *buf;            // [pair - p0][nfc][10]
};

}  // namespace

__device__ __forceinline__ int gp1_class(const GeoDev &g, int ti, int tj) {
    const int32_t vi[3] = {g.tv0[ti], g.tv1[ti], g.tv2[ti]}, vj[3] = {g.tv0[tj], g.tv1[tj], g.tv2[tj]};
    int shared = 0;
    for (int x = 0; x < 3; ++x)
        for (int y = 0; y < 3; ++y) shared += vi[x] == vj[y];
    if (shared > 0) return GP1_VERTEX + shared - 1;
    GP1Tri Ti, Tj;
    gp1_load(g, ti, Ti);
    gp1_load(g, tj, Tj);
    const double dcx = Ti.c[0] - Tj.c[0], dcy = Ti.c[1] - Tj.c[1], dcz = Ti.c[2] - Tj.c[2];
    const double qd = sqrt(dcx * dcx + dcy * dcy + dcz * dcz) / fmax(Ti.h, Tj.h);
    return qd >= 4.0 ? GP1_FAR : qd >= 2.0 ? GP1_MID : GP1_NEAR;
}

// the chunk of row ti: the last with chunk_of[c] <= ti
__device__ __forceinline__ int gp1_chunk(const int32_t *chunk_of, int nchunk, int ti) {
    int lo = 0, hi = nchunk - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (chunk_of[mid] <= ti) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

__global__ void __launch_bounds__(256) gp1_zero_kernel(unsigned long long *v, int n) {
    for (int i = threadIdx.x; i < n; i += 256) v[i] = 0;
}

// one wave per row: a lane ORs a word of the row's sets and writes its bits after those of the lanes below
__global__ void __launch_bounds__(256)
    gp1_fill_kernel(GeoDev g, const uint64_t *sets, int words, const int32_t *rowsetptr, const int32_t *rowset,
                    const int64_t *rowptr, int64_t T, const int32_t *chunk_of, int nchunk, int2 *pairs, uint8_t *cls,
                    unsigned long long *count) {
    const int64_t ti = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (ti >= T) return;   // the whole wave; no barrier below
    int64_t at = rowptr[ti];
    int n[kGp1Classes] = {0, 0, 0, 0, 0, 0};
    for (int w0 = 0; w0 < words; w0 += 64) {
        const int w = w0 + lane;
        uint64_t bits = 0;
        if (w < words)
            for (int s = rowsetptr[ti]; s < rowsetptr[ti + 1]; ++s) bits |= sets[(int64_t)rowset[s] * words + w];
        int before = __popcll(bits);   // inclusive prefix sum
        for (int d = 1; d < 64; d <<= 1) {
            const int v = __shfl_up(before, d, 64);
            if (lane >= d) before += v;
        }
        int64_t p = at + before - __popcll(bits);
        at += __shfl(before, 63, 64);
        while (bits) {
            const int tj = 64 * w + __ffsll((unsigned long long)bits) - 1;
            bits &= bits - 1;
            const int c = gp1_class(g, (int)ti, tj);
            pairs[p] = make_int2((int)ti, tj);
            cls[p++] = (uint8_t)c;
#pragma unroll
            for (int k = 0; k < kGp1Classes; ++k) n[k] += c == k;
        }
    }
    const int ch = gp1_chunk(chunk_of, nchunk, (int)ti);
#pragma unroll
    for (int k = 0; k < kGp1Classes; ++k) {
        int s = n[k];
        for (int d = 32; d > 0; d >>= 1) s += __shfl_down(s, d, 64);
        if (lane == 0 && s > 0) atomicAdd(&count[ch * kGp1Classes + k], (unsigned long long)s);
    }
}

// The order within a class is that of the waves' arrival: a pair's integrals have their own place.
__global__ void __launch_bounds__(256)
    gp1_list_kernel(const int2 *pairs, const uint8_t *cls, int64_t np, const int32_t *chunk_of, int nchunk,
                    unsigned long long *next, int32_t *list) {
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int lane = threadIdx.x & 63;
    int key = -1;
    if (p < np) key = gp1_chunk(chunk_of, nchunk, pairs[p].x) * kGp1Classes + cls[p];
    // one place for all lanes of the wave with the same key
    unsigned long long left = __ballot(key >= 0);
    while (left) {
        const int k = __builtin_amdgcn_readlane(key, __ffsll(left) - 1);
        const unsigned long long same = __ballot(key == k);
        left &= ~same;
        if (key == k) {
            const int leader = __ffsll(same) - 1;
            unsigned long long base = 0;
            if (lane == leader) base = atomicAdd(&next[k], (unsigned long long)__popcll(same));
            base = __shfl(base, leader, 64);
            list[base + __popcll(same & ((1ull << lane) - 1))] = (int32_t)p;
        }
    }
}

// 6 x 6 points, one lane per pair; collapsed n4 x n4 on both, 16 lanes per pair
template <int OP, bool MID>
__global__ void __launch_bounds__(256) gp1_product_kernel(PairArgs A) {
    constexpr int LG = MID ? 4 : 0;
    const int64_t t = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> LG;
    const int sub = threadIdx.x & ((1 << LG) - 1);
    const int k0 = blockIdx.y * NF, l0 = A.l0 + k0, nl = min(NF, A.nfc - k0);
    const bool on = t < A.cnt;
    const int p = A.list[on ? t : 0];
    const int ti = A.pairs[p].x, tj = A.pairs[p].y;
    const GeoDev &g = A.g;
    GP1Tri Ti, Tj;
    gp1_load(g, ti, Ti);
    gp1_load(g, tj, Tj);
    Local M;
    M.zero();
    if (!(OP == 1 && coplanar(Ti, Tj))) {
        double sr[NF][3] = {}, si[NF][3] = {};
        if constexpr (!MID) {
            const int64_t T = g.T;
            for (int a = 0; a < 6; ++a) {
                const double x[3] = {g.q6x[a * T + ti], g.q6y[a * T + ti], g.q6z[a * T + ti]};
                for (int b = 0; b < 6; ++b) {
                    const double y[3] = {g.q6x[b * T + tj], g.q6y[b * T + tj], g.q6z[b * T + tj]};
                    const double wb[3] = {g.q6wl[b * T + tj], g.q6wl[(6 + b) * T + tj], g.q6wl[(12 + b) * T + tj]};
                    add_inner<OP>(x, y, wb, Ti.n, A.f, l0, nl, sr, si);
                }
                const double wa[3] = {g.q6wl[a * T + ti], g.q6wl[(6 + a) * T + ti], g.q6wl[(12 + a) * T + ti]};
                fold_outer(wa, sr, si, M);
            }
        } else {
            const int n = A.q.n4;
            const double *gt = A.q.g4;
            for (int a = sub; a < n * n; a += 16) {
                const int iu = a / n, iv = a - iu * n;
                const double u = gt[2 * iu], v = gt[2 * iv];
                double x[3], wx;
                gp1_collapsed_pt(Ti.v[0], Ti.v[1], Ti.v[2], u, v, gt[2 * iu + 1] * gt[2 * iv + 1], x, wx);
                for (int ju = 0; ju < n; ++ju)
                    for (int jv = 0; jv < n; ++jv) {
                        const double u2 = gt[2 * ju], v2 = gt[2 * jv];
                        double y[3], wy;
                        gp1_collapsed_pt(Tj.v[0], Tj.v[1], Tj.v[2], u2, v2, gt[2 * ju + 1] * gt[2 * jv + 1], y, wy);
                        const double wb[3] = {wy * (1.0 - u2), wy * (u2 - u2 * v2), wy * (u2 * v2)};
                        add_inner<OP>(x, y, wb, Ti.n, A.f, l0, nl, sr, si);
                    }
                const double wa[3] = {wx * (1.0 - u), wx * (u - u * v), wx * (u * v)};
                fold_outer(wa, sr, si, M);
            }
        }
    }
    const int id[3] = {0, 1, 2};
    store_local<LG>(M, on && sub == 0, nl, id, id, A.buf + ((p - A.p0) * A.nfc + k0) * 10);
}

// disjoint pairs with q < 2: outer collapsed n x n on ti, inner rule split at the closest point
template <int OP>
__global__ void __launch_bounds__(64) gp1_near_kernel(PairArgs A) {
    constexpr int PC = 32;   // outer points per pass
    const int lane = threadIdx.x, p = A.list[blockIdx.x];
    const int k0 = blockIdx.y * NF, l0 = A.l0 + k0, nl = min(NF, A.nfc - k0);
    __shared__ double xs[PC][3], la[PC][3], cp[PC][3], lc[PC][3], wp[PC][3];   // point, w l_a, closest point, its l_b, weights of the pieces
    GP1Tri Ti, Tj;
    gp1_load(A.g, A.pairs[p].x, Ti);
    gp1_load(A.g, A.pairs[p].y, Tj);
    Local M;
    M.zero();
    const int n = A.q.ng, nn = n * n;
    const double *gt = A.q.gg;
    if (!(OP == 1 && coplanar(Ti, Tj)))
        for (int a0 = 0; a0 < nn; a0 += PC) {
            const int na = min(PC, nn - a0);
            __syncthreads();
            if (lane < na) {
                const int a = a0 + lane, iu = a / n, iv = a - iu * n;
                const double u = gt[2 * iu], v = gt[2 * iv];
                double x[3], wx, c[3];
                gp1_collapsed_pt(Ti.v[0], Ti.v[1], Ti.v[2], u, v, gt[2 * iu + 1] * gt[2 * iv + 1], x, wx);
                gp1_closest(x, Tj.v[0], Tj.v[1], Tj.v[2], c);
                la[lane][0] = wx * (1.0 - u);
                la[lane][1] = wx * (u - u * v);
                la[lane][2] = wx * (u * v);
                for (int k = 0; k < 3; ++k) {
                    xs[lane][k] = x[k];
                    cp[lane][k] = c[k];
                    lc[lane][k] = gp1_bary(Tj, c, k);
                    double y[3];
                    gp1_collapsed_pt(c, Tj.v[(k + 1) % 3], Tj.v[(k + 2) % 3], 1.0, 0.0, 1.0, y, wp[lane][k]);
                }
            }
            __syncthreads();
            for (int t = lane; t < na * 3 * nn; t += 64) {
                const int a = t / (3 * nn), rest = t - a * 3 * nn, piece = rest / nn, e = rest - piece * nn;
                const int ju = e / n, jv = e - ju * n;
                const double u = gt[2 * ju], uv = u * gt[2 * jv];
                const double w = gt[2 * ju + 1] * gt[2 * jv + 1] * u * wp[a][piece];
                // y = c + u (b - c) + u v (d - b), b and d the piece's other corners
                const int ib = piece == 2 ? 0 : piece + 1, id = ib == 2 ? 0 : ib + 1;
                double x[3], y[3], lb[3], lx[3];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    x[k] = xs[a][k];
                    lx[k] = la[a][k];
                    const double vb = ib == 0 ? Tj.v[0][k] : ib == 1 ? Tj.v[1][k] : Tj.v[2][k];
                    const double vd = id == 0 ? Tj.v[0][k] : id == 1 ? Tj.v[1][k] : Tj.v[2][k];
                    const double c = cp[a][k];
                    y[k] = c + u * (vb - c) + uv * (vd - vb);
                    lb[k] = (1.0 - u) * lc[a][k] + (k == ib ? u - uv : k == id ? uv : 0.0);
                }
                add_point<OP>(x, lx, y, lb, w, Ti.n, A.f, l0, nl, M);
            }
        }
    const int id[3] = {0, 1, 2};
    store_local<6>(M, lane == 0, nl, id, id, A.buf + ((p - A.p0) * A.nfc + k0) * 10);
}

// touching pairs (REL shared vertices) by the regularising maps
template <int OP, int REL>
__global__ void __launch_bounds__(64) gp1_touch_kernel(PairArgs A) {
    constexpr int NREG = REL == 3 ? 6 : REL == 2 ? 5 : 2;
    const int lane = threadIdx.x, p = A.list[blockIdx.x];
    const int k0 = blockIdx.y * NF, l0 = A.l0 + k0, nl = min(NF, A.nfc - k0);
    const int ti = A.pairs[p].x, tj = A.pairs[p].y;
    const GeoDev &g = A.g;
    GP1Tri Ti, Tj;
    gp1_load(g, ti, Ti);
    gp1_load(g, tj, Tj);
    const int32_t vi[3] = {g.tv0[ti], g.tv1[ti], g.tv2[ti]}, vj[3] = {g.tv0[tj], g.tv1[tj], g.tv2[tj]};
    // reordered vertices, as gp1_pair: the shared ones first, in ti's order
    int pa[3] = {0, 1, 2}, pb[3] = {0, 1, 2};
    if (REL < 3) {
        int shared = 0, si[2] = {0, 0}, sj[2] = {0, 0};
        for (int x = 0; x < 3; ++x)
            for (int y = 0; y < 3; ++y)
                if (vi[x] == vj[y] && shared < 2) {
                    if (shared == 0) {
                        si[0] = x;
                        sj[0] = y;
                    } else {
                        si[1] = x;
                        sj[1] = y;
                    }
                    ++shared;
                }
        if (REL == 2) {   // found in ti's order already
            pa[0] = si[0]; pa[1] = si[1]; pa[2] = 3 - si[0] - si[1];
            pb[0] = sj[0]; pb[1] = sj[1]; pb[2] = 3 - sj[0] - sj[1];
        } else {
            for (int c = 0; c < 3; ++c) {
                pa[c] = (si[0] + c) % 3;
                pb[c] = (sj[0] + c) % 3;
            }
        }
    }
    double P[3][3], Q[3][3];
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            P[c][k] = pa[c] == 0 ? Ti.v[0][k] : pa[c] == 1 ? Ti.v[1][k] : Ti.v[2][k];
            Q[c][k] = pb[c] == 0 ? Tj.v[0][k] : pb[c] == 1 ? Tj.v[1][k] : Tj.v[2][k];
        }
#pragma unroll
    for (int k = 0; k < 3; ++k) {   // edge vectors P1 - P0, P2 - P1
        P[2][k] -= P[1][k];
        P[1][k] -= P[0][k];
        Q[2][k] -= Q[1][k];
        Q[1][k] -= Q[0][k];
    }
    Local M;
    M.zero();
    const double jij = 4.0 * Ti.area * Tj.area;
    const int n = A.q.ns, n4 = n * n * n * n;
    const double *gs = A.q.gs;
    if (!(OP == 1 && coplanar(Ti, Tj)))
        for (int t = lane; t < n4; t += 64) {
            const int t3 = t / n, i4 = t - t3 * n, t2 = t3 / n, i3 = t3 - t2 * n, i1 = t2 / n, i2 = t2 - i1 * n;
            const double xi = gs[2 * i1], e1 = gs[2 * i2], e2 = gs[2 * i3], e3 = gs[2 * i4];
            const double w0 = gs[2 * i1 + 1] * gs[2 * i2 + 1] * gs[2 * i3 + 1] * gs[2 * i4 + 1] * jij;
#pragma unroll 1
            for (int r = 0; r < NREG; ++r) {
                double X[2], Y[2], jac, x[3], y[3];
                gp1_ss_region(REL, r, xi, e1, e2, e3, X, Y, jac);
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    x[k] = P[0][k] + X[0] * P[1][k] + X[1] * P[2][k];
                    y[k] = Q[0][k] + Y[0] * Q[1][k] + Y[1] * Q[2][k];
                }
                const double lx[3] = {1.0 - X[0], X[0] - X[1], X[1]}, ly[3] = {1.0 - Y[0], Y[0] - Y[1], Y[1]};
                add_point<OP>(x, lx, y, ly, w0 * jac, Ti.n, A.f, l0, nl, M);
            }
        }
    store_local<6>(M, lane == 0, nl, pa, pb, A.buf + ((p - A.p0) * A.nfc + k0) * 10);
}

// The part of the rows [t0, t1) in the entries of the chunk's frequencies, from the pair integrals: one
// thread per (vertex pair, frequency).  The first chunk of rows (t0 = 0) sets the entries, others add.
template <int OP>
__global__ void __launch_bounds__(256)
    gp1_assemble_kernel(GeoDev g, FreqDev f, const NearPair *__restrict__ vp, int64_t nvp,
                        const NearBlockDev *__restrict__ blocks, const int64_t *__restrict__ rowptr,
                        const int2 *__restrict__ pairs, const double2 *__restrict__ buf, int l0, int nfc, int t0,
                        int t1, int64_t p0, double2 *out64) {
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= nvp) return;
    const int k = blockIdx.y, l = l0 + k;
    const NearPair pr = vp[p];
    const NearBlockDev B = blocks[pr.blk];
    const int64_t i = B.r0 + pr.i, j = B.c0 + pr.j;
    const double sr = f.re[l], si = f.im[l];
    const double s2r = sr * sr - si * si, s2i = 2.0 * sr * si;
    double ar = 0.0, ai = 0.0;
    bool any = false;
    for (int32_t e = g.pptr[i]; e < g.pptr[i + 1]; ++e) {
        const int ti = g.ptri[e], a = g.ploc[e];
        if (ti < t0 || ti >= t1) continue;
        any = true;
        const int64_t q0 = rowptr[ti], q1 = rowptr[ti + 1];
        double ca[3];
        if (OP == 0) gp1_curl(g, ti, a, ca);
        for (int32_t e2 = g.pptr[j]; e2 < g.pptr[j + 1]; ++e2) {
            const int tj = g.ptri[e2], b = g.ploc[e2];
            int64_t lo = q0, hi = q1 - 1;   // the row's pairs ascend in tj
            while (lo < hi) {
                const int64_t mid = (lo + hi) >> 1;
                if (pairs[mid].y < tj) lo = mid + 1;
                else hi = mid;
            }
            const double2 *slot = buf + ((lo - p0) * nfc + k) * 10;
            const double2 M = slot[3 * a + b];
            if (OP == 1) {
                ar += M.x;
                ai += M.y;
            } else {
                double cb[3];
                gp1_curl(g, tj, b, cb);
                const double cc = ca[0] * cb[0] + ca[1] * cb[1] + ca[2] * cb[2];
                const double nn = g.nx[ti] * g.nx[tj] + g.ny[ti] * g.ny[tj] + g.nz[ti] * g.nz[tj];
                const double2 S = slot[9];
                ar += cc * S.x + nn * (s2r * M.x - s2i * M.y);
                ai += cc * S.y + nn * (s2r * M.y + s2i * M.x);
            }
        }
    }
    const int64_t base = B.off + (int64_t)pr.i * f.L * B.n + pr.j;
    if (t0 > 0) {
        if (!any) return;
        const double2 s = out64[base + (int64_t)l * B.n];
        ar += s.x;
        ai += s.y;
    }
    out64[base + (int64_t)l * B.n] = make_double2(ar, ai);
    if (f.mirror && f.L - 1 - l != l) out64[base + (int64_t)(f.L - 1 - l) * B.n] = make_double2(ar, -ai);
}

void launch_gp1_fill(const GeoDev &g, const uint64_t *sets, int words, const int32_t *rowsetptr,
                     const int32_t *rowset, const int64_t *rowptr, int64_t T, const int32_t *chunk_of, int nchunk,
                     int2 *pairs, uint8_t *cls, unsigned long long *count, hipStream_t st) {
    gp1_zero_kernel<<<1, 256, 0, st>>>(count, nchunk * kGp1Classes);
    gp1_fill_kernel<<<(unsigned)((T + 3) / 4), 256, 0, st>>>(g, sets, words, rowsetptr, rowset, rowptr, T, chunk_of,
                                                            nchunk, pairs, cls, count);
}

void launch_gp1_list(const int2 *pairs, const uint8_t *cls, int64_t np, const int32_t *chunk_of, int nchunk,
                     unsigned long long *next, int32_t *list, hipStream_t st) {
    gp1_list_kernel<<<(unsigned)((np + 255) / 256), 256, 0, st>>>(pairs, cls, np, chunk_of, nchunk, next, list);
}

template <int OP>
static void launch_pairs(const Gp1Pairs &P, const Gp1Chunk &C, PairArgs A, hipStream_t st) {
    const unsigned ny = (unsigned)((A.nfc + NF - 1) / NF);
    auto cls = [&](int c) {
        A.list = P.list + C.first[c];
        A.cnt = C.first[c + 1] - C.first[c];
        return A.cnt > 0;
    };
    // the classes with the most points per pair first
    if (cls(GP1_VERTEX + 2)) gp1_touch_kernel<OP, 3><<<dim3((unsigned)A.cnt, ny), 64, 0, st>>>(A);
    if (cls(GP1_VERTEX + 1)) gp1_touch_kernel<OP, 2><<<dim3((unsigned)A.cnt, ny), 64, 0, st>>>(A);
    if (cls(GP1_VERTEX)) gp1_touch_kernel<OP, 1><<<dim3((unsigned)A.cnt, ny), 64, 0, st>>>(A);
    if (cls(GP1_NEAR)) gp1_near_kernel<OP><<<dim3((unsigned)A.cnt, ny), 64, 0, st>>>(A);
    if (cls(GP1_MID)) gp1_product_kernel<OP, true><<<dim3((unsigned)((A.cnt + 15) / 16), ny), 256, 0, st>>>(A);
    if (cls(GP1_FAR)) gp1_product_kernel<OP, false><<<dim3((unsigned)((A.cnt + 255) / 256), ny), 256, 0, st>>>(A);
}

template <int OP>
static void near_gp1_pairs(const GeoDev &g, const QuadDev &q, const FreqDev &f, const Gp1Pairs &P, double2 *buf,
                           int nfc_max, const NearPair *vp, int64_t nvp, const NearBlockDev *blocks,
                           double2 *out64, hipStream_t st) {
    for (int l0 = 0; l0 < f.L_eval; l0 += nfc_max) {
        const int nfc = f.L_eval - l0 < nfc_max ? f.L_eval - l0 : nfc_max;
        const dim3 grid((unsigned)((nvp + 255) / 256), (unsigned)nfc);
        for (int c = 0; c < P.nchunk; ++c) {
            const Gp1Chunk &C = P.chunks[c];
            launch_pairs<OP>(P, C, PairArgs{g, q, f, P.pairs, nullptr, 0, l0, nfc, C.p0, buf}, st);
            gp1_assemble_kernel<OP><<<grid, 256, 0, st>>>(g, f, vp, nvp, blocks, P.rowptr, P.pairs, buf, l0, nfc, C.t0,
                                                          C.t1, C.p0, out64);
        }
    }
}

void launch_near_gp1_pairs(int op, const GeoDev &g, const QuadDev &q, const FreqDev &f, const Gp1Pairs &P,
                           double2 *buf, int nfc_max, const NearPair *vp, int64_t nvp,
                           const NearBlockDev *blocks, double2 *out64, hipStream_t st) {
    if (nvp <= 0) return;
    if (op == 0) near_gp1_pairs<0>(g, q, f, P, buf, nfc_max, vp, nvp, blocks, out64, st);
    else near_gp1_pairs<1>(g, q, f, P, buf, nfc_max, vp, nvp, blocks, out64, st);
}

}  // namespace gaca
