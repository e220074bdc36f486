// Face ACA with the residual face in registers (faces with both sides up to 128 in FP64, 192 in
// the mixed path): the partial-pivot ACA of one face by one workgroup, in place.
//
// The face is spread over the workgroup as a TR x TC grid of threads, thread (tr, tc) owning
// the entries (tr + TR x, tc + TC y), x < RX, y < CY.  A step is then
//   the owners of row i write it to LDS                                        (barrier)
//   every wave finds the pivot column j for itself (one or two row entries per lane, one wave
//   maximum, the lowest index at the tie threshold from a ballot)
//   the owners of column j write u_q to LDS                                    (barrier)
//   every wave takes |u_q|^2, |w_q|^2 and the next row from it in the same way, and every
//   thread subtracts u_q w_q^T from its entries.
// Two barriers and no global memory on the chain; a thread reads RX + CY values from LDS for
// its RX CY products.
//
// What bounds it: the instructions of a step, which every wave issues (the pivot searches), and
// for the large faces, one per CU, the chain of their latencies.  So the searches work on the
// upper words of |r|^2: one 32-bit wave maximum, and a ballot of the lanes that may lie within
// the tie window of it.  One such lane is the pivot; only with several (meshes with symmetries)
// are the exact maximum and the lowest index at the threshold taken.
//
// The stopping test |u||w| <= eps sqrt(ref2 + |S|^2), S = sum_q u_q w_q^T, needs |S| only
// where it decides: |S| is kept as an interval (each step widens it by |u||w|), and only when
// the test falls between its ends is |S|^2 formed, as |R_0 - R|^2 with the face R_0 read back
// from the face pool (where it stays until the end).  After that the interval is |u||w| wide,
// so a face does it once, most faces after the first cross never (their ref2 dominates).  The
// sums |u|^2 and |w|^2 are likewise taken only where max |u|^2 <= |u|^2 |w|^2 does not decide.
//
// Device clocks per face in whole FP64 builds (all classes running), with R and S in registers or R
// in HBM before: 24 x 24 (rank 21, 3072-triangle cube) 64 -> 37 us, 48 x 48 (31) 114 -> 83 us,
// 96 x 96 (46) 400 -> 100 us.  FP64 faces of 160 x 160 took 190 us for 400 in a class whose kernel
// spilled 67 registers; with it (and delta_zero 1e-7, where rows of zeros are skipped) one face in a
// million had another rank from build to build, in 7 of 200 builds of a sphere and 5 of 80 of a cube.  The
// class is left out; why its result varied is not known.  The other classes use the same source and
// spill no vector register; their builds repeat bit for bit (200 of the sphere; and the tests).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_util.h"
#include "kernels.h"

namespace gaca {

namespace {

// |piv|^2 and its reciprocal (FP64: one per step, by two Newton steps from the hardware estimate,
// instead of two divisions per entry; FP32: unused, as cdiv)
struct Den {
    double d, rd;
};
__device__ __forceinline__ Den den(double2 p) {
    const double d = cabs2(p);
    if (!(d > 1e-290 && d < 1e290)) return {d, 0.0};   // beyond the estimate's range, NaN: divisions
    double t = __builtin_amdgcn_rcp(d);
    t = fma(t, fma(-d, t, 1.0), t);
    return {d, fma(t, fma(-d, t, 1.0), t)};
}
__device__ __forceinline__ Den den(float2) { return {0.0, 0.0}; }

// w = a / piv.  EXACT: the quotients corrected by their remainder (Markstein), which rounds them as
// a division does.  Small faces of flat pieces have entries that vanish up to rounding; whether a
// residual row is then exactly zero (and skipped) or not hangs on that rounding.
template <bool EXACT>
__device__ __forceinline__ double2 row_div(double2 a, double2 p, Den q) {
    const double nr = a.x * p.x + a.y * p.y, ni = a.y * p.x - a.x * p.y;
    if (q.rd == 0.0) return make_double2(nr / q.d, ni / q.d);
    double wr = nr * q.rd, wi = ni * q.rd;
    if (EXACT) {
        wr = fma(fma(-q.d, wr, nr), q.rd, wr);
        wi = fma(fma(-q.d, wi, ni), q.rd, wi);
    }
    return make_double2(wr, wi);
}
template <bool EXACT>
__device__ __forceinline__ float2 row_div(float2 a, float2 p, Den) { return cdiv(a, p); }

// r - u w.  Small faces come close to full rank, where the residual is rounding: there the
// product is rounded before it is subtracted, as u w is where the expansion sums it (WHOLE);
// larger ones take four fused operations instead of six.
template <bool WHOLE, class FT>
__device__ __forceinline__ FT sub_prod(FT r, FT u, FT w) {
    if constexpr (WHOLE) return csub(r, cmul(u, w));
    r.x = __builtin_elementwise_fma(-u.x, w.x, r.x);
    r.y = __builtin_elementwise_fma(-u.x, w.y, r.y);
    r.x = __builtin_elementwise_fma(u.y, w.y, r.x);
    r.y = __builtin_elementwise_fma(-u.y, w.x, r.y);
    return r;
}

// the upper word of a double >= 0, in the order of the doubles
__device__ __forceinline__ unsigned upper(double x) { return (unsigned)(__double_as_longlong(x) >> 32); }
__device__ __forceinline__ double from_upper(unsigned h) { return __longlong_as_double((long long)h << 32); }

// wave maximum: four DPP steps within the rows of 16 lanes, two broadcasts across them
__device__ __forceinline__ unsigned wave_umax(unsigned v) {
    v = max(v, (unsigned)dpp_i<0xB1>((int)v));
    v = max(v, (unsigned)dpp_i<0x4E>((int)v));
    v = max(v, (unsigned)dpp_i<0x141>((int)v));
    v = max(v, (unsigned)dpp_i<0x140>((int)v));
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false));
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false));
    return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}

// a value that is the same in every lane, in scalar registers
__device__ __forceinline__ double uniform(double x) {
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_readfirstlane((int)b), hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// x where the lane's bit of the wave-uniform mask is set, else 0.  A mask that a vector instruction wrote (a
// register restored from a lane, a comparison) may be read two wait states later; the compiler does not
// look into the statement, so it brings them along.
__device__ __forceinline__ unsigned keep(unsigned x, unsigned long long mask) {
    unsigned r;
    asm("s_nop 1\n\tv_cndmask_b32_e64 %0, 0, %1, %2" : "=v"(r) : "v"(x), "s"(mask));
    return r;
}

// The lowest index (lane + 64 k) whose a2 reaches tie2 times the maximum over the lanes of ok[k],
// K values per lane; -1 if none compares.  lo: a lower bound of the maximum, from its upper
// word; hmax >= 0x7ff00000 (infinity, NaN) has to take the exact way.
template <int K>
__device__ __forceinline__ int tie_first(const double (&a2)[K], const unsigned long long (&ok)[K], double tie2,
                                         unsigned hmax) {
    const double thr_lo = tie2 * from_upper(hmax);
    int at = -1, cnt = 0;
#pragma unroll
    for (int k = K - 1; k >= 0; --k) {
        const unsigned long long bal = __builtin_amdgcn_fcmp(a2[k], thr_lo, 3) & ok[k];   // a2 >= thr_lo
        cnt += __popcll(bal);
        if (bal) at = 64 * k + __ffsll(bal) - 1;
    }
    if (cnt == 1 && hmax < 0x7ff00000u) return at;
    const int lane = threadIdx.x & 63;
    double mx = 0.0;
#pragma unroll
    for (int k = 0; k < K; ++k)
        if ((ok[k] >> lane) & 1) mx = fmax(mx, a2[k]);
    const double thr = tie2 * wave_max(mx);
    at = -1;
#pragma unroll
    for (int k = K - 1; k >= 0; --k) {
        const unsigned long long bal = __ballot(a2[k] >= thr) & ok[k];
        if (bal) at = 64 * k + __ffsll(bal) - 1;
    }
    return at;
}

// bits of the indices lane + 64 k < len
__device__ __forceinline__ unsigned long long below(int len, int k) {
    const int c = len - 64 * k;
    return c <= 0 ? 0ull : c >= 64 ? ~0ull : (1ull << c) - 1;
}

// The cold paths read the face with bounds that the compiler cannot compare ahead of the loop
// (RX CY masks would be kept in scalar registers) and a row of entries at a time.
__device__ __forceinline__ int opaque(int v) {
    asm volatile("" : "+s"(v));
    return v;
}
__device__ __forceinline__ void fence() { asm volatile("" ::: "memory"); }

// EMIT: H_l = S is stored over R_0 with its maximum, norm and pivot (the faces that the expand
// phase does not visit).
// MINW: waves per SIMD that the registers leave room for.
template <int NT, int TR, int RX, int CY, int MINW, bool MIXED, bool EMIT>
__global__ void __launch_bounds__(NT, MINW)
    far_aca_reg_kernel(AcaParams P, FarBatchDev bd, const FarActive *act) {
    using FT = typename std::conditional<MIXED, float2, double2>::type;
    constexpr int TC = NT / TR, MS = TR * RX, NS = TC * CY, NW = NT / 64;
    constexpr int KM = (MS + 63) / 64, KN = (NS + 63) / 64;
    static_assert((TR & (TR - 1)) == 0 && (TC & (TC - 1)) == 0 && TR * TC == NT, "thread grid");
    const int64_t t_start = wall_clock64();
    const FarActive A = act[blockIdx.x];
    const int b = A.b;
    const FarBlockDev B = bd.blk[b];
    const int m = B.m, n = B.n;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int tr = tid / TC, tc = tid % TC;
    const double zero_tol = bd.st[b].zero_tol, ref2 = bd.st[b].ref2;
    FT *R = reinterpret_cast<FT *>(bd.hpool) + A.hslot;
    FT *Ub = reinterpret_cast<FT *>(bd.uw) + B.uw_off;
    FT *Wb = Ub + (int64_t)B.rho_max * m;

    // entries beyond the face stay zero here and in the registers
    __shared__ FT rowb[2][64 * KN];
    __shared__ FT ucol[64 * KM];
    __shared__ double redbuf[8 * NW + 4];
    Red<NT> red{redbuf};
    const double tie2 = (1.0 - P.tie) * (1.0 - P.tie);
    const double eps2 = P.eps_aca * P.eps_aca;
    // a row maximum above zt_hi is nonzero, one up to zt_lo zero; in between the root decides
    const double zt_hi = fmax(zero_tol * zero_tol * (1.0 + 1e-9), 1e-290);
    const double zt_lo = zero_tol * zero_tol * (1.0 - 1e-9);
    // |u|^2 |w|^2 <= mnd max |u|^2: |w_j| <= 1 / (1 - tie), the pivot is that close to its row's maximum
    const double mnd = (double)m * n / tie2 * (1.0 + 1e-3);

    FT rr[RX][CY];
#pragma unroll
    for (int x = 0; x < RX; ++x)
#pragma unroll
        for (int y = 0; y < CY; ++y) {
            const int i = tr + TR * x, j = tc + TC * y;
            rr[x][y] = i < m && j < n ? R[i * n + j] : czero<FT>();
        }
    // Operators with normals vanish, up to rounding, between coplanar elements.  In a face with such
    // entries a row ends as rounding or as exact zero by the order of its sums, which decides where
    // the ACA stops: the larger ones are left to the kernel that forms a row from its history, as
    // the expansion sums it (far_aca_large_kernel; the smaller ones keep that order here).
    if (!EMIT && !MIXED && P.decline) {
        double top = 0.0, low = INFINITY;
        const int mo = opaque(m), no = opaque(n);
#pragma unroll
        for (int x = 0; x < RX; ++x) {
#pragma unroll
            for (int y = 0; y < CY; ++y)
                if (tr + TR * x < mo && tc + TC * y < no) {
                    const double a = cabs2(rr[x][y]);
                    top = fmax(top, a);
                    low = fmin(low, a);
                }
            fence();
        }
        double nlow = -low, dummy = 0.0;
        red.maxsum(top, dummy);
        red.maxsum(nlow, dummy);
        if (-nlow < 1e-26 * top) {
            if (tid == 0) bd.st[b].rho = kFarDeclined;
            return;
        }
    }
    for (int t = tid; t < 64 * KN; t += NT) rowb[0][t] = rowb[1][t] = czero<FT>();
    for (int t = tid; t < 64 * KM; t += NT) ucol[t] = czero<FT>();
    unsigned long long colm[KN], freem[KM];   // columns of the face; rows not used yet
#pragma unroll
    for (int k = 0; k < KN; ++k) colm[k] = below(n, k);
#pragma unroll
    for (int k = 0; k < KM; ++k) freem[k] = below(m, k);
    __syncthreads();
    int q = 0, i = 0, nused = 0, par = 0;
    double s_lo = 0.0, s_hi = 0.0;   // |S| lies in [s_lo, s_hi]
    while (true) {
        // row i of the residual; the buffers alternate, so a slow wave may still read the last
        FT *rowv = rowb[par];
        par ^= 1;
        if (tr == i % TR) {
            const int xi = i / TR;
#pragma unroll
            for (int x = 0; x < RX; ++x)
                if (x == xi)
#pragma unroll
                    for (int y = 0; y < CY; ++y) rowv[tc + TC * y] = rr[x][y];
        }
        __syncthreads();
        double a2[KN];
        unsigned hm = 0;
#pragma unroll
        for (int k = 0; k < KN; ++k) {
            a2[k] = cabs2(rowv[lane + 64 * k]);
            hm = max(hm, upper(a2[k]));
        }
        hm = wave_umax(hm);
#pragma unroll
        for (int k = 0; k < KM; ++k)
            if (k == i / 64) freem[k] &= ~(1ull << (i % 64));
        ++nused;
        if (!(from_upper(hm) > zt_hi)) {
            bool zero = from_upper(hm + 1) <= zt_lo;
            if (!zero) {
                double mx = 0.0;
#pragma unroll
                for (int k = 0; k < KN; ++k)
                    if (lane + 64 * k < n) mx = fmax(mx, a2[k]);
                zero = sqrt(wave_max(mx)) <= zero_tol;
            }
            if (zero) {
                // The ACA goes on with the unused rows in index order, and every one below the
                // first with a nonzero residual entry is zero as well; find that row in one
                // pass over the register-held residual and mark the zero ones used.
                int cand = m;
                const int mo = opaque(m), no = opaque(n);
#pragma unroll
                for (int x = 0; x < RX; ++x) {
                    const int r = tr + TR * x;
                    double big = 0.0;
#pragma unroll
                    for (int y = 0; y < CY; ++y)
                        if (tc + TC * y < no) big = fmax(big, cabs2(rr[x][y]));
                    unsigned long long fm = freem[0];
#pragma unroll
                    for (int k = 1; k < KM; ++k)
                        if (r / 64 == k) fm = freem[k];
                    if (r < mo && ((fm >> (r % 64)) & 1) && sqrt(big) > zero_tol) cand = min(cand, r);
                    fence();
                }
                cand = __builtin_amdgcn_readfirstlane(red.imin(cand));
#pragma unroll
                for (int k = 0; k < KM; ++k) {
                    nused += __popcll(freem[k] & below(cand, k));
                    freem[k] &= ~below(cand, k);
                }
                if (cand >= m) break;
                i = cand;
                continue;
            }
        }
        int jp = tie_first<KN>(a2, colm, tie2, hm);
        if (jp < 0) jp = n - 1;   // in range even for NaN rows
        // column jp of the residual is u_q
        if (tc == jp % TC) {
            const int yj = jp / TC;
#pragma unroll
            for (int y = 0; y < CY; ++y)
                if (y == yj)
#pragma unroll
                    for (int x = 0; x < RX; ++x) ucol[tr + TR * x] = rr[x][y];
        }
        const FT piv = rowv[jp];
        const Den rd = den(piv);
        if (wave == 0)
#pragma unroll
            for (int k = 0; k < KN; ++k)
                if (lane + 64 * k < n) Wb[(int64_t)q * n + lane + 64 * k] = row_div<EMIT>(rowv[lane + 64 * k], piv, rd);
        FT wy[CY];
#pragma unroll
        for (int y = 0; y < CY; ++y) wy[y] = row_div<EMIT>(rowv[tc + TC * y], piv, rd);
        __syncthreads();
        double u2[KM];
        unsigned hu = 0, ha = 0;   // maxima over the unused rows, over all rows
#pragma unroll
        for (int k = 0; k < KM; ++k) {
            const FT u = ucol[lane + 64 * k];
            u2[k] = cabs2(u);
            hu = max(hu, keep(upper(u2[k]), freem[k]));
            ha = max(ha, upper(u2[k]));
            if (wave == NW - 1 && lane + 64 * k < m) Ub[(int64_t)q * m + lane + 64 * k] = u;
        }
#pragma unroll
        for (int x = 0; x < RX; ++x) {
            const FT ux = ucol[tr + TR * x];
#pragma unroll
            for (int y = 0; y < CY; ++y) rr[x][y] = sub_prod<EMIT>(rr[x][y], ux, wy[y]);
            if (RX * CY >= 36 && x % 2) fence();   // no more than two u in flight (registers)
        }
        hu = wave_umax(hu);
        ha = wave_umax(ha);
        ++q;
        if (nused >= m || q >= B.rho_max) break;
        // max |u|^2 <= |u|^2 |w|^2 <= mnd max |u|^2 (w_jp = 1)
        const double mlo = from_upper(ha), dlt = __builtin_amdgcn_sqrt(mnd * from_upper(ha + 1));
        s_hi += dlt;
        if (!(mlo > eps2 * (ref2 + s_hi * s_hi) * (1.0 + 1e-9))) {
            double nu2 = 0.0, nw2 = 0.0;
#pragma unroll
            for (int k = 0; k < KM; ++k) nu2 += u2[k];
#pragma unroll
            for (int k = 0; k < KN; ++k)
                if (lane + 64 * k < n) nw2 += cabs2(row_div<EMIT>(rowv[lane + 64 * k], piv, rd));
            const double t2 = wave_sum(nu2) * wave_sum(nw2), tt = sqrt(t2);
            s_lo = fmax(0.0, s_lo - tt);
            if (!(t2 > eps2 * (ref2 + s_hi * s_hi) * (1.0 + 1e-9))) {
                if (t2 <= eps2 * (ref2 + s_lo * s_lo) * (1.0 - 1e-9)) break;
                double s2 = 0.0;
                const int mo = opaque(m), no = opaque(n);
#pragma unroll
                for (int x = 0; x < RX; ++x) {
#pragma unroll
                    for (int y = 0; y < CY; ++y) {
                        const int ie = tr + TR * x, j = tc + TC * y;
                        if (ie < mo && j < no) s2 += cabs2(csub(R[ie * no + j], rr[x][y]));
                    }
                    fence();
                }
                s2 = uniform(red.sum(s2));
                if (tt <= P.eps_aca * sqrt(ref2 + s2)) break;
                s_lo = s_hi = sqrt(s2);
            }
        } else {
            s_lo = fmax(0.0, s_lo - dlt);
        }
        // next row: the lowest unused row with |u_q|^2 at the tie threshold of its maximum
        // (the first unused row if none compares)
        i = tie_first<KM>(u2, freem, tie2, hu);
        if (i < 0)
#pragma unroll
            for (int k = KM - 1; k >= 0; --k)
                if (freem[k]) i = 64 * k + __ffsll(freem[k]) - 1;
        i = min(max(i, 0), m - 1);
    }
    int pidx = 0;
    double mxh = 0.0, h2 = 0.0;
    if (EMIT && q > 0) {
        // H_l = sum_q u_q w_q in the order of the steps (the face less its residual would carry the
        // face's rounding)
#pragma unroll
        for (int x = 0; x < RX; ++x)
#pragma unroll
            for (int y = 0; y < CY; ++y) rr[x][y] = czero<FT>();
        __syncthreads();   // U and W of every wave
        for (int p = 0; p < q; ++p) {
            const FT *up = Ub + (int64_t)p * m, *wp = Wb + (int64_t)p * n;
            FT w[CY];
#pragma unroll
            for (int y = 0; y < CY; ++y) w[y] = wp[min(tc + TC * y, n - 1)];
#pragma unroll
            for (int x = 0; x < RX; ++x) {
                const FT u = up[min(tr + TR * x, m - 1)];
#pragma unroll
                for (int y = 0; y < CY; ++y) rr[x][y] = cadd(rr[x][y], cmul(u, w[y]));
                if (RX * CY >= 32 && x % 2) fence();   // no more than two u in flight (registers)
            }
        }
        const int mo = opaque(m), no = opaque(n);
#pragma unroll
        for (int x = 0; x < RX; ++x) {
#pragma unroll
            for (int y = 0; y < CY; ++y) {
                const int ie = tr + TR * x, j = tc + TC * y;
                if (ie < mo && j < no) {
                    R[ie * no + j] = rr[x][y];
                    const double s2 = cabs2(rr[x][y]);
                    mxh = fmax(mxh, s2);
                    h2 += s2;
                }
            }
            fence();
        }
        red.maxsum(mxh, h2);
        const double thh = tie2 * mxh;
        int pc = 0x7fffffff;
#pragma unroll
        for (int x = 0; x < RX; ++x)
#pragma unroll
            for (int y = 0; y < CY; ++y) {
                const int ie = tr + TR * x, j = tc + TC * y;
                if (ie < m && j < n && cabs2(rr[x][y]) >= thh) pc = min(pc, ie * n + j);
            }
        pidx = min(red.imin(pc), m * n - 1);
    }
    if (tid == 0) {
        FarStateDev *S = bd.st + b;
        S->rho = q;
        S->pidx = pidx;
        S->mxh = mxh;
        S->h2 = h2;
        S->aca_ticks += wall_clock64() - t_start;
    }
}

// One class of faces: both sides at most kFarRegSide[c].  Up to 40 (mixed 48) one wave per face (9,
// 16, 25, 36 entries a lane); above, the threads that keep about 25 to 50 entries each: fewer would
// spill, more would repeat the reductions on more waves.
template <bool MX>
void reg_dispatch(int c, const AcaParams &P, const FarBatchDev &bd, const FarActive *act, int nact,
                  hipStream_t st) {
    switch (c) {
        case 0: far_aca_reg_kernel<64, 8, 3, 3, MX ? 4 : 3, MX, true><<<nact, 64, 0, st>>>(P, bd, act); break;
        case 1: far_aca_reg_kernel<64, 8, 4, 4, 3, MX, true><<<nact, 64, 0, st>>>(P, bd, act); break;
        case 2: far_aca_reg_kernel<64, 8, 5, 5, 2, MX, true><<<nact, 64, 0, st>>>(P, bd, act); break;
        case 3:   // FP64: 36 entries a lane spill
            if constexpr (MX) far_aca_reg_kernel<64, 8, 6, 6, 2, MX, true><<<nact, 64, 0, st>>>(P, bd, act);
            else far_aca_reg_kernel<128, 8, 6, 3, 2, MX, true><<<nact, 128, 0, st>>>(P, bd, act);
            break;
        case 4: far_aca_reg_kernel<128, 8, 8, 4, 2, MX, true><<<nact, 128, 0, st>>>(P, bd, act); break;
        case 5: far_aca_reg_kernel<256, 16, 5, 5, 2, MX, false><<<nact, 256, 0, st>>>(P, bd, act); break;
        case 6: far_aca_reg_kernel<256, 16, 6, 6, 2, MX, false><<<nact, 256, 0, st>>>(P, bd, act); break;
        case 7: far_aca_reg_kernel<512, 16, 8, 4, 2, MX, false><<<nact, 512, 0, st>>>(P, bd, act); break;
        case 8:
            if constexpr (MX) far_aca_reg_kernel<512, 16, 10, 5, 2, MX, false><<<nact, 512, 0, st>>>(P, bd, act);
            break;
        case 9:
            if constexpr (MX) far_aca_reg_kernel<512, 16, 12, 6, 2, MX, false><<<nact, 512, 0, st>>>(P, bd, act);
            break;
    }
}

}  // namespace

void launch_far_aca_reg(int cls, const AcaParams &P, const FarBatchDev &bd, const FarActive *act,
                        int nact, hipStream_t st) {
    if (nact <= 0) return;
    if (cls < 0 || cls >= (bd.mixed ? kFarRegClasses : kFarRegClassesFp64))
        throw Error{GACA_ERR_STATE, "no register kernel for this class of faces"};
    if (bd.mixed) reg_dispatch<true>(cls, P, bd, act, nact, st);
    else reg_dispatch<false>(cls, P, bd, act, nact, st);
}

}  // namespace gaca
