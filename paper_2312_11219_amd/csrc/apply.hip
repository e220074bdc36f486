// Reordered product eq. (product) of the compressed operator:
//   SUM:      Y[:, b] = sum_l C(s_l) X_l[:, b]
//             far blocks: z_l = W_l^T (sum_k f_l[k] X_k[tau]),  y_b = sum_l U_l z_l
//             near blocks: Y[sigma] += sum_k N_k X_k[tau]
//   PER_FREQ: Y_k = C(s_k) X_k.
// Templated on the storage of factors / near field (FacT: double2 for the FP64 build,
// float2 for the mixed build) and on the right-hand sides (XT: complex128 or complex64),
// whose type also sets the arithmetic.  Owner-computes per leaf cluster: no atomics,
// every sum in a fixed order (deterministic).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>

#include "device_util.h"
#include "kernels.h"

namespace gaca {

// ---------------------------------------------------------------------------------------
// Workspace of the allocation-free apply: one fixed array per device, alive until the
// process ends.  Host code never passes `scratch` itself to a kernel (in host code the name
// is a host-side stand-in): it uses the device address that hipGetSymbolAddress returns,
// taken once per device with that device current.
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {
std::mutex g_scratch_mu;
void *g_scratch_addr[kMaxDevices] = {};
}  // namespace

hipError_t scratch_setup(int device) {
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (g_scratch_addr[device]) return hipSuccess;
    void *ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_addr[device] = ptr;
    return hipSuccess;
}

void *scratch_address(int device) {
    if (device < 0 || device >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    return g_scratch_addr[device];
}

// Per-block offsets of z from the block metadata (what the host computes for the allocated
// workspace): prefix of sum_rho * nrhs (SUM) or sum_rho * L * nrhs (PER_FREQ).
// One workgroup: each thread sums a contiguous run of blocks,
// the run totals are scanned in LDS, then each thread writes its run's prefixes.
__global__ void __launch_bounds__(1024) apply_offsets_kernel(ApplyDev a, int mode, int64_t *zoff) {
    __shared__ int64_t sz[1024];
    const int nb = a.nfar, t = threadIdx.x;
    const int per = (nb + 1023) / 1024;
    const int b0 = min(nb, t * per), b1 = min(nb, b0 + per);
    const int64_t zmul = mode == 0 ? a.nrhs : (int64_t)a.L * a.nrhs;
    int64_t z = 0;
    for (int b = b0; b < b1; ++b) z += a.meta[b].sum_rho * zmul;
    sz[t] = z;
    __syncthreads();
    for (int d = 1; d < 1024; d <<= 1) {
        const int64_t vz = t >= d ? sz[t - d] : 0;
        __syncthreads();
        sz[t] += vz;
        __syncthreads();
    }
    z = sz[t] - z;
    for (int b = b0; b < b1; ++b) {
        zoff[b] = z;
        z += a.meta[b].sum_rho * zmul;
    }
}

void launch_apply_offsets(const ApplyDev &a, int mode, int64_t *zoff, hipStream_t st) {
    if (a.nfar < 1) return;
    apply_offsets_kernel<<<1, 1024, 0, st>>>(a, mode, zoff);
}

template <class XT>
__global__ void permute_x_kernel(const XT *X, XT *Xp, const int64_t *perm, int L, int64_t M,
                                 int nrhs) {
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t total = (int64_t)L * M * nrhs;
    if (t >= total) return;
    int c = (int)(t % nrhs);
    int64_t rest = t / nrhs;
    int64_t p = rest % M;
    int64_t l = rest / M;
    Xp[t] = X[(l * M + perm[p]) * nrhs + c];
}

__device__ __forceinline__ int64_t readlane_i64(int64_t v, int l) {
    const int lo = __builtin_amdgcn_readlane((int)v, l), hi = __builtin_amdgcn_readlane((int)(v >> 32), l);
    return ((int64_t)hi << 32) | (unsigned)lo;
}

// sum over the eight lanes of a group, in every one of them (FP64 partial sums)
template <class XT>
__device__ __forceinline__ XT sum8(XT v) {
    double x = v.x, y = v.y;
    x += dpp_d<0xB1>(x);
    y += dpp_d<0xB1>(y);
    x += dpp_d<0x4E>(x);
    y += dpp_d<0x4E>(y);
    x += dpp_d<0x141>(x);
    y += dpp_d<0x141>(y);
    v.x = x;
    v.y = y;
    return v;
}

// 16 x 16 complex tiles of the matrix cores, four steps of the contraction at a time
template <class XT>
struct Mma;
template <>
struct Mma<double2> {
    typedef double v4 __attribute__((ext_vector_type(4)));
    // lane l holds rows l / 16 + 4 t, t = 0..3, of column l % 16
    static __device__ int row(int lane, int t) { return (lane >> 4) + 4 * t; }
    static __device__ v4 mac(double a, double b, v4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
};
template <>
struct Mma<float2> {
    typedef float v4 __attribute__((ext_vector_type(4)));
    static __device__ int row(int lane, int t) { return 4 * (lane >> 4) + t; }
    static __device__ v4 mac(float a, float b, v4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
};

template <class XT>
struct CTile16 {   // 16 x 16 complex
    typename Mma<XT>::v4 r = {0, 0, 0, 0}, i = {0, 0, 0, 0};
    __device__ void mac(XT a, XT b) {
        r = Mma<XT>::mac(a.x, b.x, r);
        r = Mma<XT>::mac(-a.y, b.y, r);
        i = Mma<XT>::mac(a.x, b.y, i);
        i = Mma<XT>::mac(a.y, b.x, i);
    }
    __device__ XT get(int t) const {
        XT v;
        v.x = r[t];
        v.y = i[t];
        return v;
    }
};

// SUM, in two launches after the permutation of X:
//   parts   far blocks: T_l = sum_k f_l[k] X_k[tau] (n x nrhs) and z_l = W_l^T T_l for every cross,
//           one workgroup per block; then, in the same launch, near rows: sum_k N_k X_k, four rows
//           per workgroup;
//   rows    Y[leaf] = near part + sum_b U_b z_b, eight waves per leaf, every U read once.
// What bounds them: the stored operator read once from HBM.  6912-triangle sphere, L = 128, one
// complex128 right-hand side (13.1 GB near field, 6.5 GB factors): far blocks 1.3 ms, near rows
// 2.4 ms (5.5 TB/s), rows 0.8 ms (4 TB/s).  With T in global memory, y per far block and the near
// rows read by one thread per row and block: 6.9 ms for 4.5.  Far blocks and near rows in turn
// rather than one kind after the other took 4.8 ms for the 3.7 of the launch.

// Far block b, up to 16 crosses and kFarTC columns (j, rhs) at a time: T = F X on the matrix cores,
// a wave per 16 columns, into LDS (its operands come straight from L2: the crosses of a block fill
// a tile, and X is read once for all of them); then the rows of z = W^T T, 8 lanes each over j (W
// read in order) for RC right-hand sides, summed in a fixed order.
constexpr int kFarTC = 128;
template <class FacT, class XT, int RC>
__device__ void far_z(const ApplyDev &a, int b, const XT *Xp, XT *zbuf, XT (*s_t)[kFarTC + 1]) {
    constexpr int KS = 4, WU = 4;   // loads in flight: steps of the contraction, steps along a row of W
    __shared__ int64_t s_w[16];
    __shared__ int s_row[17];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, kq = lane >> 4, c16 = lane & 15;
    const int m = a.far4[4 * b + 1], c0 = a.far4[4 * b + 2], n = a.far4[4 * b + 3];
    const int rank = a.meta[b].rank, L = a.L, nr = a.nrhs;
    const int64_t ks = a.M * nr;
    XT *z = zbuf + a.z_off[b];
    const FacT *arena = reinterpret_cast<const FacT *>(a.arena);
    const double2 *F = a.fib_arena + a.fib_off[b];
    const int RB = min(nr, kFarTC), JC = kFarTC / RB;   // columns of one pass: JC entries j, RB right-hand sides
    for (int cg = 0; cg < rank; cg += 16) {
        const int cb = min(16, rank - cg);
        __syncthreads();   // the last group's z rows are read from s_row, s_w and s_t
        if (tid < 64) {
            const int cl = cg + min(c16, cb - 1);
            const int rho = a.cmeta[(int64_t)b * a.rcap + cl].rho;
            int q1 = c16 < cb ? rho : 0;
#pragma unroll
            for (int d = 1; d < 16; d <<= 1) {
                const int v = __shfl_up(q1, d, 16);
                if (c16 >= d) q1 += v;
            }
            if (tid < 16) {
                s_w[tid] = a.cross_off[(int64_t)b * a.rcap + cl] + (int64_t)rho * m;
                s_row[tid + 1] = q1;
                if (tid == 0) s_row[0] = 0;
            }
        }
        const double2 *f = F + (int64_t)(cg + min(c16, cb - 1)) * L;
        for (int r0 = 0; r0 < nr; r0 += RB) {
            const int rb = min(RB, nr - r0);
            for (int j0 = 0; j0 < n; j0 += JC) {
                const int jn = min(JC, n - j0), nt = jn * rb;
                __syncthreads();   // s_t is free, s_row is there
                for (int t0 = 16 * wave; t0 < nt; t0 += 64) {
                    const int t = t0 + c16, tc = min(t, nt - 1), jl = tc / rb;
                    const XT *x = Xp + (int64_t)(c0 + j0 + jl) * nr + r0 + (tc - jl * rb);
                    CTile16<XT> acc;
                    for (int k0 = 0; k0 < L; k0 += 4 * KS) {
                        XT av[KS], bv[KS];
#pragma unroll
                        for (int s = 0; s < KS; ++s) {
                            const int k = k0 + 4 * s + kq, kc = min(k, L - 1);
                            av[s] = cast_c<XT>(f[kc]);
                            bv[s] = x[kc * ks];
                            if (k >= L) av[s] = bv[s] = czero<XT>();
                        }
#pragma unroll
                        for (int s = 0; s < KS; ++s) acc.mac(av[s], bv[s]);
                    }
                    if (t < nt)
#pragma unroll
                        for (int i = 0; i < 4; ++i) s_t[Mma<XT>::row(lane, i)][t] = acc.get(i);
                }
                __syncthreads();
                const int rows = s_row[cb], l8 = tid & 7;
                int c = 0;
                for (int ri = tid >> 3; ri < rows; ri += 32) {
                    while (s_row[c + 1] <= ri) ++c;
                    const FacT *w = arena + s_w[c] + (int64_t)(ri - s_row[c]) * n + j0;
                    for (int cr = 0; cr < rb; cr += RC) {
                        XT acc[RC];
#pragma unroll
                        for (int v = 0; v < RC; ++v) acc[v] = czero<XT>();
                        for (int jb = l8; jb < jn; jb += 8 * WU) {
                            XT wv[WU];
#pragma unroll
                            for (int u = 0; u < WU; ++u) {
                                wv[u] = cast_c<XT>(w[min(jb + 8 * u, jn - 1)]);
                                if (jb + 8 * u >= jn) wv[u] = czero<XT>();
                            }
#pragma unroll
                            for (int u = 0; u < WU; ++u) {
                                const XT *tr = s_t[c] + min(jb + 8 * u, jn - 1) * rb + cr;
#pragma unroll
                                for (int v = 0; v < RC; ++v)
                                    if (cr + v < rb && jb + 8 * u < jn) acc[v] = cfma(wv[u], tr[v], acc[v]);
                            }
                        }
                        XT *zp = z + (int64_t)ri * nr + r0 + cr;
#pragma unroll
                        for (int v = 0; v < RC; ++v) {
                            const XT r = sum8(acc[v]);
                            if (l8 == v && cr + v < rb) zp[v] = j0 > 0 ? cadd(zp[v], r) : r;
                        }
                    }
                }
            }
        }
        z += (int64_t)s_row[cb] * nr;
    }
}

// SUM, compressed near blocks: T_l = sum_k f_l[k] X_k[tau] ([crank][n][nrhs]) per block;
// one workgroup per near block (dense ones return at once).
template <class XT>
__global__ void __launch_bounds__(256) apply_near_t_kernel(ApplyDev a, const XT *Xp, XT *tn) {
    const NearBlockDev nb = a.nblocks[blockIdx.x];
    if (!nb.comp || nb.crank == 0) return;
    const int L = a.L, nr = a.nrhs, n = nb.n;
    const int64_t M = a.M;
    const double2 *F = a.near_fib + nb.foff;
    XT *T = tn + a.tn_off[blockIdx.x];
    const int64_t tot = (int64_t)nb.crank * n * nr;
    for (int64_t t = threadIdx.x; t < tot; t += blockDim.x) {
        const int cc = (int)(t % nr);
        const int64_t rest = t / nr;
        const int j = (int)(rest % n), l = (int)(rest / n);
        const XT *xp = Xp + (int64_t)(nb.c0 + j) * nr + cc;
        XT acc = czero<XT>();
        for (int k = 0; k < L; ++k) acc = cfma(cast_c<XT>(F[(int64_t)l * L + k]), xp[(int64_t)k * M * nr], acc);
        T[t] = acc;
    }
}

// Near part of four rows of a leaf: a near block stores a row as L n contiguous entries
// ([m][L][n]), which the lanes read in order (entry t: frequency t / n, column t % n), four rows at
// a time so that an element of X serves four products; the four waves take every fourth near
// block.  The sums go to Yn (tree order).
template <class NearT, class XT, int RC>
__device__ void near_rows(const ApplyDev &a, int leaf, int rg, const XT *Xp, XT *Yn, const XT *tn,
                          XT (*part)[4 * RC]) {
    constexpr int RW = 4, LU = 2;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int lm = a.leaf_m[leaf], r0 = RW * rg;
    if (r0 >= lm) return;   // the whole workgroup
    const int L = a.L, nr = a.nrhs;
    const int64_t M = a.M;
    const NearT *nearv = a.near64 ? reinterpret_cast<const NearT *>(a.near64)
                                  : reinterpret_cast<const NearT *>(a.near32);
    int row[RW];
#pragma unroll
    for (int r = 0; r < RW; ++r) row[r] = a.leaf_r0[leaf] + min(r0 + r, lm - 1);
    const int e1 = a.leaf_near_ptr[leaf + 1];
    for (int cr = 0; cr < nr; cr += RC) {
        XT acc[RW][RC];
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int c = 0; c < RC; ++c) acc[r][c] = czero<XT>();
        for (int e0 = a.leaf_near_ptr[leaf] + wave; e0 < e1; e0 += 4 * 64) {
            // the descriptors of the wave's next 64 blocks, a lane each
            const int ib_l = a.leaf_near_idx[min(e0 + 4 * lane, e1 - 1)];
            const NearBlockDev nb_l = a.nblocks[ib_l];
            for (int i = 0; i < min(64, (e1 - e0 + 3) / 4); ++i) {
                const int ib = __builtin_amdgcn_readlane(ib_l, i);
                NearBlockDev nb;
                nb.r0 = __builtin_amdgcn_readlane(nb_l.r0, i);
                nb.m = __builtin_amdgcn_readlane(nb_l.m, i);
                nb.c0 = __builtin_amdgcn_readlane(nb_l.c0, i);
                nb.n = __builtin_amdgcn_readlane(nb_l.n, i);
                nb.off = readlane_i64(nb_l.off, i);
                nb.comp = __builtin_amdgcn_readlane(nb_l.comp, i);
                nb.crank = __builtin_amdgcn_readlane(nb_l.crank, i);
                const int n = nb.n;
                const NearT *base[RW];
                int64_t rs;   // entries per step of the row index t / n
                const XT *xb;
                int E;
                if (nb.comp) {
                    // row ro of sum_l H_l (T_l): entry t = (l, j), H_l row ro at l m n + ro n
                    const int mn = nb.m * n;
#pragma unroll
                    for (int r = 0; r < RW; ++r)
                        base[r] = reinterpret_cast<const NearT *>(a.near_faces) + nb.off + (int64_t)(row[r] - nb.r0) * n;
                    rs = mn - n;
                    xb = tn + a.tn_off[ib] + cr;
                    E = nb.crank * n;
                } else {
#pragma unroll
                    for (int r = 0; r < RW; ++r) base[r] = nearv + nb.off + (int64_t)(row[r] - nb.r0) * L * n;
                    rs = 0;
                    xb = Xp + (int64_t)nb.c0 * nr + cr;
                    E = L * n;
                }
                const int64_t xs = nb.comp ? (int64_t)n : M;   // X rows per frequency (T rows per cross)
                // (k, j) of entry t = lane + 64 i, advanced by 64 entries per step
                int k = lane / n, j = lane - k * n;
                const int dk = 64 / n, dj = 64 - dk * n;
                for (int t = lane; t < E; t += 64 * LU) {
                    XT nv[LU][RW], xv[LU][RC];
#pragma unroll
                    for (int u = 0; u < LU; ++u) {
                        const bool ok = t + 64 * u < E;   // past the end: the first entry, times 0
                        const int64_t to = ok ? t + 64 * u + k * rs : 0;
                        const XT *xp = xb + (ok ? (k * xs + j) * nr : 0);
#pragma unroll
                        for (int r = 0; r < RW; ++r) nv[u][r] = cast_c<XT>(base[r][to]);
#pragma unroll
                        for (int c = 0; c < RC; ++c) xv[u][c] = ok && cr + c < nr ? xp[c] : czero<XT>();
                        if (!ok)
#pragma unroll
                            for (int r = 0; r < RW; ++r) nv[u][r] = czero<XT>();
                        k += dk;
                        j += dj;
                        if (j >= n) {
                            j -= n;
                            ++k;
                        }
                    }
#pragma unroll
                    for (int u = 0; u < LU; ++u)
#pragma unroll
                        for (int c = 0; c < RC; ++c)
#pragma unroll
                            for (int r = 0; r < RW; ++r) acc[r][c] = cfma(nv[u][r], xv[u][c], acc[r][c]);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int c = 0; c < RC; ++c) {
                XT v;
                v.x = wave_sum((double)acc[r][c].x);
                v.y = wave_sum((double)acc[r][c].y);
                if (lane == 0) part[wave][r * RC + c] = v;
            }
        __syncthreads();
        const int r = threadIdx.x / RC, c = threadIdx.x - r * RC;
        if (r < RW && r0 + r < lm && cr + c < nr)
            Yn[(int64_t)(a.leaf_r0[leaf] + r0 + r) * nr + cr + c] =
                cadd(cadd(part[0][threadIdx.x], part[1][threadIdx.x]), cadd(part[2][threadIdx.x], part[3][threadIdx.x]));
        __syncthreads();   // the next columns' sums take the same place
    }
}

template <class FacT, class XT, int RC>
__global__ void __launch_bounds__(256) apply_sum_parts_kernel(ApplyDev a, const XT *Xp, XT *zbuf, XT *Yn,
                                                              const XT *tn) {
    __shared__ XT s[16][kFarTC + 1];
    if ((int)blockIdx.x < a.nfar) {
        far_z<FacT, XT, RC>(a, blockIdx.x, Xp, zbuf, s);
        return;
    }
    XT (*part)[4 * RC] = reinterpret_cast<XT (*)[4 * RC]>(s[0]);
    const int w = blockIdx.x - a.nfar, groups = (a.max_leaf_m + 3) / 4;
    near_rows<FacT, XT, RC>(a, w / groups, w % groups, Xp, Yn, tn, part);
}

// Y[leaf rows] = near part + sum over the far blocks of U z, in the caller's order: RL rows at a
// time on adjacent lanes, the wave's 64 / RL lane groups take every (64 / RL)-th step q, the eight
// waves every eighth far block
template <class FacT, class XT, int RC, int RL>
__global__ void __launch_bounds__(512) apply_sum_rows_kernel(ApplyDev a, const XT *zbuf, const XT *Yn, XT *Y) {
    constexpr int QS = 64 / RL, NW = 8, SU = 4;
    __shared__ XT part[NW * QS][RL][RC];
    __shared__ int64_t s_off[NW][64];
    __shared__ int s_q1[NW][64];
    const int leaf = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int lm = min(RL, a.leaf_m[leaf] - RL * (int)blockIdx.y), row0 = a.leaf_r0[leaf] + RL * blockIdx.y;
    if (lm <= 0) return;
    const int nr = a.nrhs, r = lane & (RL - 1), rc = min(r, lm - 1), qs = lane / RL;
    const FacT *arena = reinterpret_cast<const FacT *>(a.arena);
    const int fp1 = a.leaf_far_ptr[leaf + 1];
    for (int cr = 0; cr < nr; cr += RC) {
        XT acc[RC];
#pragma unroll
        for (int c = 0; c < RC; ++c) acc[c] = czero<XT>();
        for (int e0 = a.leaf_far_ptr[leaf] + wave; e0 < fp1; e0 += NW * 64) {
            // the descriptors of the wave's next 64 blocks, a lane each
            const int b_l = a.leaf_far_idx[min(e0 + NW * lane, fp1 - 1)];
            const int m_l = a.far4[4 * b_l + 1], ro_l = row0 - a.far4[4 * b_l], rank_l = a.meta[b_l].rank;
            const int64_t zo_l = a.z_off[b_l];
            for (int i = 0; i < min(64, (fp1 - e0 + NW - 1) / NW); ++i) {
                const int b = __builtin_amdgcn_readlane(b_l, i), m = __builtin_amdgcn_readlane(m_l, i);
                const int ro = __builtin_amdgcn_readlane(ro_l, i) + rc;
                const int rank = __builtin_amdgcn_readlane(rank_l, i);
                const XT *z = zbuf + readlane_i64(zo_l, i) + cr;
                for (int cb = 0; cb < rank; cb += 64) {
                    // first entry and first step of the crosses, a lane each
                    const int nc = min(64, rank - cb), cl = cb + min(lane, nc - 1);
                    const int64_t off_l = a.cross_off[(int64_t)b * a.rcap + cl];
                    const int rho_l = lane < nc ? a.cmeta[(int64_t)b * a.rcap + cl].rho : 0;
                    int q0_l = rho_l;   // inclusive prefix sum
#pragma unroll
                    for (int d = 1; d < 64; d <<= 1) {
                        const int v = __shfl_up(q0_l, d, 64);
                        if (lane >= d) q0_l += v;
                    }
                    const int steps = __builtin_amdgcn_readlane(q0_l, 63);
                    s_q1[wave][lane] = q0_l;
                    s_off[wave][lane] = off_l - (int64_t)(q0_l - rho_l) * m;
                    wave_sync();
                    // step s of the block's sum: cross c with s_q1[c - 1] <= s < s_q1[c]
                    int c = 0;
                    for (int s0 = qs; s0 < steps; s0 += SU * QS) {
                        const FacT *U[SU];
#pragma unroll
                        for (int u = 0; u < SU; ++u) {
                            const int s = min(s0 + u * QS, steps - 1);
                            while (s >= s_q1[wave][c]) ++c;
                            U[u] = arena + s_off[wave][c] + (int64_t)s * m + ro;
                        }
                        XT uv[SU], zv[SU][RC];
#pragma unroll
                        for (int u = 0; u < SU; ++u) {
                            const bool ok = s0 + u * QS < steps;
                            const XT *zp = z + (int64_t)min(s0 + u * QS, steps - 1) * nr;
                            uv[u] = cast_c<XT>(*U[u]);
#pragma unroll
                            for (int v = 0; v < RC; ++v) zv[u][v] = cr + v < nr ? zp[v] : czero<XT>();
                            if (!ok) {
                                uv[u] = czero<XT>();
#pragma unroll
                                for (int v = 0; v < RC; ++v) zv[u][v] = czero<XT>();
                            }
                        }
#pragma unroll
                        for (int u = 0; u < SU; ++u)
#pragma unroll
                            for (int v = 0; v < RC; ++v) acc[v] = cfma(uv[u], zv[u][v], acc[v]);
                    }
                    z += (int64_t)steps * nr;
                    wave_sync();   // the next crosses take the same place
                }
            }
        }
#pragma unroll
        for (int v = 0; v < RC; ++v) part[wave * QS + qs][r][v] = acc[v];
        __syncthreads();
        for (int t = tid; t < RL * RC; t += 512) {
            const int rr = t / RC, v = t - rr * RC;
            if (rr < lm && cr + v < nr) {
                XT s = Yn[(int64_t)(row0 + rr) * nr + cr + v];
                for (int w = 0; w < NW * QS; ++w) s = cadd(s, part[w][rr][v]);
                Y[a.perm[row0 + rr] * nr + cr + v] = s;
            }
        }
        __syncthreads();   // the next columns' sums take the same place
    }
}

// PER_FREQ.  The far blocks are products with L nrhs columns and run on the matrix cores
// (16 x 16 x 4 tiles; a complex product is four real ones), FP64 for complex128, FP32 for
// complex64:
//   Z_b = diag(f) W_b^T X[tau]  (sum_rho x n) . (n x L nrhs), row (l, q) scaled by f_l[k],
//   Y[sigma] = sum_b U_b Z_b    (leaf rows x sum_rho) . (sum_rho x L nrhs);
// the near field differs from frequency to frequency and is streamed once.  What bounds it: the
// reads of Z and the factors from L2 (a wave's operands come straight from there, four K steps
// in flight), the near field from HBM.  1728-triangle cube, L = 32, 3 right-hand sides: 1.1 ms, the
// near field 0.23 of it at 4 TB/s (one thread per element of Z and Y with strided reads: 7.8 ms).
// Z_b: a wave per 32 rows x 16 columns; the workgroup's waves take neighbouring columns, its
// blockIdx.z every gridDim.z-th group of 32 rows
template <class FacT, class XT>
__global__ void __launch_bounds__(256) apply_freq_z_kernel(ApplyDev a, const XT *Xp, XT *zbuf) {
    constexpr int KS = 4;   // K steps of 4 with their loads in flight together
    __shared__ int64_t s_w[256];
    __shared__ int s_row[257];
    const int b = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int m = a.far4[4 * b + 1], c0 = a.far4[4 * b + 2], n = a.far4[4 * b + 3];
    const int rank = a.meta[b].rank, sr = a.meta[b].sum_rho, L = a.L, nr = a.nrhs, NC = L * nr;
    if (blockIdx.z * 32 >= sr) return;
    for (int c = tid; c < rank; c += 256) {
        const int rho = a.cmeta[(int64_t)b * a.rcap + c].rho;
        s_w[c] = a.cross_off[(int64_t)b * a.rcap + c] + (int64_t)rho * m;
        s_row[c + 1] = rho;
    }
    __syncthreads();
    if (tid == 0) {
        s_row[0] = 0;
        for (int c = 0; c < rank; ++c) s_row[c + 1] += s_row[c];
    }
    __syncthreads();
    const int kq = lane >> 4;
    const FacT *arena = reinterpret_cast<const FacT *>(a.arena);
    const double2 *F = a.fib_arena + a.fib_off[b];
    XT *z = zbuf + a.z_off[b];
    // groups of 64 columns blockIdx.y, + gridDim.y, ...; no barrier below
    for (int64_t cg = (int64_t)blockIdx.y * 64 + wave * 16; cg < NC; cg += (int64_t)gridDim.y * 64) {
        const int col = (int)cg + (lane & 15);
        const bool cok = col < NC;
        const int lf = (cok ? col : 0) / nr;
        const XT *x = Xp + ((int64_t)lf * a.M + c0) * nr + ((cok ? col : 0) - lf * nr);
        for (int q0 = blockIdx.z * 32; q0 < sr; q0 += 32 * gridDim.z) {
            const FacT *w[2];
            bool rok[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int q = q0 + 16 * h + (lane & 15), qc = min(q, sr - 1);
                int c = 0;
                while (s_row[c + 1] <= qc) ++c;
                w[h] = arena + s_w[c] + (int64_t)(qc - s_row[c]) * n;
                rok[h] = q < sr;
            }
            CTile16<XT> acc[2];
            for (int k0 = 0; k0 < n; k0 += 4 * KS) {
                XT av[2][KS], bv[KS];
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    const int k = k0 + 4 * s + kq, kc = min(k, n - 1);
                    const bool ok = k < n;
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        av[h][s] = cast_c<XT>(w[h][kc]);
                        if (!(ok && rok[h])) av[h][s] = czero<XT>();
                    }
                    bv[s] = x[(int64_t)kc * nr];
                    if (!(ok && cok)) bv[s] = czero<XT>();
                }
#pragma unroll
                for (int s = 0; s < KS; ++s)
#pragma unroll
                    for (int h = 0; h < 2; ++h) acc[h].mac(av[h][s], bv[s]);
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int q = q0 + 16 * h + Mma<XT>::row(lane, t);
                    if (cok && q < sr) {
                        int c = 0;
                        while (s_row[c + 1] <= q) ++c;
                        z[(int64_t)q * NC + col] = cmul(cast_c<XT>(F[(int64_t)c * L + lf]), acc[h].get(t));
                    }
                }
        }
    }
}

// Far part of the rows of one leaf (32 of them), 16 columns: the four waves take every fourth far
// block, their sums are added in order
template <class FacT, class XT>
__global__ void __launch_bounds__(256) apply_freq_far_kernel(ApplyDev a, const XT *zbuf, XT *Yp) {
    constexpr int KS = 4;
    __shared__ XT part[4][32][16];
    const int leaf = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int lm = min(32, a.leaf_m[leaf] - 32 * (int)blockIdx.z), row0 = a.leaf_r0[leaf] + 32 * blockIdx.z;
    if (lm <= 0) return;
    const int L = a.L, nr = a.nrhs, NC = L * nr, kq = lane >> 4;
    const FacT *arena = reinterpret_cast<const FacT *>(a.arena);
    const int fp1 = a.leaf_far_ptr[leaf + 1];
    for (int ct = blockIdx.y; ct < (NC + 15) / 16; ct += gridDim.y) {
        const int col = ct * 16 + (lane & 15), cc = min(col, NC - 1);
        CTile16<XT> acc[2];
        for (int e = a.leaf_far_ptr[leaf] + wave; e < fp1; e += 4) {
            const int b = a.leaf_far_idx[e], m = a.far4[4 * b + 1], ro = row0 - a.far4[4 * b];
            const int rank = a.meta[b].rank;
            const XT *z = zbuf + a.z_off[b] + cc;
            for (int cb = 0; cb < rank; cb += 64) {
                // the crosses' offsets and ranks, a lane each
                const int cl = min(cb + lane, rank - 1);
                const int64_t off_l = a.cross_off[(int64_t)b * a.rcap + cl];
                const int rho_l = a.cmeta[(int64_t)b * a.rcap + cl].rho;
                for (int c = 0; c < min(64, rank - cb); ++c) {
                    const int rho = __shfl(rho_l, c, 64);
                    const FacT *U = arena + __shfl((long long)off_l, c, 64) + ro;
                    for (int k0 = 0; k0 < rho; k0 += 4 * KS) {
                        XT av[2][KS], bv[KS];
#pragma unroll
                        for (int s = 0; s < KS; ++s) {
                            const int k = k0 + 4 * s + kq, kc = min(k, rho - 1);
#pragma unroll
                            for (int h = 0; h < 2; ++h) {
                                const int r = 16 * h + (lane & 15);
                                av[h][s] = cast_c<XT>(U[(int64_t)kc * m + min(r, lm - 1)]);
                                if (k >= rho || r >= lm) av[h][s] = czero<XT>();
                            }
                            bv[s] = z[(int64_t)kc * NC];
                            if (k >= rho || col >= NC) bv[s] = czero<XT>();
                        }
#pragma unroll
                        for (int s = 0; s < KS; ++s)
                            if (k0 + 4 * s < rho)
#pragma unroll
                                for (int h = 0; h < 2; ++h) acc[h].mac(av[h][s], bv[s]);
                    }
                    z += (int64_t)rho * NC;
                }
            }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int t = 0; t < 4; ++t) part[wave][16 * h + Mma<XT>::row(lane, t)][lane & 15] = acc[h].get(t);
        __syncthreads();
        for (int t = tid; t < 32 * 16; t += 256) {
            const int r = t >> 4, c = ct * 16 + (t & 15);
            if (r < lm && c < NC) {
                const int lf = c / nr;
                Yp[((int64_t)lf * a.M + row0 + r) * nr + c - lf * nr] =
                    cadd(cadd(part[0][r][t & 15], part[1][r][t & 15]), cadd(part[2][r][t & 15], part[3][r][t & 15]));
            }
        }
        __syncthreads();   // the next columns' sums take the same place
    }
}

// Near part of four rows per wave at eight frequencies (8 lanes each), added to the far part in Yp
// (if there is one) and written in the caller's order.  A near row's entries of one frequency are
// contiguous over the columns.
template <class NearT, class XT, int RC>
__global__ void __launch_bounds__(256) apply_freq_near_kernel(ApplyDev a, const XT *Xp, const XT *Yp, XT *Y) {
    constexpr int RW = 4;
    const int leaf = blockIdx.x, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int lm = a.leaf_m[leaf], r0 = 16 * (int)blockIdx.z + RW * wave;
    if (r0 >= lm) return;   // the whole wave; no barrier below
    const int L = a.L, nr = a.nrhs, sub = lane & 7, lf = 8 * (int)blockIdx.y + (lane >> 3), lc = min(lf, L - 1);
    const int64_t M = a.M;
    const NearT *nearv = a.near64 ? reinterpret_cast<const NearT *>(a.near64)
                                  : reinterpret_cast<const NearT *>(a.near32);
    int row[RW];
#pragma unroll
    for (int r = 0; r < RW; ++r) row[r] = a.leaf_r0[leaf] + min(r0 + r, lm - 1);
    for (int cr = 0; cr < nr; cr += RC) {
        XT acc[RW][RC];
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int c = 0; c < RC; ++c) acc[r][c] = czero<XT>();
        for (int e = a.leaf_near_ptr[leaf]; e < a.leaf_near_ptr[leaf + 1]; ++e) {
            const NearBlockDev nb = a.nblocks[a.leaf_near_idx[e]];
            const int n = nb.n;
            const XT *x = Xp + ((int64_t)lc * M + nb.c0) * nr + cr;
            auto add = [&](int j, const XT (&nv)[RW]) {
#pragma unroll
                for (int c = 0; c < RC; ++c) {
                    const XT xv = cr + c < nr ? x[(int64_t)j * nr + c] : czero<XT>();
#pragma unroll
                    for (int r = 0; r < RW; ++r) acc[r][c] = cfma(nv[r], xv, acc[r][c]);
                }
            };
            if (nb.comp) {   // sum_l f_l[k] H_l
                const NearT *fc = reinterpret_cast<const NearT *>(a.near_faces) + nb.off;
                const int mn = nb.m * n;
                for (int j = sub; j < n; j += 8) {
                    XT nv[RW];
#pragma unroll
                    for (int r = 0; r < RW; ++r) nv[r] = czero<XT>();
                    for (int l = 0; l < nb.crank; ++l) {
                        const XT f = cast_c<XT>(a.near_fib[nb.foff + (int64_t)l * L + lc]);
#pragma unroll
                        for (int r = 0; r < RW; ++r)
                            nv[r] = cfma(cast_c<XT>(fc[(int64_t)l * mn + (int64_t)(row[r] - nb.r0) * n + j]), f, nv[r]);
                    }
                    add(j, nv);
                }
                continue;
            }
            const NearT *base = nearv + nb.off + (int64_t)lc * n;
#pragma unroll 2
            for (int j = sub; j < n; j += 8) {
                XT nv[RW];
#pragma unroll
                for (int r = 0; r < RW; ++r) nv[r] = cast_c<XT>(base[(int64_t)(row[r] - nb.r0) * L * n + j]);
                add(j, nv);
            }
        }
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int c = 0; c < RC; ++c) {
                double vx = acc[r][c].x, vy = acc[r][c].y;
                vx += dpp_d<0xB1>(vx);
                vy += dpp_d<0xB1>(vy);
                vx += dpp_d<0x4E>(vx);
                vy += dpp_d<0x4E>(vy);
                vx += dpp_d<0x141>(vx);
                vy += dpp_d<0x141>(vy);
                if (sub == r && lf < L && r0 + r < lm && cr + c < nr) {
                    XT v;
                    v.x = vx;
                    v.y = vy;
                    if (a.nfar > 0) v = cadd(v, Yp[((int64_t)lf * M + row[r]) * nr + cr + c]);
                    Y[((int64_t)lf * M + a.perm[row[r]]) * nr + cr + c] = v;
                }
            }
    }
}

template <class FacT, class XT, int RC>
static void launch_freq_near(const ApplyDev &a, const XT *Xp, const XT *Yp, XT *Y, hipStream_t st) {
    const dim3 grid(a.nleaf, (a.L + 7) / 8, (a.max_leaf_m + 15) / 16);
    apply_freq_near_kernel<FacT, XT, RC><<<grid, 256, 0, st>>>(a, Xp, Yp, Y);
}

template <class FacT, class XT, int RC>
static void launch_sum(const ApplyDev &a, const XT *Xp, XT *zbuf, XT *Yn, const XT *tn,
                       XT *Y, hipStream_t st) {
    const int64_t nwg = a.nfar + (int64_t)a.nleaf * ((a.max_leaf_m + 3) / 4);
    apply_sum_parts_kernel<FacT, XT, RC><<<(unsigned)nwg, 256, 0, st>>>(a, Xp, zbuf, Yn, tn);
    // 16 rows at a time where no leaf has more
    if (a.max_leaf_m <= 16)
        apply_sum_rows_kernel<FacT, XT, RC, 16><<<dim3(a.nleaf, 1), 512, 0, st>>>(a, zbuf, Yn, Y);
    else
        apply_sum_rows_kernel<FacT, XT, RC, 32>
            <<<dim3(a.nleaf, (a.max_leaf_m + 31) / 32), 512, 0, st>>>(a, zbuf, Yn, Y);
}

template <class FacT, class XT>
static void apply_impl(const ApplyDev &a, int mode, const XT *X, XT *Y, XT *Xp, XT *Yp, XT *zbuf,
                       hipStream_t st, XT *tnbuf) {
    const int64_t totx = (int64_t)a.L * a.M * a.nrhs;
    permute_x_kernel<XT><<<(unsigned)((totx + 255) / 256), 256, 0, st>>>(X, Xp, a.perm, a.L, a.M,
                                                                          a.nrhs);
    if (mode == 0) {
        if (a.near_faces && a.nnear > 0)
            apply_near_t_kernel<XT><<<a.nnear, 256, 0, st>>>(a, Xp, tnbuf);
        if (a.nrhs == 1) launch_sum<FacT, XT, 1>(a, Xp, zbuf, Yp, tnbuf, Y, st);
        else if (a.nrhs == 2) launch_sum<FacT, XT, 2>(a, Xp, zbuf, Yp, tnbuf, Y, st);
        else launch_sum<FacT, XT, 4>(a, Xp, zbuf, Yp, tnbuf, Y, st);
        return;
    }
    if (a.nfar > 0) {
        const unsigned nc = (unsigned)(a.L * a.nrhs);
        apply_freq_z_kernel<FacT, XT><<<dim3(a.nfar, std::min((nc + 63) / 64, 65535u), 4), 256, 0, st>>>(a, Xp, zbuf);
        apply_freq_far_kernel<FacT, XT>
            <<<dim3(a.nleaf, std::min((nc + 15) / 16, 65535u), (a.max_leaf_m + 31) / 32), 256, 0, st>>>(a, zbuf, Yp);
    }
    if (a.nrhs == 1) launch_freq_near<FacT, XT, 1>(a, Xp, Yp, Y, st);
    else if (a.nrhs == 2) launch_freq_near<FacT, XT, 2>(a, Xp, Yp, Y, st);
    else launch_freq_near<FacT, XT, 4>(a, Xp, Yp, Y, st);
}

void launch_apply(const ApplyDev &a, int mode, int x_fp32, const void *X, void *Y, void *Xp,
                  void *Yp, void *zbuf, hipStream_t st, void *tnbuf) {
#define GACA_APPLY(FT, XTT)                                                                  \
    apply_impl<FT, XTT>(a, mode, (const XTT *)X, (XTT *)Y, (XTT *)Xp, (XTT *)Yp, (XTT *)zbuf, \
                        st, (XTT *)tnbuf)
    if (a.fac_fp32) {
        if (x_fp32) GACA_APPLY(float2, float2);
        else GACA_APPLY(float2, double2);
    } else {
        if (x_fp32) GACA_APPLY(double2, float2);
        else GACA_APPLY(double2, double2);
    }
#undef GACA_APPLY
}

}  // namespace gaca
