// Flexible GMRES (the paper's outer solver, Section 4.3) with FP64 Arnoldi on the device and a
// preconditioner slot: identity, diagonal (the paper's indirect-BEM choice: a constant added to
// the diagonal), or the exact inverse of the operator restricted to each octree leaf.
//
// Arnoldi uses classical Gram-Schmidt with a second pass when the first one cancelled most of the
// new vector (norm drop below 1/sqrt(2), the Daniel-Gragg-Kaufman-Stewart test): each pass is one
// batched set of inner products (two-stage, fixed-order reductions, so runs are bitwise
// reproducible) and one batched update, coefficients and the test kept on the device.  Givens
// rotations and the small least-squares problem live on the host; one short copy per step.
#include <chrono>
#include <functional>
#include <type_traits>

#include "internal.h"

namespace fmm {

constexpr int DOT_BLOCKS = 512;

// Krylov vectors are stored as double2 or (mixed-precision solves) float2; every inner product and
// update is computed in FP64.
__device__ inline double2 ldc(const double2 *p, int64_t i) { return p[i]; }
__device__ inline double2 ldc(const float2 *p, int64_t i) {
    const float2 v = p[i];
    return make_double2(v.x, v.y);
}
__device__ inline void stc(double2 *p, int64_t i, double2 v) { p[i] = v; }
__device__ inline void stc(float2 *p, int64_t i, double2 v) { p[i] = make_float2((float)v.x, (float)v.y); }

// sum of the workgroup's 256 values, halving the range each step (valid in thread 0)
__device__ inline double2 sum_workgroup(double2 s) {
    __shared__ double2 red[256];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int q = blockDim.x / 2; q > 0; q >>= 1) {
        if ((int)threadIdx.x < q) red[threadIdx.x] = cadd(red[threadIdx.x], red[threadIdx.x + q]);
        __syncthreads();
    }
    return red[0];
}

// partial[blk] = sum_{i in blk's stride} |w[i]|^2
__global__ void __launch_bounds__(256) k_norm_partial(int64_t n, const double2 *w, double2 *partial) {
    double2 s = cmk(0, 0);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        s = cadd(s, cmulc(w[i], w[i]));
    s = sum_workgroup(s);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// sum of nblk partial sums over the workgroup, in a fixed order (valid in thread 0)
__device__ inline double2 sum_partials(int nblk, const double2 *partial) {
    double2 s = cmk(0, 0);
    for (int i = threadIdx.x; i < nblk; i += blockDim.x) s = cadd(s, partial[i]);
    return sum_workgroup(s);
}

__global__ void __launch_bounds__(256) k_norm_final(int nblk, const double2 *partial, double2 *out) {
    const double2 s = sum_partials(nblk, partial);
    if (threadIdx.x == 0) *out = s;
}

// One Gram-Schmidt step of up to GS_MAX systems, w against their V_0 .. V_{nv-1}: eight launches
// (inner products, their sums, update, norm; twice) for all systems, then the next basis vector, with no
// word from the host in between.  Results of a system, at res (m: the restart length):
//   [0, m]                first-pass inner products
//   [m + 1, 2 m + 1]      second-pass ones (where there was a second pass)
//   2 m + 2, 3, 4         |w|^2 before, after the first pass, after the second (.x)
//   2 m + 5               .x: 1 if the second pass is taken
// The second pass's launches end at once where it is not.  Bound by launches and the one copy for small
// n, by reading V for large n.  Measured against a host decision after every norm (five copies and host
// waits per step for one system, four for a lock-step group): a solve of 2,664 elements in 27 steps
// 8.4 -> 6.1 ms, four of 90,972 elements in lock step with FP32 bases 60.6 -> 53.2 ms.
// Vectors of at most GS_FEW partial sums (FEW): the kernels that need a sum add it up themselves, in every
// workgroup, so that a step is five launches instead of nine (2,664 elements, 27 steps: its kernels 1.12 ->
// 0.71 ms, the solve 3 % less; the line: N = 8,192, where every workgroup reads 32 sums a vector); with
// more, every workgroup would read the whole array of partial sums.
constexpr int GS_MAX = 4, GS_FEW = 32, GS_FEW_NV = 256;
constexpr int DOT_G = 8;
template <class S>
struct GsSys {
    const S *V;
    S *Vnext;  // V_nv: w / |w|
    double2 *w, *res, *part;
    int nv;
};
template <class S>
struct GsArgs {
    GsSys<S> s[GS_MAX];
};
constexpr int gs_len(int m) { return 2 * m + 6; }
// FEW: sum of nblk partial sums, by every thread
__device__ inline double2 sum_few(int nblk, const double2 *partial) {
    double2 s = cmk(0, 0);
#pragma unroll 4
    for (int i = 0; i < nblk; ++i) s = cadd(s, partial[i]);
    return s;
}
// the choice of a second pass: reorth 1 where the first removed most of w (|w| fell below
// |w_0| / sqrt(2)), 2 always, 0 never
__device__ inline bool gs_second(int reorth, double w0sq, double hsq) {
    return reorth == 2 || (reorth == 1 && !(sqrt(fmax(hsq, 0.0)) > 0.7071067811865476 * sqrt(fmax(w0sq, 0.0))));
}

// partial[v * gridDim.x + blk] = sum_{i in blk's stride} conj(V_v[i]) w[i], v < nv, and in the first pass of
// |w|^2 (v = nv).  A workgroup takes DOT_G vectors (blockIdx.y group): each element of w it loads serves
// all of them, so w is read nv / DOT_G times rather than nv times (with FP32 Krylov vectors, w's 16 bytes
// per element would otherwise be twice the vector's own 8).  The
// update's partial sums of |w|^2 are at part + (FEW ? nv + 1 : 0) gridDim.x.
template <class S, bool FEW>
__global__ void __launch_bounds__(256) k_gs_dots(int64_t n, int m, int pass, int reorth, GsArgs<S> A) {
    const GsSys<S> q = A.s[blockIdx.z];
    if (FEW && pass) {
        const double2 h = sum_few(gridDim.x, q.part + (int64_t)(q.nv + 1) * gridDim.x);
        const bool second = gs_second(reorth, q.res[2 * m + 2].x, h.x);
        if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
            q.res[2 * m + 3] = q.res[2 * m + 4] = h;
            q.res[2 * m + 5] = cmk(second ? 1.0 : 0.0, 0.0);
        }
        if (!second) return;
    } else if (pass && q.res[2 * m + 5].x == 0.0) {
        return;
    }
    const int v0 = blockIdx.y * DOT_G, all = q.nv + (pass == 0), ng = min(DOT_G, all - v0);
    if (ng <= 0) return;
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, di = (int64_t)gridDim.x * blockDim.x;
    double2 s[DOT_G];
#pragma unroll
    for (int g = 0; g < DOT_G; ++g) s[g] = cmk(0, 0);
    if (v0 + DOT_G <= q.nv) {
        // whole group: the DOT_G loads of a row are issued before any of them is used
        for (int64_t i = i0; i < n; i += di) {
            const double2 wi = q.w[i];
            double2 x[DOT_G];
#pragma unroll
            for (int g = 0; g < DOT_G; ++g) x[g] = ldc(q.V + (int64_t)(v0 + g) * n, i);
#pragma unroll
            for (int g = 0; g < DOT_G; ++g) s[g] = cadd(s[g], cmulc(wi, x[g]));  // conj(V_v) w
        }
    } else {
        for (int64_t i = i0; i < n; i += di) {
            const double2 wi = q.w[i];
#pragma unroll
            for (int g = 0; g < DOT_G; ++g)
                if (g < ng) s[g] = cadd(s[g], cmulc(wi, v0 + g < q.nv ? ldc(q.V + (int64_t)(v0 + g) * n, i) : wi));
        }
    }
    __shared__ double2 red[DOT_G][256];
#pragma unroll
    for (int g = 0; g < DOT_G; ++g) red[g][threadIdx.x] = s[g];
    __syncthreads();
    for (int h = blockDim.x / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h)
#pragma unroll
            for (int g = 0; g < DOT_G; ++g) red[g][threadIdx.x] = cadd(red[g][threadIdx.x], red[g][threadIdx.x + h]);
        __syncthreads();
    }
    if ((int)threadIdx.x < ng) q.part[(int64_t)(v0 + threadIdx.x) * gridDim.x + blockIdx.x] = red[threadIdx.x][0];
}

template <class S>
__global__ void __launch_bounds__(256) k_gs_final(int nblk, int m, int pass, GsArgs<S> A) {
    const GsSys<S> q = A.s[blockIdx.y];
    const int v = blockIdx.x;
    if (v >= q.nv + (pass == 0) || (pass && q.res[2 * m + 5].x == 0.0)) return;
    const double2 s = sum_partials(nblk, q.part + (int64_t)v * nblk);
    if (threadIdx.x == 0) q.res[v == q.nv ? 2 * m + 2 : pass * (m + 1) + v] = s;
}

// w -= sum_v h[v] V_v, in the order of v, and the partial sums of the new |w|^2; vectors are read
// COMBO_U at a time, all loads of a group issued before the group's updates (one load per iteration
// would leave one 1 KB request in flight per wavefront)
constexpr int COMBO_U = 8;
template <class S, bool FEW>
__global__ void __launch_bounds__(256) k_gs_update(int64_t n, int m, int pass, GsArgs<S> A) {
    const GsSys<S> q = A.s[blockIdx.y];
    if (pass && q.res[2 * m + 5].x == 0.0) return;
    __shared__ double2 hs[FEW ? GS_FEW_NV : 1];
    if (FEW) {
        const int all = q.nv + (pass == 0);
        if ((int)threadIdx.x < all) {
            const int v = threadIdx.x;
            const double2 d = sum_few(gridDim.x, q.part + (int64_t)v * gridDim.x);
            hs[v] = d;
            if (blockIdx.x == 0) q.res[v == q.nv ? 2 * m + 2 : pass * (m + 1) + v] = d;
        }
        __syncthreads();
    }
    const double2 *h = FEW ? hs : q.res + pass * (m + 1);
    double2 d = cmk(0, 0);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        double2 s = q.w[i];
        int v = 0;
        for (; v + COMBO_U <= q.nv; v += COMBO_U) {
            double2 x[COMBO_U];
#pragma unroll
            for (int u = 0; u < COMBO_U; ++u) x[u] = ldc(q.V, (int64_t)(v + u) * n + i);
#pragma unroll
            for (int u = 0; u < COMBO_U; ++u) s = csub(s, cmul(h[v + u], x[u]));
        }
        for (; v < q.nv; ++v) s = csub(s, cmul(h[v], ldc(q.V, (int64_t)v * n + i)));
        q.w[i] = s;
        d = cadd(d, cmulc(s, s));
    }
    d = sum_workgroup(d);
    if (threadIdx.x == 0) q.part[(FEW ? (int64_t)(q.nv + 1) * gridDim.x : 0) + blockIdx.x] = d;
}

// |w|^2 after the pass and, after the first, the choice of a second one
template <class S>
__global__ void __launch_bounds__(256) k_gs_norm(int nblk, int m, int pass, int reorth, GsArgs<S> A) {
    const GsSys<S> q = A.s[blockIdx.x];
    if (pass && q.res[2 * m + 5].x == 0.0) return;
    const double2 s = sum_partials(nblk, q.part);
    if (threadIdx.x != 0) return;
    q.res[2 * m + 3 + pass] = s;
    if (pass) return;
    q.res[2 * m + 4] = s;
    q.res[2 * m + 5] = cmk(gs_second(reorth, q.res[2 * m + 2].x, s.x) ? 1.0 : 0.0, 0.0);
}

// the next basis vector w / |w| (left alone where |w| is 0 or not a number: the host ends the cycle)
template <class S, bool FEW>
__global__ void __launch_bounds__(256) k_gs_next(int64_t n, int m, int nblk, int reorth, GsArgs<S> A) {
    const GsSys<S> q = A.s[blockIdx.y];
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double h2;
    if (FEW && (reorth == 0 || q.res[2 * m + 5].x != 0.0)) {  // the last update's norm is not summed yet
        const double2 s = sum_few(nblk, q.part + (int64_t)(q.nv + 1) * nblk);
        h2 = s.x;
        if (i == 0) {
            q.res[2 * m + 4] = s;
            if (reorth == 0) {
                q.res[2 * m + 3] = s;
                q.res[2 * m + 5] = cmk(0.0, 0.0);
            }
        }
    } else {
        h2 = q.res[2 * m + 4].x;
    }
    const double hn = sqrt(fmax(h2, 0.0));
    if (i < n && hn > 0.0) stc(q.Vnext, i, cscale(q.w[i], 1.0 / hn));
}

// the whole step, enqueued
template <class S>
static void gs_step(int64_t n, int m, int nsys, int reorth, const GsArgs<S> &A, hipStream_t st) {
    int nv = 0;
    for (int k = 0; k < nsys; ++k) nv = std::max(nv, A.s[k].nv);
    const int nblk = (int)std::min<int64_t>(DOT_BLOCKS, std::max<int64_t>(1, (n + 255) / 256));
    const bool few = nblk <= GS_FEW && nv < GS_FEW_NV;
    for (int pass = 0; pass < (reorth == 0 ? 1 : 2); ++pass) {
        const dim3 gd(nblk, ceil_div(nv + (pass == 0), DOT_G), nsys), gu(nblk, nsys);
        if (few) {
            k_gs_dots<S, true><<<gd, 256, 0, st>>>(n, m, pass, reorth, A);
            LAUNCH_OK();
            k_gs_update<S, true><<<gu, 256, 0, st>>>(n, m, pass, A);
            LAUNCH_OK();
            continue;
        }
        k_gs_dots<S, false><<<gd, 256, 0, st>>>(n, m, pass, reorth, A);
        LAUNCH_OK();
        k_gs_final<S><<<dim3(nv + (pass == 0), nsys), 256, 0, st>>>(nblk, m, pass, A);
        LAUNCH_OK();
        k_gs_update<S, false><<<gu, 256, 0, st>>>(n, m, pass, A);
        LAUNCH_OK();
        k_gs_norm<S><<<nsys, 256, 0, st>>>(nblk, m, pass, reorth, A);
        LAUNCH_OK();
    }
    const dim3 gn(ceil_div(n, 256), nsys);
    if (few) k_gs_next<S, true><<<gn, 256, 0, st>>>(n, m, nblk, reorth, A);
    else k_gs_next<S, false><<<gn, 256, 0, st>>>(n, m, nblk, reorth, A);
    LAUNCH_OK();
}

// x += sum_v y[v] Z_v (same grouping)
template <class S>
__global__ void k_add_combo(int64_t n, const S *Z, int64_t ldz, int nv, const double2 *y, double2 *x) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double2 s = x[i];
    int v = 0;
    for (; v + COMBO_U <= nv; v += COMBO_U) {
        double2 z[COMBO_U];
#pragma unroll
        for (int u = 0; u < COMBO_U; ++u) z[u] = ldc(Z, (int64_t)(v + u) * ldz + i);
#pragma unroll
        for (int u = 0; u < COMBO_U; ++u) s = cadd(s, cmul(y[v + u], z[u]));
    }
    for (; v < nv; ++v) s = cadd(s, cmul(y[v], ldc(Z, (int64_t)v * ldz + i)));
    x[i] = s;
}

// y = a x (stored in y's type)
template <class S>
__global__ void k_scale_copy(int64_t n, double a, const double2 *x, S *y) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) stc(y, i, cscale(x[i], a));
}

template <class S>
__global__ void k_widen(int64_t n, const S *x, double2 *y) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) y[i] = ldc(x, i);
}

__global__ void k_sub(int64_t n, const double2 *a, const double2 *b, double2 *out) {  // out = a - b
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = csub(a[i], b[i]);
}

__global__ void k_mul_diag(int64_t n, const double2 *d, const double2 *v, double2 *z) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) z[i] = cmul(d[i], v[i]);
}

// ------------------------------------------------------------------ preconditioners
// inverse diagonal, caller order: 1 / (1/2 + M_ii - i k beta_i L_ii + shift)
__global__ void k_diag_inv(int64_t n, const int32_t *perm, const int32_t *near_start, const int32_t *near_col,
                           const double2 *nL, const double2 *nM, const double2 *beta, double k, double shift,
                           double2 *dinv) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double2 a = cmk(0.5 + shift, 0.0);
    for (int e = near_start[i]; e < near_start[i + 1]; ++e)
        if (near_col[e] == i) {
            double2 ikb = cmk(-k * beta[i].y, k * beta[i].x);
            a = cadd(a, csub(nM[e], cmul(ikb, nL[e])));
        }
    dinv[perm[i]] = cdiv(cmk(1, 0), a);
}

// inverse diagonal of the combined (Burton-Miller) direct operator, caller order:
//   1/2 + shift + (alpha i k / 2) beta_i + M_ii - i k beta_i L_ii + alpha (M'_ii - i k beta_i L'_ii)
__global__ void k_diag_bm_inv(int64_t n, const int32_t *perm, const int32_t *near_start, const int32_t *near_col,
                              const double2 *nL, const double2 *nM, const double2 *nLp, const double2 *nMp,
                              const double2 *beta, double k, double2 alpha, double shift, double2 *dinv) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double2 ikb = cscale(cmuli(beta[i]), k);
    double2 a = cadd(cmk(0.5 + shift, 0.0), cscale(cmul(alpha, ikb), 0.5));
    for (int e = near_start[i]; e < near_start[i + 1]; ++e)
        if (near_col[e] == i) {
            a = cadd(a, csub(nM[e], cmul(ikb, nL[e])));
            a = cadd(a, cmul(alpha, csub(nMp[e], cmul(ikb, nLp[e]))));
        }
    dinv[perm[i]] = cdiv(cmk(1, 0), a);
}

// dense operator block of each leaf, row-major n_b x n_b at blk_off[b] (sorted element order)
__global__ void __launch_bounds__(256) k_leaf_blocks(int nleaf, const int32_t *leaf_start, const int64_t *blk_off,
                                                     const double4 *ec, const double4 *en, const double2 *beta,
                                                     double k, double rc2, const int32_t *near_start,
                                                     const int32_t *near_col, const double2 *nL, const double2 *nM,
                                                     double2 *A) {
    const int b = blockIdx.x;
    const int s = leaf_start[b], nb = leaf_start[b + 1] - s;
    double2 *Ab = A + blk_off[b];
    const double inv4pi = 1.0 / (4.0 * FMM_PI);
    for (int e = threadIdx.x; e < nb * nb; e += blockDim.x) {
        int i = s + e / nb, j = s + e % nb;
        double4 ci = ec[i], cj = ec[j];
        double d2 = dist2_exact(ci.x, ci.y, ci.z, cj.x, cj.y, cj.z);
        double2 v = cmk(0, 0);
        if (i != j && d2 >= rc2) {
            double4 nj = en[j];
            double r = sqrt(d2), sn, cs;
            sincos(k * r, &sn, &cs);
            double2 G = cmk(cs / r * inv4pi * cj.w, sn / r * inv4pi * cj.w);  // A_j G
            double u = ((cj.x - ci.x) * nj.x + (cj.y - ci.y) * nj.y + (cj.z - ci.z) * nj.z) / d2;
            double2 M = cmul(G, cmk(-u, k * r * u));
            double2 ikb = cmk(-k * beta[j].y, k * beta[j].x);
            v = csub(M, cmul(ikb, G));
        }
        if (i == j) v.x += 0.5;
        Ab[e] = v;
    }
    __syncthreads();
    for (int r = threadIdx.x; r < nb; r += blockDim.x) {
        int i = s + r;
        for (int e = near_start[i]; e < near_start[i + 1]; ++e) {
            int j = near_col[e];
            if (j < s || j >= s + nb) continue;
            double2 ikb = cmk(-k * beta[j].y, k * beta[j].x);
            Ab[(int64_t)r * nb + (j - s)] = cadd(Ab[(int64_t)r * nb + (j - s)], csub(nM[e], cmul(ikb, nL[e])));
        }
    }
}

// dense block of the indirect operator (Eq. ibem5) on each leaf's unknowns, row-major
// 2 n_b x 2 n_b at blk_off[b]: rows (psi- equation of the leaf's elements, then psi+ equation),
// columns (psi- of the leaf's elements, then psi+), elements in sorted order.  With
// sigma_j = -i k (beta-_j psi-_j + beta+_j psi+_j) and mu_j = psi-_j - psi+_j, the equations are
//   V_i + (psi-_i + psi+_i) / 2                            (V = sum_j L_ij sigma_j + M_ij mu_j)
//   W_i + i k (beta-_i psi-_i - beta+_i psi+_i) / 2        (W = sum_j L'_ij sigma_j + M'_ij mu_j)
// the pair entries L, M, L', M' from the near tables where |c_i - c_j| < r_c, from the one-point
// rule of the near field elsewhere.
__global__ void __launch_bounds__(256) k_leaf_blocks_ind(int nleaf, const int32_t *leaf_start, const int64_t *blk_off,
                                                         const double4 *ec, const double4 *en, const double2 *bm,
                                                         const double2 *bp, double k, double rc2,
                                                         const int32_t *near_start, const int32_t *near_col,
                                                         const double2 *nL, const double2 *nM, const double2 *nLp,
                                                         const double2 *nMp, double2 *A) {
    const int b = blockIdx.x;
    const int s = leaf_start[b], nb = leaf_start[b + 1] - s, n2 = 2 * nb;
    double2 *Ab = A + blk_off[b];
    const double inv4pi = 1.0 / (4.0 * FMM_PI);
    // the four entries of pair (i, j) into the 2 x 2 sub-block (rows i, i + nb; columns j, j + nb)
    auto put = [&](int r, int q, double2 L, double2 M, double2 Lp, double2 Mp, bool add) {
        const int j = s + q;
        const double2 ikm = cscale(cmuli(bm[j]), k), ikp = cscale(cmuli(bp[j]), k);  // i k beta-+_j
        const double2 e00 = csub(M, cmul(ikm, L)), e01 = csub(cscale(M, -1.0), cmul(ikp, L));
        const double2 e10 = csub(Mp, cmul(ikm, Lp)), e11 = csub(cscale(Mp, -1.0), cmul(ikp, Lp));
        double2 *r0 = Ab + (int64_t)r * n2, *r1 = Ab + (int64_t)(r + nb) * n2;
        if (add) {
            r0[q] = cadd(r0[q], e00);
            r0[q + nb] = cadd(r0[q + nb], e01);
            r1[q] = cadd(r1[q], e10);
            r1[q + nb] = cadd(r1[q + nb], e11);
        } else {
            r0[q] = e00;
            r0[q + nb] = e01;
            r1[q] = e10;
            r1[q + nb] = e11;
        }
    };
    for (int e = threadIdx.x; e < nb * nb; e += blockDim.x) {
        const int r = e / nb, q = e % nb, i = s + r, j = s + q;
        const double4 ci = ec[i], cj = ec[j];
        const double d2 = dist2_exact(ci.x, ci.y, ci.z, cj.x, cj.y, cj.z);
        double2 L = cmk(0, 0), M = L, Lp = L, Mp = L;
        if (i != j && d2 >= rc2) {
            const double4 ni = en[i], nj = en[j];
            const double dx = cj.x - ci.x, dy = cj.y - ci.y, dz = cj.z - ci.z;
            const double r1 = sqrt(d2), ir = 1.0 / r1, ir2 = ir * ir;
            double sn, cs;
            sincos(k * r1, &sn, &cs);
            const double2 E = cmk(cs * inv4pi * cj.w, sn * inv4pi * cj.w);  // A_j e^{ikr} / 4 pi
            const double2 G = cscale(E, ir);
            const double dny = dx * nj.x + dy * nj.y + dz * nj.z, dnx = dx * ni.x + dy * ni.y + dz * ni.z;
            const double nn = ni.x * nj.x + ni.y * nj.y + ni.z * nj.z;
            const double2 g1 = cmul(G, cmk(-1.0, k * r1));  // G (ikr - 1)
            L = G;
            M = cscale(g1, dny * ir2);
            Lp = cscale(g1, -dnx * ir2);
            const double2 k3 = cmul(E, cmk(3.0 - k * k * d2, -3.0 * k * r1));
            Mp = csub(cscale(k3, -dnx * dny * ir2 * ir2 * ir), cscale(cmul(E, cmk(-1.0, k * r1)), nn * ir2 * ir));
        }
        put(r, q, L, M, Lp, Mp, false);
    }
    __syncthreads();
    // near-table entries (each row's entries belong to one thread: no two threads touch one row)
    for (int r = threadIdx.x; r < nb; r += blockDim.x) {
        const int i = s + r;
        for (int e = near_start[i]; e < near_start[i + 1]; ++e) {
            const int j = near_col[e];
            if (j < s || j >= s + nb) continue;
            put(r, j - s, nL[e], nM[e], nLp[e], nMp[e], true);
        }
        // local terms
        const double2 ikm = cscale(cmuli(bm[i]), k), ikp = cscale(cmuli(bp[i]), k);
        double2 *r0 = Ab + (int64_t)r * n2, *r1 = Ab + (int64_t)(r + nb) * n2;
        r0[r] = cadd(r0[r], cmk(0.5, 0.0));
        r0[r + nb] = cadd(r0[r + nb], cmk(0.5, 0.0));
        r1[r] = cadd(r1[r], cscale(ikm, 0.5));
        r1[r + nb] = cadd(r1[r + nb], cscale(ikp, -0.5));
    }
}

// dense block of the combined (Burton-Miller) direct operator on each leaf, row-major n_b x n_b:
//   1/2 delta_ij + (alpha i k / 2) beta_i delta_ij + M_ij - i k beta_j L_ij + alpha (M'_ij - i k beta_j L'_ij)
// pair entries from the near tables or the near field's one-point rule, as for the indirect blocks
__global__ void __launch_bounds__(256) k_leaf_blocks_bm(int nleaf, const int32_t *leaf_start, const int64_t *blk_off,
                                                        const double4 *ec, const double4 *en, const double2 *beta,
                                                        double k, double2 alpha, double rc2, const int32_t *near_start,
                                                        const int32_t *near_col, const double2 *nL, const double2 *nM,
                                                        const double2 *nLp, const double2 *nMp, double2 *A) {
    const int b = blockIdx.x;
    const int s = leaf_start[b], nb = leaf_start[b + 1] - s;
    double2 *Ab = A + blk_off[b];
    const double inv4pi = 1.0 / (4.0 * FMM_PI);
    auto entry = [&](int j, double2 L, double2 M, double2 Lp, double2 Mp) {
        const double2 ikb = cscale(cmuli(beta[j]), k);
        return cadd(csub(M, cmul(ikb, L)), cmul(alpha, csub(Mp, cmul(ikb, Lp))));
    };
    for (int e = threadIdx.x; e < nb * nb; e += blockDim.x) {
        const int r = e / nb, q = e % nb, i = s + r, j = s + q;
        const double4 ci = ec[i], cj = ec[j];
        const double d2 = dist2_exact(ci.x, ci.y, ci.z, cj.x, cj.y, cj.z);
        double2 v = cmk(0, 0);
        if (i != j && d2 >= rc2) {
            const double4 ni = en[i], nj = en[j];
            const double dx = cj.x - ci.x, dy = cj.y - ci.y, dz = cj.z - ci.z;
            const double r1 = sqrt(d2), ir = 1.0 / r1, ir2 = ir * ir;
            double sn, cs;
            sincos(k * r1, &sn, &cs);
            const double2 E = cmk(cs * inv4pi * cj.w, sn * inv4pi * cj.w);  // A_j e^{ikr} / 4 pi
            const double2 G = cscale(E, ir);
            const double dny = dx * nj.x + dy * nj.y + dz * nj.z, dnx = dx * ni.x + dy * ni.y + dz * ni.z;
            const double nn = ni.x * nj.x + ni.y * nj.y + ni.z * nj.z;
            const double2 g1 = cmul(G, cmk(-1.0, k * r1));  // G (ikr - 1)
            const double2 k3 = cmul(E, cmk(3.0 - k * k * d2, -3.0 * k * r1));
            const double2 Mp =
                csub(cscale(k3, -dnx * dny * ir2 * ir2 * ir), cscale(cmul(E, cmk(-1.0, k * r1)), nn * ir2 * ir));
            v = entry(j, G, cscale(g1, dny * ir2), cscale(g1, -dnx * ir2), Mp);
        }
        Ab[e] = v;
    }
    __syncthreads();
    for (int r = threadIdx.x; r < nb; r += blockDim.x) {
        const int i = s + r;
        for (int e = near_start[i]; e < near_start[i + 1]; ++e) {
            const int j = near_col[e];
            if (j < s || j >= s + nb) continue;
            Ab[(int64_t)r * nb + (j - s)] = cadd(Ab[(int64_t)r * nb + (j - s)], entry(j, nL[e], nM[e], nLp[e], nMp[e]));
        }
        const double2 ikb = cscale(cmuli(beta[i]), k);
        Ab[(int64_t)r * nb + r] = cadd(Ab[(int64_t)r * nb + r], cadd(cmk(0.5, 0.0), cscale(cmul(alpha, ikb), 0.5)));
    }
}

// in-place Gauss-Jordan inversion with partial pivoting, one workgroup per leaf block
// (block dimension m n_b: m unknowns per element; at most 1024)
__global__ void __launch_bounds__(256) k_leaf_invert(int nleaf, const int32_t *leaf_start, const int64_t *blk_off,
                                                     double2 *A, int32_t *piv_ws, int *status, int m) {
    const int b = blockIdx.x;
    const int nb = m * (leaf_start[b + 1] - leaf_start[b]);
    double2 *M = A + blk_off[b];
    int32_t *piv = piv_ws + (int64_t)m * leaf_start[b];
    __shared__ int sp;
    __shared__ double sbest[256];
    __shared__ int sidx[256];
    __shared__ double2 prow[1024];
    for (int c = 0; c < nb; ++c) {
        // pivot search in column c, rows c..nb-1
        double best = -1.0;
        int bi = c;
        for (int r = c + threadIdx.x; r < nb; r += blockDim.x) {
            double2 v = M[(int64_t)r * nb + c];
            double a = v.x * v.x + v.y * v.y;
            if (a > best) {
                best = a;
                bi = r;
            }
        }
        sbest[threadIdx.x] = best;
        sidx[threadIdx.x] = bi;
        __syncthreads();
        if (threadIdx.x == 0) {
            double bb = -1.0;
            int ii = c;
            for (int t = 0; t < (int)blockDim.x; ++t)
                if (sbest[t] > bb) {
                    bb = sbest[t];
                    ii = sidx[t];
                }
            sp = ii;
            piv[c] = ii;
            if (!(bb > 0.0)) atomicExch(status, 1);
        }
        __syncthreads();
        const int pr = sp;
        if (pr != c)
            for (int q = threadIdx.x; q < nb; q += blockDim.x) {
                double2 t = M[(int64_t)c * nb + q];
                M[(int64_t)c * nb + q] = M[(int64_t)pr * nb + q];
                M[(int64_t)pr * nb + q] = t;
            }
        __syncthreads();
        const double2 pv = M[(int64_t)c * nb + c];
        const double2 ipv = cdiv(cmk(1, 0), pv);
        // scale pivot row: row c <- row c / pv, with the inverse's column c set to 1/pv
        for (int q = threadIdx.x; q < nb; q += blockDim.x) {
            double2 v = (q == c) ? cmk(1, 0) : M[(int64_t)c * nb + q];
            prow[q] = cmul(v, ipv);
        }
        __syncthreads();
        for (int q = threadIdx.x; q < nb; q += blockDim.x) M[(int64_t)c * nb + q] = prow[q];
        __syncthreads();
        // eliminate column c from every other row (each thread owns whole rows)
        for (int r = threadIdx.x; r < nb; r += blockDim.x) {
            if (r == c) continue;
            double2 f = M[(int64_t)r * nb + c];
            for (int q = 0; q < nb; ++q) {
                double2 v = (q == c) ? cmk(0, 0) : M[(int64_t)r * nb + q];
                M[(int64_t)r * nb + q] = csub(v, cmul(f, prow[q]));
            }
        }
        __syncthreads();
    }
    // undo the column permutation implied by the row swaps (in reverse order)
    for (int c = nb - 1; c >= 0; --c) {
        const int pr = piv[c];
        if (pr != c)
            for (int r = threadIdx.x; r < nb; r += blockDim.x) {
                double2 t = M[(int64_t)r * nb + c];
                M[(int64_t)r * nb + c] = M[(int64_t)r * nb + pr];
                M[(int64_t)r * nb + pr] = t;
            }
        __syncthreads();
    }
}

// z = blockdiag(A_BB^{-1}) v, vectors in caller order; m unknowns per element (block index
// q of element s + (q mod n_b) is unknown (q / n_b) n + perm[s + q mod n_b])
__global__ void __launch_bounds__(128) k_leaf_apply(int nleaf, const int32_t *leaf_start, const int64_t *blk_off,
                                                    const double2 *Ainv, const int32_t *perm, const double2 *v,
                                                    double2 *z, int m, int64_t n) {
    const int b = blockIdx.x;
    const int s = leaf_start[b], ne = leaf_start[b + 1] - s, nb = m * ne;
    const double2 *M = Ainv + blk_off[b];
    __shared__ double2 vs[1024];
    auto idx = [&](int q) -> int64_t { return (int64_t)(q / ne) * n + perm[s + q % ne]; };
    for (int q = threadIdx.x; q < nb; q += blockDim.x) vs[q] = v[idx(q)];
    __syncthreads();
    for (int r = threadIdx.x; r < nb; r += blockDim.x) {
        double2 acc = cmk(0, 0);
        for (int q = 0; q < nb; ++q) acc = cfma(M[(int64_t)r * nb + q], vs[q], acc);
        z[idx(r)] = acc;
    }
}

// ------------------------------------------------------------------ host helpers
struct Blas {
    hipStream_t st;
    DeviceBuffers &scr;
    int64_t n;
    std::string tag;  // scratch-name prefix, so nested solves keep separate buffers
    double nrm(const double2 *w) {
        double2 *part = dget<double2>(scr, tag + "dot_part", DOT_BLOCKS), *res = dget<double2>(scr, tag + "dot_res", 1);
        const int nblk = (int)std::min<int64_t>(DOT_BLOCKS, std::max<int64_t>(1, (n + 255) / 256));
        k_norm_partial<<<nblk, 256, 0, st>>>(n, w, part);
        LAUNCH_OK();
        k_norm_final<<<1, 256, 0, st>>>(nblk, part, res);
        LAUNCH_OK();
        double2 d;
        HIP_OK(hipMemcpyAsync(&d, res, sizeof(double2), hipMemcpyDeviceToHost, st));
        HIP_OK(hipStreamSynchronize(st));
        return sqrt(std::max(d.x, 0.0));
    }
    template <class S>
    void add_combo(const S *Z, int64_t ldz, int nv, const double2 *y_host, double2 *x) {
        double2 *h = dget<double2>(scr, tag + "combo_y", std::max(nv, 1));
        HIP_OK(hipMemcpyAsync(h, y_host, sizeof(double2) * nv, hipMemcpyHostToDevice, st));
        k_add_combo<S><<<ceil_div(n, 256), 256, 0, st>>>(n, Z, ldz, nv, h, x);
        LAUNCH_OK();
    }
    template <class S>
    void scale_copy(double a, const double2 *x, S *y) {
        k_scale_copy<S><<<ceil_div(n, 256), 256, 0, st>>>(n, a, x, y);
        LAUNCH_OK();
    }
    template <class S>
    void widen(const S *x, double2 *y) {
        k_widen<S><<<ceil_div(n, 256), 256, 0, st>>>(n, x, y);
        LAUNCH_OK();
    }
    void sub(const double2 *a, const double2 *b, double2 *out) {
        k_sub<<<ceil_div(n, 256), 256, 0, st>>>(n, a, b, out);
        LAUNCH_OK();
    }
};

static inline double cabs_(double2 a) { return hypot(a.x, a.y); }

// Restarted FGMRES(m).  matvec(x, y) and precond(v, z) act on device vectors of length n; the
// preconditioner may change from one call to the next (an inner solve, a learned map).
// Returns FMMBEM_OK / FMMBEM_ENOCONV / error codes.  rel_res is the true relative residual of the
// last restart, computed with `matvec_check` (the FP64 operator); with final_residual false, a
// solve that stops at maxit skips that last product and reports the Arnoldi estimate instead
// (inner solves).  history, when given, receives the estimate after every iteration.
// S: storage type of the Krylov vectors V and Z (double2, or float2 for mixed-precision solves:
// half the basis traffic; inner products, Hessenberg matrix, rotations, the iterate and the
// restart residual stay FP64).
template <class S>
static int fgmres_t(int64_t n, hipStream_t st, DeviceBuffers &scr, const char *tag,
                    const std::function<void(const double2 *, double2 *)> &matvec,
                    const std::function<void(const double2 *, double2 *)> &matvec_check,
                    const std::function<void(const double2 *, double2 *)> &precond, const double2 *b, double2 *x,
                    double tol, int m, int maxit, bool x0_given, bool final_residual, std::vector<double> *history,
                    int &iters, int &restarts, double &rel_res, const FgmresHooks *hooks, int reorth) {
    constexpr bool wide = std::is_same<S, double2>::value;
    const std::string tg(tag);
    Blas B{st, scr, n, tg};
    S *V = dget<S>(scr, tg + (wide ? "fg_V" : "fg_V32"), (size_t)(m + 1) * n);
    S *Z = dget<S>(scr, tg + (wide ? "fg_Z" : "fg_Z32"), (size_t)m * n);
    double2 *w = dget<double2>(scr, tg + "fg_w", n);
    double2 *r = dget<double2>(scr, tg + "fg_r", n);
    double2 *gsr = dget<double2>(scr, tg + "fg_gs", gs_len(m));
    double2 *gsp = dget<double2>(scr, tg + "fg_part", (size_t)DOT_BLOCKS * (m + 1));
    // FP64 copies of the current basis vector and its preconditioned image (narrow storage only)
    double2 *tv = wide ? nullptr : dget<double2>(scr, tg + "fg_tv", n);
    double2 *tz = wide ? nullptr : dget<double2>(scr, tg + "fg_tz", n);
    if (!x0_given) HIP_OK(hipMemsetAsync(x, 0, sizeof(double2) * n, st));
    const double bn = B.nrm(b);
    iters = 0;
    restarts = 0;
    rel_res = 1.0;
    if (!(bn > 0.0)) {
        HIP_OK(hipMemsetAsync(x, 0, sizeof(double2) * n, st));
        rel_res = 0.0;
        return FMMBEM_OK;
    }
    std::vector<double2> H((size_t)(m + 1) * m), g(m + 1), cs(m), sn(m), hr(gs_len(m)), y(m);
    auto Hc = [&](int i, int j) -> double2 & { return H[(size_t)i * m + j]; };
    int status = FMMBEM_ENOCONV;
    double est = 1.0;
    while (true) {
        if (!final_residual && restarts > 0 && iters >= maxit) {
            rel_res = est;
            break;
        }
        // true residual
        if (x0_given || restarts > 0) {
            matvec_check(x, w);
            B.sub(b, w, r);
        } else {
            HIP_OK(hipMemcpyAsync(r, b, sizeof(double2) * n, hipMemcpyDeviceToDevice, st));
        }
        double beta = B.nrm(r);
        rel_res = beta / bn;
        if (!std::isfinite(beta)) return FMMBEM_ENAN;
        if (hooks && hooks->on_restart) hooks->on_restart(x, r, rel_res);
        if (rel_res < tol) {
            status = FMMBEM_OK;
            break;
        }
        if (iters >= maxit) break;
        B.scale_copy(1.0 / beta, r, V);
        std::fill(g.begin(), g.end(), cmk(0, 0));
        g[0] = cmk(beta, 0);
        int j = 0;
        bool done = false;
        for (j = 0; j < m && iters < maxit; ++j) {
            S *vjs = V + (size_t)j * n, *zjs = Z + (size_t)j * n;
            const double2 *vj;
            double2 *zj;
            if constexpr (wide) {
                vj = vjs;
                zj = zjs;
            } else {
                B.widen(vjs, tv);
                vj = tv;
                zj = tz;
            }
            precond(vj, zj);
            if constexpr (!wide) B.scale_copy(1.0, zj, zjs);
            matvec(zj, w);
            ++iters;
            // classical Gram-Schmidt and the next basis vector
            GsArgs<S> ga{};
            ga.s[0] = {V, V + (size_t)(j + 1) * n, w, gsr, gsp, j + 1};
            gs_step<S>(n, m, 1, reorth, ga, st);
            HIP_OK(hipMemcpyAsync(hr.data(), gsr, sizeof(double2) * gs_len(m), hipMemcpyDeviceToHost, st));
            HIP_OK(hipStreamSynchronize(st));
            const bool second = hr[2 * m + 5].x != 0.0;
            for (int i = 0; i <= j; ++i) Hc(i, j) = second ? cadd(hr[i], hr[m + 1 + i]) : hr[i];
            const double hn = sqrt(std::max(hr[2 * m + 4].x, 0.0));
            if (!std::isfinite(hn) || !std::isfinite(hr[2 * m + 4].x)) return FMMBEM_ENAN;
            Hc(j + 1, j) = cmk(hn, 0);
            for (int i = 0; i < j; ++i) {
                double2 a = Hc(i, j), c = Hc(i + 1, j);
                Hc(i, j) = cadd(cscale(a, cs[i].x), cmul(sn[i], c));
                Hc(i + 1, j) = csub(cscale(c, cs[i].x), cmul(cconj(sn[i]), a));
            }
            double2 a = Hc(j, j), c = Hc(j + 1, j);
            double den = hypot(cabs_(a), cabs_(c));
            if (den == 0) {
                cs[j] = cmk(1, 0);
                sn[j] = cmk(0, 0);
            } else {
                double aa = cabs_(a);
                cs[j] = cmk(aa / den, 0);
                double2 ph = aa > 0 ? cscale(a, 1.0 / aa) : cmk(1, 0);
                sn[j] = cscale(cmul(ph, cconj(c)), 1.0 / den);
            }
            Hc(j, j) = cadd(cscale(a, cs[j].x), cmul(sn[j], c));
            Hc(j + 1, j) = cmk(0, 0);
            g[j + 1] = cscale(cmul(cconj(sn[j]), g[j]), -1.0);
            g[j] = cscale(g[j], cs[j].x);
            est = cabs_(g[j + 1]) / bn;
            if (history) history->push_back(est);
            if (hooks && hooks->on_iter) hooks->on_iter(iters, est);
            if (est < tol || hn == 0) {
                ++j;
                done = true;
                break;
            }
        }
        // y = H^{-1} g (upper triangular)
        for (int i = j - 1; i >= 0; --i) {
            double2 s = g[i];
            for (int q = i + 1; q < j; ++q) s = csub(s, cmul(Hc(i, q), y[q]));
            if (cabs_(Hc(i, i)) == 0) return FMMBEM_EBREAKDOWN;
            y[i] = cdiv(s, Hc(i, i));
        }
        B.add_combo(Z, n, j, y.data(), x);
        ++restarts;
        x0_given = true;
        (void)done;
    }
    return status;
}

int fgmres(int64_t n, hipStream_t st, DeviceBuffers &scr, const char *tag,
           const std::function<void(const double2 *, double2 *)> &matvec,
           const std::function<void(const double2 *, double2 *)> &matvec_check,
           const std::function<void(const double2 *, double2 *)> &precond, const double2 *b, double2 *x, double tol,
           int m, int maxit, bool x0_given, bool final_residual, std::vector<double> *history, int &iters,
           int &restarts, double &rel_res, const FgmresHooks *hooks, bool basis32, int reorth) {
    if (basis32)
        return fgmres_t<float2>(n, st, scr, tag, matvec, matvec_check, precond, b, x, tol, m, maxit, x0_given,
                                final_residual, history, iters, restarts, rel_res, hooks, reorth);
    return fgmres_t<double2>(n, st, scr, tag, matvec, matvec_check, precond, b, x, tol, m, maxit, x0_given,
                             final_residual, history, iters, restarts, rel_res, hooks, reorth);
}

// Lock-step FGMRES over groups of systems.  A group is nv systems A x_s = b_s that share one
// operator (one context: the same mesh, wavenumber and admittance, one source each): every step of
// a group gathers the preconditioned vectors of its systems still iterating and applies one batched
// product, so the kernel evaluations, basis functions and translation tables of the FMM are shared
// between them.  Each system keeps its own Krylov basis, Hessenberg matrix and restarts, exactly as
// fgmres().  Several groups (contexts of other frequencies or rooms, each with its own N, octree and
// truncation numbers) advance in turn from one host thread: a group's next product is enqueued on
// its own streams as soon as its Arnoldi step is done, and a group's Arnoldi step waits for its own
// stream only, so the products of the other groups keep the device busy meanwhile.
template <class S>
struct BatchSys {
    S *V = nullptr, *Z = nullptr;
    double2 *r = nullptr;
    std::vector<double2> H, g, cs, sn, y;
    double bn = 0.0, est = 1.0;
    int j = 0, cycle = 0;  // cycle = restarts so far
    bool in_cycle = false, done = false;
};

template <class T>
struct GroupSolver {
    static constexpr bool wide = std::is_same<T, double2>::value;
    FgmresGroup &G;
    Blas Bl;
    std::vector<BatchSys<T>> S;
    double2 *tv = nullptr, *Sin = nullptr, *Sout = nullptr;
    double2 *part = nullptr;             // partial sums of GS_MAX systems' inner products (one stream: shared)
    double2 *dres = nullptr;             // per system: the results of a Gram-Schmidt step
    double2 *dy = nullptr;               // per system: the coefficients y of x += Z y
    double2 *hres = nullptr, *hy = nullptr;  // pinned host copies
    std::vector<int> act;                // systems whose product is in flight, in Sin/Sout order
    std::vector<int> need;               // systems whose true residual is being formed
    bool pending = false;                // work enqueued whose results the host reads next
    explicit GroupSolver(FgmresGroup &g) : G(g), Bl{g.st, *g.scr, g.n, g.tag + "bt_"} {}
    ~GroupSolver() {
        if (hres) (void)hipHostFree(hres);
        if (hy) (void)hipHostFree(hy);
    }
    int RS() const { return gs_len(G.m); }  // stride of dres / hres per system
    int RN() const { return 2 * G.m + 2; }  // where a norm by itself is put
    double2 *parts(int k) { return part + (size_t)k * DOT_BLOCKS * (G.m + 1); }
    double2 *res(int s) { return dres + (size_t)s * RS(); }
    double2 *hr(int s) { return hres + (size_t)s * RS(); }

    // |w|^2 of a system, enqueued only
    void norm_to(int s, const double2 *w) {
        const int nblk = (int)std::min<int64_t>(DOT_BLOCKS, std::max<int64_t>(1, (G.n + 255) / 256));
        k_norm_partial<<<nblk, 256, 0, G.st>>>(G.n, w, part);
        LAUNCH_OK();
        k_norm_final<<<1, 256, 0, G.st>>>(nblk, part, res(s) + RN());
        LAUNCH_OK();
        to_host(s);
    }
    void to_host(int s) {  // the system's inner products and norms to the pinned copy
        HIP_OK(hipMemcpyAsync(hr(s), res(s), sizeof(double2) * RS(), hipMemcpyDeviceToHost, G.st));
        pending = true;
    }
    void wait() {
        if (pending) HIP_OK(hipStreamSynchronize(G.st));
        pending = false;
    }

    void init() {
        const int64_t n = G.n;
        const int nv = G.nv, m = G.m;
        S.assign(nv, BatchSys<T>());
        tv = wide ? nullptr : dget<double2>(*G.scr, G.tag + "bt_tv", n);
        G.iters.assign(nv, 0);
        G.restarts.assign(nv, 0);
        G.rel_res.assign(nv, 1.0);
        G.status.assign(nv, FMMBEM_ENOCONV);
        Sin = dget<double2>(*G.scr, G.tag + "bt_in", (size_t)nv * n);
        Sout = dget<double2>(*G.scr, G.tag + "bt_out", (size_t)nv * n);
        part = dget<double2>(*G.scr, G.tag + "bt_part", (size_t)std::min(nv, GS_MAX) * DOT_BLOCKS * (m + 1));
        dres = dget<double2>(*G.scr, G.tag + "bt_res", (size_t)nv * RS());
        dy = dget<double2>(*G.scr, G.tag + "bt_y", (size_t)nv * (m + 1));
        HIP_OK(hipHostMalloc((void **)&hres, sizeof(double2) * nv * RS()));
        HIP_OK(hipHostMalloc((void **)&hy, sizeof(double2) * nv * (m + 1)));
        for (int s = 0; s < nv; ++s) {
            BatchSys<T> &q = S[s];
            const std::string id = G.tag + std::to_string(s);
            q.V = dget<T>(*G.scr, (wide ? "bt_V" : "bt_V32_") + id, (size_t)(m + 1) * n);
            q.Z = dget<T>(*G.scr, (wide ? "bt_Z" : "bt_Z32_") + id, (size_t)m * n);
            q.r = dget<double2>(*G.scr, "bt_r" + id, n);
            q.H.assign((size_t)(m + 1) * m, cmk(0, 0));
            q.g.assign(m + 1, cmk(0, 0));
            q.cs.assign(m, cmk(0, 0));
            q.sn.assign(m, cmk(0, 0));
            q.y.assign(m, cmk(0, 0));
            double2 *x = G.X + (int64_t)s * n;
            if (!G.x0_given) HIP_OK(hipMemsetAsync(x, 0, sizeof(double2) * n, G.st));
            norm_to(s, G.B + (int64_t)s * n);
        }
    }
    void init_done() {
        for (int s = 0; s < G.nv; ++s) {
            BatchSys<T> &q = S[s];
            q.bn = sqrt(std::max(hr(s)[RN()].x, 0.0));
            if (!(q.bn > 0.0)) {
                HIP_OK(hipMemsetAsync(G.X + (int64_t)s * G.n, 0, sizeof(double2) * G.n, G.st));
                G.rel_res[s] = 0.0;
                G.status[s] = FMMBEM_OK;
                q.done = true;
            }
        }
    }

    // ---- restarts: systems between cycles get their true residual (one batched FP64 product)
    void restart_products() {
        const int64_t n = G.n;
        need.clear();
        std::vector<int> prod;
        for (int s = 0; s < G.nv; ++s)
            if (!S[s].done && !S[s].in_cycle) need.push_back(s);
        if (need.empty()) return;
        for (int s : need)
            if (G.x0_given || S[s].cycle > 0) prod.push_back(s);
        for (size_t k = 0; k < prod.size(); ++k)
            HIP_OK(hipMemcpyAsync(Sin + k * n, G.X + (int64_t)prod[k] * n, sizeof(double2) * n,
                                  hipMemcpyDeviceToDevice, G.st));
        if (!prod.empty()) G.matvec_check((int)prod.size(), Sin, Sout);
        for (size_t k = 0; k < prod.size(); ++k) Bl.sub(G.B + (int64_t)prod[k] * n, Sout + k * n, S[prod[k]].r);
        for (int s : need) {
            BatchSys<T> &q = S[s];
            if (!(G.x0_given || q.cycle > 0))
                HIP_OK(hipMemcpyAsync(q.r, G.B + (int64_t)s * n, sizeof(double2) * n, hipMemcpyDeviceToDevice, G.st));
            norm_to(s, q.r);
        }
    }
    void restart_decide() {
        for (int s : need) {
            BatchSys<T> &q = S[s];
            const double beta = sqrt(std::max(hr(s)[RN()].x, 0.0));
            G.rel_res[s] = beta / q.bn;
            if (!std::isfinite(beta)) {
                G.status[s] = FMMBEM_ENAN;
                q.done = true;
                continue;
            }
            if (G.rel_res[s] < G.tol) {
                G.status[s] = FMMBEM_OK;
                q.done = true;
                continue;
            }
            if (G.iters[s] >= G.maxit) {
                q.done = true;
                continue;
            }
            Bl.scale_copy(1.0 / beta, q.r, q.V);
            std::fill(q.g.begin(), q.g.end(), cmk(0, 0));
            q.g[0] = cmk(beta, 0);
            q.j = 0;
            q.in_cycle = true;
        }
        need.clear();
    }

    // ---- the next batched product of the systems in a cycle
    bool products() {
        const int64_t n = G.n;
        act.clear();
        for (int s = 0; s < G.nv; ++s)
            if (S[s].in_cycle) act.push_back(s);
        if (act.empty()) return false;
        for (size_t k = 0; k < act.size(); ++k) {
            BatchSys<T> &q = S[act[k]];
            if constexpr (wide) {
                G.precond(q.V + (size_t)q.j * n, q.Z + (size_t)q.j * n);
                HIP_OK(hipMemcpyAsync(Sin + k * n, q.Z + (size_t)q.j * n, sizeof(double2) * n,
                                      hipMemcpyDeviceToDevice, G.st));
            } else {
                Bl.widen(q.V + (size_t)q.j * n, tv);
                G.precond(tv, Sin + k * n);
                Bl.scale_copy(1.0, Sin + k * n, q.Z + (size_t)q.j * n);
            }
        }
        G.matvec((int)act.size(), Sin, Sout);
        return true;
    }

    // ---- Arnoldi step of every system in flight: Gram-Schmidt and the next basis vectors
    void gs() {
        for (size_t k0 = 0; k0 < act.size(); k0 += GS_MAX) {
            const int ns = (int)std::min<size_t>(GS_MAX, act.size() - k0);
            GsArgs<T> A{};
            for (int k = 0; k < ns; ++k) {
                const int s = act[k0 + k];
                BatchSys<T> &q = S[s];
                ++G.iters[s];
                A.s[k] = {q.V, q.V + (size_t)(q.j + 1) * G.n, Sout + (k0 + k) * G.n, res(s), parts(k), q.j + 1};
            }
            gs_step<T>(G.n, G.m, ns, G.reorth, A, G.st);
            for (int k = 0; k < ns; ++k) to_host(act[k0 + k]);
        }
    }
    // Hessenberg column and Givens rotations; at the end of a cycle x += Z y
    void gs_finish() {
        const int m = G.m;
        for (size_t k = 0; k < act.size(); ++k) {
            const int s = act[k];
            BatchSys<T> &q = S[s];
            auto Hc = [&](int i, int jj) -> double2 & { return q.H[(size_t)i * m + jj]; };
            const int j = q.j;
            const double2 *h = hr(s);
            const bool second = h[2 * m + 5].x != 0.0;
            const double hn = sqrt(std::max(h[2 * m + 4].x, 0.0));
            for (int i = 0; i <= j; ++i) Hc(i, j) = second ? cadd(h[i], h[m + 1 + i]) : h[i];
            if (!std::isfinite(hn) || !std::isfinite(h[2 * m + 4].x)) {
                G.status[s] = FMMBEM_ENAN;
                q.done = true;
                q.in_cycle = false;
                continue;
            }
            Hc(j + 1, j) = cmk(hn, 0);
            for (int i = 0; i < j; ++i) {
                double2 a = Hc(i, j), c = Hc(i + 1, j);
                Hc(i, j) = cadd(cscale(a, q.cs[i].x), cmul(q.sn[i], c));
                Hc(i + 1, j) = csub(cscale(c, q.cs[i].x), cmul(cconj(q.sn[i]), a));
            }
            double2 a = Hc(j, j), c = Hc(j + 1, j);
            const double den = hypot(cabs_(a), cabs_(c));
            if (den == 0) {
                q.cs[j] = cmk(1, 0);
                q.sn[j] = cmk(0, 0);
            } else {
                const double aa = cabs_(a);
                q.cs[j] = cmk(aa / den, 0);
                const double2 ph = aa > 0 ? cscale(a, 1.0 / aa) : cmk(1, 0);
                q.sn[j] = cscale(cmul(ph, cconj(c)), 1.0 / den);
            }
            Hc(j, j) = cadd(cscale(a, q.cs[j].x), cmul(q.sn[j], c));
            Hc(j + 1, j) = cmk(0, 0);
            q.g[j + 1] = cscale(cmul(cconj(q.sn[j]), q.g[j]), -1.0);
            q.g[j] = cscale(q.g[j], q.cs[j].x);
            q.est = cabs_(q.g[j + 1]) / q.bn;
            q.j = j + 1;
            if (q.est < G.tol || hn == 0 || q.j == m || G.iters[s] >= G.maxit) {
                // end of cycle: x += Z y with y = H^{-1} g
                const int jj = q.j;
                for (int i = jj - 1; i >= 0; --i) {
                    double2 sum = q.g[i];
                    for (int t = i + 1; t < jj; ++t) sum = csub(sum, cmul(Hc(i, t), q.y[t]));
                    if (cabs_(Hc(i, i)) == 0) throw FmmError(FMMBEM_EBREAKDOWN, "batched solver breakdown");
                    q.y[i] = cdiv(sum, Hc(i, i));
                }
                double2 *hys = hy + (size_t)s * (m + 1);
                for (int i = 0; i < jj; ++i) hys[i] = q.y[i];
                double2 *dys = dy + (size_t)s * (m + 1);
                HIP_OK(hipMemcpyAsync(dys, hys, sizeof(double2) * jj, hipMemcpyHostToDevice, G.st));
                k_add_combo<T><<<ceil_div(G.n, 256), 256, 0, G.st>>>(G.n, q.Z, G.n, jj, dys, G.X + (int64_t)s * G.n);
                LAUNCH_OK();
                q.in_cycle = false;
                ++q.cycle;
                G.restarts[s] = q.cycle;
            }
        }
        // the pinned coefficients of a cycle's end are read by the copies above before the next
        // phase that could rewrite them (a later cycle of the same system, after several waits)
    }
};

// Every phase is enqueued for all groups before the host waits for any, so one host round trip
// serves every system of every group and the groups' kernels overlap on the device.
void fgmres_groups(std::vector<FgmresGroup> &groups) {
    std::vector<GroupSolver<double2>> wide;
    std::vector<GroupSolver<float2>> narrow;
    wide.reserve(groups.size());
    narrow.reserve(groups.size());
    for (auto &g : groups) {
        if (g.basis32) narrow.emplace_back(g);
        else wide.emplace_back(g);
    }
    auto all = [&](auto &&f) {
        for (auto &g : wide) f(g);
        for (auto &g : narrow) f(g);
    };
    auto any_of = [&](auto &&f) {
        bool r = false;
        for (auto &g : wide) r = f(g) || r;
        for (auto &g : narrow) r = f(g) || r;
        return r;
    };
    auto wait_all = [&]() { all([](auto &g) { g.wait(); }); };
    all([](auto &g) { g.init(); });
    wait_all();
    all([](auto &g) { g.init_done(); });
    all([](auto &g) { g.restart_products(); });
    wait_all();
    all([](auto &g) { g.restart_decide(); });
    while (any_of([](auto &g) { return g.products(); })) {
        all([](auto &g) { g.gs(); });
        wait_all();
        all([](auto &g) { g.gs_finish(); });
        all([](auto &g) { g.restart_products(); });
        wait_all();
        all([](auto &g) { g.restart_decide(); });
    }
    wait_all();
    all([](auto &g) { HIP_OK(hipStreamSynchronize(g.G.st)); });
}

int fgmres_batch(int64_t n, hipStream_t st, DeviceBuffers &scr, int nv,
                 const std::function<void(int, const double2 *, double2 *)> &matvec,
                 const std::function<void(int, const double2 *, double2 *)> &matvec_check,
                 const std::function<void(const double2 *, double2 *)> &precond, const double2 *B, double2 *X,
                 double tol, int m, int maxit, bool x0_given, std::vector<int> &iters, std::vector<int> &restarts,
                 std::vector<double> &rel_res, std::vector<int> &status, bool basis32, int reorth) {
    std::vector<FgmresGroup> g(1);
    FgmresGroup &q = g[0];
    q.n = n;
    q.st = st;
    q.scr = &scr;
    q.nv = nv;
    q.matvec = matvec;
    q.matvec_check = matvec_check;
    q.precond = precond;
    q.B = B;
    q.X = X;
    q.tol = tol;
    q.m = m;
    q.maxit = maxit;
    q.x0_given = x0_given;
    q.basis32 = basis32;
    q.reorth = reorth;
    fgmres_groups(g);
    iters = q.iters;
    restarts = q.restarts;
    rel_res = q.rel_res;
    status = q.status;
    return FMMBEM_OK;
}

}  // namespace fmm
