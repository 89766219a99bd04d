// Lowest eigenpair of the Lanczos tridiagonal T_k (FP64), shared by the
// single-problem and the batched Lanczos kernels; one work group of kTriBlock
// threads per matrix.
//
// T_k has diagonal a[0..k-1] and off-diagonal e[1..k-1] (e[0] = 0).  Its
// lowest eigenvalue comes from multisection: each round evaluates T_k - x I at
// kTriBlock points of the bracket and keeps the piece in which it stops being
// positive definite.  The test at one point is the three-term recurrence of
// the leading principal minors,
//     p_i = (a_i - x) p_{i-1} - e_i^2 p_{i-2}
// (x lies above the lowest eigenvalue exactly when some p_i < 0), with the
// pair (p_{i-1}, p_i) rescaled by a power of two every kTriBatch steps: one
// multiply-add on the serial chain per step.  The pivots q_i = p_i / p_{i-1}
// obey q_i = (a_i - x) - e_i^2 / q_{i-1}, nine dependent operations a step
// with a refined hardware reciprocal; with them a solve took 40 us on average
// over k = 1..100.
//
// The eigenvector comes from three steps of inverse iteration with a shift
// just below the bracket, so T_k - sigma I is positive definite and its
// LDL^T factorisation needs no pivoting; its pivots are ratios of the same
// minors, divided by all threads at once.
#pragma once

#include <hip/hip_runtime.h>

namespace pdz {

constexpr int kTriBlock = 256;
constexpr int kTriBatch = 8;

// LDS of one solve of order at most N.
template <int N>
struct TriShared {
    double2 ae[N];       // scaled a_i and e_i^2
    double e[N + 1];     // scaled e_i (e[k] = 0)
    double2 pp[N];       // (p_{i-1}, p_i) at the shift, then (e_i / pivot_{i-1}, 1 / pivot_i)
    double z[N];         // eigenvector
    double red[kTriBlock / 64], red2[kTriBlock / 64];
    int first[2][kTriBlock / 64];
    double nrm;
};

// Minors of T - x I from i = 1 on: calls f(i, p_{i-1}, p_i); both values of a
// call carry the same scale.  Operands are read a batch ahead of their use.
template <typename F>
__device__ __forceinline__ void tri_minors(const double2* ae, int k, double x, F&& f) {
    double p2 = 1.0, p1 = ae[0].x - x;
    f(0, p2, p1);
    auto step = [&](int i, double2 q) {
        const double p = fma(q.x - x, p1, -(q.y * p2));
        p2 = p1;
        p1 = p;
        f(i, p2, p1);
    };
    int i = 1;
    double2 cur[kTriBatch];
    if (i + kTriBatch <= k)
#pragma unroll
        for (int j = 0; j < kTriBatch; ++j) cur[j] = ae[i + j];
    while (i + kTriBatch <= k) {
        const int n = i + kTriBatch;
        double2 nxt[kTriBatch];
        if (n + kTriBatch <= k)
#pragma unroll
            for (int j = 0; j < kTriBatch; ++j) nxt[j] = ae[n + j];
#pragma unroll
        for (int j = 0; j < kTriBatch; ++j) step(i + j, cur[j]);
        const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(p1), fabs(p2)));
        p1 = __builtin_amdgcn_ldexp(p1, ex);
        p2 = __builtin_amdgcn_ldexp(p2, ex);
#pragma unroll
        for (int j = 0; j < kTriBatch; ++j) cur[j] = nxt[j];
        i = n;
    }
    for (; i < k; ++i) step(i, ae[i]);
}

// Whether T - x I has a negative eigenvalue.
__device__ __forceinline__ bool tri_below(const double2* ae, int k, double x) {
    bool neg = false;
    tri_minors(ae, k, x, [&](int, double, double p) { neg = neg || p < 0.0; });
    return neg;
}

// Index of the first thread of the group for which b holds (kTriBlock: none);
// `round` alternates the LDS slot, so one barrier per call is enough.
template <int N>
__device__ __forceinline__ int tri_first(TriShared<N>& S, bool b, int round) {
    const unsigned long long m = __ballot(b);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) S.first[round & 1][wave] = m ? 64 * wave + __ffsll(m) - 1 : kTriBlock;
    __syncthreads();
    int t = kTriBlock;
    for (int w = 0; w < kTriBlock / 64; ++w) t = min(t, S.first[round & 1][w]);
    return t;
}

// Whole work group: the lowest eigenpair.  alpha[0..k-1], beta[1..k-1] in
// global memory; returns theta to every thread, the normalised eigenvector in
// S.z.  A hint [hint_lo, hint_hi] (hint_lo < hint_hi) replaces the Gershgorin
// interval when its ends test as below and above the lowest eigenvalue.  In
// Lanczos the previous Ritz value bounds the new one from above (Cauchy
// interlacing), and the last change estimates how far it moves.
template <int N>
__device__ __forceinline__ double tridiag_min_pair(TriShared<N>& S, const double* alpha, const double* beta, int k, double hint_lo,
                                   double hint_hi) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // ---- scale by a power of two so that no entry exceeds one
    double mx = 0.0;
    for (int i = tid; i < k; i += kTriBlock) {
        const double a = alpha[i], e = i == 0 ? 0.0 : beta[i];
        S.ae[i].x = a;
        S.e[i] = e;
        mx = fmax(mx, fmax(fabs(a), fabs(e)));
    }
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) mx = fmax(mx, __shfl_xor(mx, m));
    if (lane == 0) S.red[wave] = mx;
    __syncthreads();
    for (int w = 0; w < kTriBlock / 64; ++w) mx = fmax(mx, S.red[w]);
    const int ex = mx > 0.0 && mx < 1e308 ? __builtin_amdgcn_frexp_exp(mx) : 0;
    for (int i = tid; i < k; i += kTriBlock) {
        const double e = __builtin_amdgcn_ldexp(S.e[i], -ex);
        S.e[i] = e;
        S.ae[i] = double2{__builtin_amdgcn_ldexp(S.ae[i].x, -ex), e * e};
    }
    if (tid == 0) S.e[k] = 0.0;
    __syncthreads();
    // ---- bracket
    double lo = __builtin_amdgcn_ldexp(hint_lo, -ex), hi = __builtin_amdgcn_ldexp(hint_hi, -ex);
    int round = 0;
    bool have = false;
    if (lo < hi) {
        const double w = (hi - lo) / (double)(kTriBlock - 1);
        auto point = [&](int t) { return t == kTriBlock - 1 ? hi : lo + w * (double)t; };
        const int t = tri_first(S, tri_below(S.ae, k, point(tid)), round++);
        have = t > 0 && t < kTriBlock;
        if (have) {
            const double l = point(t - 1), h = point(t);
            lo = l;
            hi = h;
        }
    }
    if (!have) {
        double l = 1e300, h = -1e300;
        for (int i = tid; i < k; i += kTriBlock) {
            const double r = fabs(S.e[i]) + fabs(S.e[i + 1]);
            l = fmin(l, S.ae[i].x - r);
            h = fmax(h, S.ae[i].x + r);
        }
#pragma unroll
        for (int m = 32; m > 0; m >>= 1) {
            l = fmin(l, __shfl_xor(l, m));
            h = fmax(h, __shfl_xor(h, m));
        }
        __syncthreads();
        if (lane == 0) {
            S.red[wave] = l;
            S.red2[wave] = h;
        }
        __syncthreads();
        for (int w = 0; w < kTriBlock / 64; ++w) {
            l = fmin(l, S.red[w]);
            h = fmax(h, S.red2[w]);
        }
        const double pad = 1e-12 * fmax(__builtin_amdgcn_ldexp(1.0, -ex), fmax(fabs(l), fabs(h)));
        lo = l - pad;
        hi = h + pad;
    }
    for (int r = 0; r < 64; ++r) {
        if (!(hi - lo > 2.0 * 2.220446049250313e-16 * fmax(fabs(lo), fabs(hi)) + 1e-300)) break;
        const double w = (hi - lo) / (double)(kTriBlock + 1);
        const int t = tri_first(S, tri_below(S.ae, k, lo + w * (double)(tid + 1)), round++);
        const double l = t == 0 ? lo : lo + w * (double)t;
        const double h = t == kTriBlock ? hi : lo + w * (double)(t + 1);
        lo = l;
        hi = h;
    }
    // ---- eigenvector: T - sigma I = L D L^T, sigma just below the bracket
    const double sigma = lo - 4.0 * 2.220446049250313e-16 * fmax(__builtin_amdgcn_ldexp(1.0, -ex), fabs(lo));
    if (tid == 0) tri_minors(S.ae, k, sigma, [&](int i, double p2, double p1) { S.pp[i] = double2{p2, p1}; });
    __syncthreads();
    // reciprocal pivots r_i, then the sweep factors: forward m_i = e_i r_{i-1}, backward r_i and r_i e_{i+1}
    for (int i = tid; i < k; i += kTriBlock) {
        double2 q = S.pp[i];
        if (fabs(q.y) < 1e-300) q.y = q.y < 0.0 ? -1e-300 : 1e-300;
        S.z[i] = q.x / q.y;
    }
    __syncthreads();
    for (int i = tid; i < k; i += kTriBlock) S.pp[i] = double2{i > 0 ? S.e[i] * S.z[i - 1] : 0.0, S.z[i]};
    __syncthreads();
    if (tid == 0) {
        constexpr int B = kTriBatch;
        double scale = 1.0, nrm = 0.0;
        for (int it = 0; it < 3; ++it) {
            // L y = z (forward; the first z is all ones), then D L^T x = y (backward); x overwrites z
            double c = 0.0;
            int i = 0;
            for (; i + B <= k; i += B) {
                double zv[B], mv[B];
#pragma unroll
                for (int j = 0; j < B; ++j) {
                    zv[j] = it == 0 ? 1.0 : S.z[i + j] * scale;
                    mv[j] = S.pp[i + j].x;
                }
#pragma unroll
                for (int j = 0; j < B; ++j) {
                    c = fma(-mv[j], c, zv[j]);
                    zv[j] = c;
                }
#pragma unroll
                for (int j = 0; j < B; ++j) S.z[i + j] = zv[j];
            }
            for (; i < k; ++i) {
                c = fma(-S.pp[i].x, c, it == 0 ? 1.0 : S.z[i] * scale);
                S.z[i] = c;
            }
            c = 0.0;
            nrm = 0.0;
            i = k - 1;
            for (; i - B + 1 >= 0; i -= B) {   // i, i - 1, ..., i - B + 1
                double yv[B], ev[B];
#pragma unroll
                for (int j = 0; j < B; ++j) {
                    const double rv = S.pp[i - j].y;
                    yv[j] = rv * S.z[i - j];
                    ev[j] = rv * S.e[i - j + 1];
                }
#pragma unroll
                for (int j = 0; j < B; ++j) {
                    c = fma(-ev[j], c, yv[j]);
                    yv[j] = c;
                    nrm = fma(c, c, nrm);
                }
#pragma unroll
                for (int j = 0; j < B; ++j) S.z[i - j] = yv[j];
            }
            for (; i >= 0; --i) {
                const double rv = S.pp[i].y;
                c = fma(-(rv * S.e[i + 1]), c, rv * S.z[i]);
                S.z[i] = c;
                nrm = fma(c, c, nrm);
            }
            nrm = sqrt(nrm);
            if (!(nrm > 0.0) || !isfinite(nrm)) {
                nrm = 1.0;
                break;
            }
            scale = 1.0 / nrm;
        }
        S.nrm = 1.0 / nrm;
    }
    __syncthreads();
    const double inv = S.nrm;
    for (int i = tid; i < k; i += kTriBlock) S.z[i] *= inv;
    __syncthreads();
    return __builtin_amdgcn_ldexp(0.5 * (lo + hi), ex);
}

// Bracket hint for lambda_min(T_k) from the Ritz values of the two previous
// steps: the new value lies below theta1 (interlacing; the pad covers the
// rounding of theta1) and, once the iteration settles, within a few times the
// last change of it.
__device__ inline void ritz_hint(double theta1, double theta2, double* lo, double* hi) {
    const double scale = fmax(1.0, fabs(theta1));
    const double w = fmax(8.0 * fabs(theta1 - theta2), 1e-12 * scale);
    *hi = theta1 + 8.0 * 2.220446049250313e-16 * scale;
    *lo = theta1 - w;
}

// ---- Ritz pairs of a block of Lanczos steps at once.
//
// Only the stopping test needs a step's Ritz pair, so for vectors whose step is
// short the solves of kRitzBlock steps run side by side after the block, one
// work group per step, instead of one between every two steps; the steps past
// the first that meets the test are dropped.  Step t of a block is step
// ctl->k + t of the run: ctl->k stays what it was until ritz_block_end.
constexpr int kRitzBlock = 12;

// Work group t of the block: the pair of T_k, k = ctl->k + t + 1.  bk1 =
// beta[k]; theta, resid: Ritz values and residuals beta[k] |s_k| by step.  No
// hint from earlier steps: which of them are known depends on where the blocks
// lie, and the last bits of the bracket on the hint.
template <int N, typename C>
__device__ __forceinline__ void ritz_block_step(TriShared<N>& S, const C* ctl, int t, const double* alpha,
                                                const double* beta, double bk1, double* theta, double* resid) {
    const int k = ctl->k + t + 1;
    const double th = tridiag_min_pair(S, alpha, beta, k, 0.0, 0.0);
    if (threadIdx.x == 0) {
        theta[k - 1] = th;
        resid[k - 1] = fabs(bk1 * S.z[k - 1]);
    }
}

// One thread: the steps of the block in turn, up to the first that ends the run.
template <typename C>
__device__ __forceinline__ void ritz_block_end(C* ctl, int steps, const double* alpha, const double* beta,
                                               const double* theta, const double* resid, double tol, int max_iter,
                                               uint32_t* err, uint32_t nonfinite) {
    const int k0 = ctl->k;
    for (int k = k0 + 1; k <= k0 + steps && k <= max_iter; ++k) {
        const double th = theta[k - 1], rs = resid[k - 1], bk1 = beta[k];
        ctl->theta = th;
        ctl->resid = rs;
        ctl->k = k;
        const bool breakdown = !(bk1 > 1e-14 * fmax(1.0, fabs(th)));
        bool done = k >= max_iter;
        if (!isfinite(th) || !isfinite(bk1) || !isfinite(alpha[k - 1])) {
            atomicOr(err, nonfinite);
            done = true;
        }
        if (breakdown || rs <= tol * fmax(fabs(th), 1e-300)) {
            ctl->converged = 1;
            ctl->breakdown = breakdown ? 1 : 0;
            done = true;
        }
        if (done) {
            ctl->done = 1;
            break;
        }
    }
}

}  // namespace pdz
