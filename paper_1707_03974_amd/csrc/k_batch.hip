// Batched H.v and Lanczos over many Hubbard clusters of uneven size.
//
// The clusters' vectors are packed back to back (each at a 64-element aligned
// offset).  Work groups walk a list of tiles (cluster, group of rows), largest
// clusters first; the clusters whose rows go with it are computed by tiles of
// the single-cluster one-pass H.v (hv_rows.h), in one launch, the others element
// by element in another.  Every element is summed by one thread in the order of
// the hop tables, diagonal first, whichever form its cluster takes.
//
// Batched Lanczos runs the recurrence of k_lanczos.hip for all clusters in
// lockstep over the packed vectors, unnormalised (v_k = sc_k q_k): per step
// one H.v, which also writes the partial sums of alpha, and one update, which
// forms alpha_k, beta_k and sc_k from partial sums itself; the Ritz pairs of
// kRitzBlock steps of every cluster then run side by side (tridiag.h).  A
// converged cluster's tiles and chunks are skipped by every later kernel.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <numeric>
#include <vector>

#include "hv_rows.h"
#include "pdz_internal.h"
#include "tridiag.h"

namespace pdz {
namespace {

constexpr int kBatchMaxIter = 2000;
constexpr int kRed = 256;
constexpr uint64_t kAlign = 64;       // packed vector offsets, elements
constexpr uint64_t kChunk = 4096;     // elements per work group of the update and the reductions

struct BProb {
    uint64_t off;                 // element offset of the cluster's vector
    uint64_t D_up, D_dn;
    double U;
    const uint32_t* up_states;
    const uint32_t* dn_states;
    const uint8_t* up_count;
    const uint8_t* dn_count;
    const uint32_t* up_ell;       // 32-bit hop tables, slot major
    const uint32_t* dn_ell;
    const double* coef64;
    const float* coef32;
    int ncoef;
    int dn_max;                   // most hops out of a down state
};

struct BTile {
    uint32_t prob;
    uint32_t u0;
    uint32_t nrows;
    uint32_t pad;
};

struct BChunk {                    // reduction chunk [begin, end) of one cluster
    uint32_t prob;
    uint32_t pad;
    uint64_t begin, end;
};

struct BCtl {                      // per-cluster Lanczos state
    int k;
    int done;
    int converged;
    int breakdown;
    double theta;
    double resid;
    double norm0;
};

__global__ void k_clear_bits1(uint32_t* w, uint32_t bits) {
    if (threadIdx.x == 0 && blockIdx.x == 0) atomicAnd(w, ~bits);
}

template <typename T>
__device__ __forceinline__ const T* bcoef(const BProb& p);
template <>
__device__ __forceinline__ const double* bcoef<double>(const BProb& p) { return p.coef64; }
template <>
__device__ __forceinline__ const float* bcoef<float>(const BProb& p) { return p.coef32; }

constexpr int kBHopNB = 8;   // hops of one element whose loads are in flight together

constexpr int kBatchRV = 4;   // rows side by side in a tile of k_batch_rows

// Sum over a work group of BLOCK threads (fixed order), valid in thread 0.
template <int BLOCK>
__device__ __forceinline__ double tile_sum(double v) {
    __shared__ double ws[BLOCK / 64];
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) v += __shfl_xor(v, m);
    if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int i = 0; i < BLOCK / 64; ++i) t += ws[i];
    return t;
}

// done: per-cluster flags with stride `dstride` ints (NULL: none skipped).
// dotp: NULL, or one partial sum of x . y per tile.  One element per thread, so
// it takes rows of any length that fit the LDS: short ones, flattened over the
// tile, and those too long for four to lie side by side (rows_form).
template <typename T, int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_batch_hv(const BProb* __restrict__ probs, const BTile* __restrict__ tiles,
                                                    uint32_t ntiles, const int* done, int dstride, double* dotp,
                                                    const T* __restrict__ x, T* __restrict__ y) {
    extern __shared__ __align__(16) unsigned char smem[];
    T* coef = reinterpret_cast<T*>(smem);
    T* rows = coef + kMaxCoef;
    for (uint32_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const BTile tl = tiles[t];
        if (done && done[(size_t)tl.prob * dstride]) continue;
        const BProb pr = probs[tl.prob];
        const T* cg = bcoef<T>(pr);
        for (int k = threadIdx.x; k < pr.ncoef; k += BLOCK) coef[k] = cg[k];
        const uint64_t D_dn = pr.D_dn, D_up = pr.D_up;
        const uint32_t nelem = tl.nrows * (uint32_t)D_dn;
        const T* xp = x + pr.off;
        T* yp = y + pr.off;
        const T* xg = xp + (uint64_t)tl.u0 * D_dn;
        for (uint32_t k = threadIdx.x; k < nelem; k += BLOCK) rows[k] = xg[k];
        __syncthreads();
        const T U = (T)pr.U;
        double dsum = 0.0;
        for (uint32_t k = threadIdx.x; k < nelem; k += BLOCK) {
            const uint32_t r = k / (uint32_t)D_dn;
            const uint32_t d = k - r * (uint32_t)D_dn;
            const uint64_t u = tl.u0 + r;
            const T* xrow = rows + (size_t)r * D_dn;
            T acc = U * (T)__builtin_popcount(pr.up_states[u] & pr.dn_states[d]) * xrow[d];
            // the barriers keep the rounding of the two-pass H.v: the diagonal
            // product and the down-hop sum are rounded before the next term
            asm volatile("" : "+v"(acc));
            // hops in order, kBHopNB at a time: a batch's table entries (and, for
            // up hops, its operands) are loaded before its first multiply-add
            const int cd = pr.dn_count[d];
            int h = 0;
            for (; h + kBHopNB <= cd; h += kBHopNB) {
                uint32_t e[kBHopNB];
#pragma unroll
                for (int j = 0; j < kBHopNB; ++j) e[j] = pr.dn_ell[(uint64_t)(h + j) * D_dn + d];
#pragma unroll
                for (int j = 0; j < kBHopNB; ++j) acc += coef[e[j] >> kTargetBits] * xrow[e[j] & kTargetMask];
            }
            for (; h < cd; ++h) {
                const uint32_t e = pr.dn_ell[(uint64_t)h * D_dn + d];
                acc += coef[e >> kTargetBits] * xrow[e & kTargetMask];
            }
            asm volatile("" : "+v"(acc));
            const int cu = pr.up_count[u];
            h = 0;
            for (; h + kBHopNB <= cu; h += kBHopNB) {
                uint32_t e[kBHopNB];
                T v[kBHopNB];
#pragma unroll
                for (int j = 0; j < kBHopNB; ++j) e[j] = pr.up_ell[(uint64_t)(h + j) * D_up + u];
#pragma unroll
                for (int j = 0; j < kBHopNB; ++j) v[j] = xp[(uint64_t)(e[j] & kTargetMask) * D_dn + d];
#pragma unroll
                for (int j = 0; j < kBHopNB; ++j) acc += coef[e[j] >> kTargetBits] * v[j];
            }
            for (; h < cu; ++h) {
                const uint32_t e = pr.up_ell[(uint64_t)h * D_up + u];
                acc += coef[e >> kTargetBits] * xp[(uint64_t)(e & kTargetMask) * D_dn + d];
            }
            yp[u * D_dn + d] = acc;
            dsum += (double)xrow[d] * (double)acc;
        }
        if (dotp) {
            dsum = tile_sum<BLOCK>(dsum);
            if (threadIdx.x == 0) dotp[t] = dsum;
        }
        __syncthreads();
    }
}

// The same for clusters in the one-pass tile (four rows side by side in LDS).
// 32 clusters of the 4x3 and 3x3 tori (8.2e6 elements): 207 us FP64 with one
// element per thread and a device work queue, 108 us so (FP32 145 / 75).
template <typename T, int BLOCK>
__global__ __launch_bounds__(BLOCK, 4) void k_batch_rows(const BProb* __restrict__ probs, const BTile* __restrict__ tiles,
                                                      uint32_t ntiles, const int* done, int dstride, double* dotp,
                                                      const T* __restrict__ x, T* __restrict__ y) {
    extern __shared__ __align__(16) unsigned char smem[];
    T* coef = reinterpret_cast<T*>(smem);
    for (uint32_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const BTile tl = tiles[t];
        if (done && done[(size_t)tl.prob * dstride]) continue;
        const BProb& pr = probs[tl.prob];
        const T* cg = bcoef<T>(pr);
        for (int k = threadIdx.x; k < pr.ncoef; k += BLOCK) coef[k] = cg[k];
        RowsProb<T> rp;
        rp.D_up = pr.D_up;
        rp.D_dn = rp.pitch = pr.D_dn;
        rp.up_states = pr.up_states;
        rp.dn_states = pr.dn_states;
        rp.up_count = pr.up_count;
        rp.dn_count = pr.dn_count;
        rp.up_ell = pr.up_ell;
        rp.dn_ell = pr.dn_ell;
        rp.U = (T)pr.U;
        rp.dn_max = pr.dn_max;
        double dsum = rows_tile<T, kBatchRV, BLOCK>(rp, tl.u0, tl.nrows, coef, smem + kMaxCoef * sizeof(T), x + pr.off,
                                                    y + pr.off);
        if (dotp) {
            dsum = tile_sum<BLOCK>(dsum);
            if (threadIdx.x == 0) dotp[t] = dsum;
        }
        __syncthreads();   // the tile's LDS is rewritten by the next
    }
}

// ------------------------------------------------------------ batched Lanczos

__device__ __forceinline__ double bsum(double v, double* red) {
    red[threadIdx.x] = v;
    __syncthreads();
    for (int s = kRed / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    const double r = red[0];
    __syncthreads();
    return r;
}

// Clear two packed vectors (the padding between clusters stays zero).
template <typename T>
__global__ __launch_bounds__(kRed) void k_bzero(uint64_t total, T* a, T* b) {
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < total; i += (uint64_t)gridDim.x * blockDim.x) {
        a[i] = (T)0;
        b[i] = (T)0;
    }
}

// Start vector of cluster p: SplitMix64 stream seeded with seed + p, output r
// mapped to 2u - 1 (the single-problem start vector of that seed).
template <typename T>
__global__ __launch_bounds__(kRed) void k_bfill(const BChunk* ch, const BProb* probs, uint64_t seed, T* v) {
    const BChunk c = ch[blockIdx.x];
    const uint64_t off = probs[c.prob].off;
    for (uint64_t i = c.begin + threadIdx.x; i < c.end; i += blockDim.x)
        v[off + i] = (T)splitmix_uniform(seed + c.prob, i);
}

// partial[c] = sum over chunk c of a*b (FP64), skipped for done clusters.
template <typename T>
__global__ __launch_bounds__(kRed) void k_bdot(const BChunk* ch, const BProb* probs, const BCtl* ctl, const T* a,
                                               const T* b, double* partial) {
    __shared__ double red[kRed];
    const BChunk c = ch[blockIdx.x];
    if (ctl[c.prob].done) return;
    const uint64_t off = probs[c.prob].off;
    double acc = 0.0;
    for (uint64_t i = c.begin + threadIdx.x; i < c.end; i += blockDim.x) acc += (double)a[off + i] * (double)b[off + i];
    acc = bsum(acc, red);
    if (threadIdx.x == 0) partial[blockIdx.x] = acc;
}

// The recurrence of step k = ctl.k + koff of every live cluster (steps from kmax
// on are dropped): w = H q_k on entry, q_{k+1} on exit.  alpha_k comes from the
// cluster's tile sums of q_k . H q_k, beta_k and sc_k = 1 / beta_k from its
// chunk sums of |q_k|^2 (norms[k & 1]; sc_0 is given); each work group adds them
// itself and the cluster's first one stores them.  norms[(k + 1) & 1][c] =
// |q_{k+1}|^2 over chunk c.  One launch in place of dot, sum, update, sum and
// scale: 83 us of a step of 32 mixed clusters (FP64) became 31.
struct BStep {
    const uint32_t* tile_begin;    // first tile of each cluster, and its tile count
    const uint32_t* tile_count;
    const uint32_t* chunk_begin;
    const double* dots;
    double* norms[2];
    double *alpha, *beta, *sc;
    int ld, koff, kmax;
};
__device__ __forceinline__ double brange_sum(const double* v, uint32_t n) {
    __shared__ double ws[kRed / 64];
    double acc = 0.0;
    for (uint32_t i = threadIdx.x; i < n; i += kRed) acc += v[i];
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) acc += __shfl_xor(acc, m);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = acc;
    __syncthreads();
    return ((ws[0] + ws[1]) + ws[2]) + ws[3];
}
template <typename T>
__global__ __launch_bounds__(kRed) void k_bupdate(const BChunk* ch, const BProb* probs, const BCtl* ctl, const BStep b,
                                                  T* __restrict__ w, const T* __restrict__ q,
                                                  const T* __restrict__ qp) {
    const BChunk c = ch[blockIdx.x];
    const BCtl st = ctl[c.prob];
    const int k = st.k + b.koff;
    if (st.done || k >= b.kmax) return;
    const size_t row = (size_t)c.prob * b.ld;
    const double dot = brange_sum(b.dots + b.tile_begin[c.prob], b.tile_count[c.prob]);
    double a, cc = 0.0, bk = 0.0;
    if (k > 0) {
        const uint32_t c0 = b.chunk_begin[c.prob];
        bk = sqrt(brange_sum(b.norms[k & 1] + c0, b.chunk_begin[c.prob + 1] - c0));
        a = 1.0 / bk;
        cc = bk * b.sc[row + k - 1];
    } else {
        a = b.sc[row];
    }
    const double ak = a * a * dot, bb = ak * a;
    if (c.begin == 0 && threadIdx.x == 0) {
        b.alpha[row + k] = ak;
        if (k > 0) {
            b.beta[row + k] = bk;
            b.sc[row + k] = a;
        }
    }
    // chunks begin at multiples of 4096 of a 64-element aligned vector: 16-byte loads
    constexpr int N = 16 / sizeof(T);
    typedef T V __attribute__((ext_vector_type(N)));
    const uint64_t off = probs[c.prob].off + c.begin;
    const uint32_t n = (uint32_t)(c.end - c.begin), nv = n / N;
    V* wv = reinterpret_cast<V*>(w + off);
    const V* qv = reinterpret_cast<const V*>(q + off);
    const V* pv = reinterpret_cast<const V*>(qp + off);
    double acc = 0.0;
#pragma unroll 4
    for (uint32_t i = threadIdx.x; i < nv; i += kRed) {
        const V w0 = wv[i], q0 = qv[i], p0 = pv[i];
        V r;
#pragma unroll
        for (int e = 0; e < N; ++e) {
            r[e] = lanczos_recurrence<T>(w0[e], T(0), q0[e], p0[e], a, bb, cc);
            acc += (double)r[e] * (double)r[e];
        }
        wv[i] = r;
    }
    for (uint32_t i = nv * N + threadIdx.x; i < n; i += kRed) {
        const T r = lanczos_recurrence<T>(w[off + i], T(0), q[off + i], qp[off + i], a, bb, cc);
        w[off + i] = r;
        acc += (double)r * (double)r;
    }
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) acc += __shfl_xor(acc, m);
    __shared__ double ws[kRed / 64];
    if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) b.norms[(k + 1) & 1][blockIdx.x] = ((ws[0] + ws[1]) + ws[2]) + ws[3];
}

// v *= 1 / norm0
__global__ __launch_bounds__(kRed) void k_bscale(const BChunk* ch, const BProb* probs, const BCtl* ctl, double* v) {
    const BChunk c = ch[blockIdx.x];
    const BCtl st = ctl[c.prob];
    if (st.done) return;
    const double inv = 1.0 / st.norm0;
    const uint64_t off = probs[c.prob].off;
    for (uint64_t i = c.begin + threadIdx.x; i < c.end; i += blockDim.x) v[off + i] *= inv;
}

// One block per cluster: norm0 = sqrt of the sum of its chunk partials, and
// sc[0] = 1 / norm0 (sc != NULL).
__global__ __launch_bounds__(kRed) void k_bnorm0(const uint32_t* ch_begin, const double* partial, BCtl* ctl,
                                                 double* sc, int ld, uint32_t* err) {
    __shared__ double red[kRed];
    const uint32_t p = blockIdx.x;
    BCtl* st = ctl + p;
    if (st->done) return;
    double acc = 0.0;
    for (uint32_t c = ch_begin[p] + threadIdx.x; c < ch_begin[p + 1]; c += blockDim.x) acc += partial[c];
    acc = bsum(acc, red);
    if (threadIdx.x == 0) {
        const double v = sqrt(acc);
        st->norm0 = v;
        if (sc) sc[(size_t)p * ld] = 1.0 / v;
        if (!isfinite(v)) atomicOr(err, kErrNonFinite);
    }
}

__global__ void k_binit(BCtl* ctl, double* beta, int ld, uint32_t n) {
    const uint32_t p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    BCtl c;
    c.k = 0;
    c.done = 0;
    c.converged = 0;
    c.breakdown = 0;
    c.theta = 0.0;
    c.resid = 0.0;
    c.norm0 = 0.0;
    ctl[p] = c;
    beta[(size_t)p * ld] = 0.0;
}

// Ritz pairs of a block of steps of every cluster: work group (t, p) the pair of
// step ctl[p].k + t of cluster p (tridiag.h).
__global__ __launch_bounds__(kTriBlock) void k_britz_block(const BCtl* ctl, const uint32_t* ch_begin,
                                                           const double* norm0, const double* norm1,
                                                           const double* alpha, double* beta, double* theta,
                                                           double* resid, int ld, int max_iter) {
    const uint32_t p = blockIdx.y;
    const BCtl* st = ctl + p;
    const int k = st->k + blockIdx.x + 1;
    if (st->done || k > max_iter) return;
    __shared__ TriShared<kBatchMaxIter> S;
    const size_t row = (size_t)p * ld;
    double bk1;
    if (blockIdx.x + 1 == gridDim.x || k == max_iter) {   // no update after this step has formed beta_{k+1}: its sum
        static_assert(kTriBlock == kRed, "brange_sum's work group");
        bk1 = sqrt(brange_sum(((k & 1) ? norm1 : norm0) + ch_begin[p], ch_begin[p + 1] - ch_begin[p]));
        if (threadIdx.x == 0) beta[row + k] = bk1;
    } else {
        bk1 = beta[row + k];
    }
    ritz_block_step(S, st, (int)blockIdx.x, alpha + row, beta + row, bk1, theta + row, resid + row);
}

__global__ void k_britz_end(BCtl* ctl, uint32_t n, int steps, const double* alpha, const double* beta,
                            const double* theta, const double* resid, int ld, double tol, int max_iter, uint32_t* err) {
    const uint32_t p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n || ctl[p].done) return;
    const size_t row = (size_t)p * ld;
    ritz_block_end(ctl + p, steps, alpha + row, beta + row, theta + row, resid + row, tol, max_iter, err,
                   kErrNonFinite);
}

// Eigenvector of every cluster's last T_k into row p of svec.
__global__ __launch_bounds__(kTriBlock) void k_britz_vector(const BCtl* ctl, const double* alpha, const double* beta,
                                                            double* svec, int ld) {
    __shared__ TriShared<kBatchMaxIter> S;
    const size_t row = (size_t)blockIdx.x * ld;
    const int k = ctl[blockIdx.x].k;
    if (k < 1) return;
    tridiag_min_pair(S, alpha + row, beta + row, k, 0.0, 0.0);
    for (int i = threadIdx.x; i < k; i += blockDim.x) svec[row + i] = S.z[i];
}

// ---- FP64 refinement of the Ritz vectors (storage FP32 or FP64)

// kfin[p] = steps the run took; counters restart for the regeneration pass.
__global__ void k_bregen_init(BCtl* ctl, int* kfin, uint32_t n) {
    const uint32_t p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const int k = ctl[p].k;
    kfin[p] = k;
    ctl[p].k = 0;
    ctl[p].done = k > 0 ? 0 : 1;
}

// y += s_k sc_k q_k (FP64) for every live cluster, s = row p of svec (eigenvector of T_kfin).
template <typename T>
__global__ __launch_bounds__(kRed) void k_baxpy_ritz(const BChunk* ch, const BProb* probs, const BCtl* ctl,
                                                     const double* svec, const double* sc, int ld, const T* v,
                                                     double* y) {
    const BChunk c = ch[blockIdx.x];
    const BCtl st = ctl[c.prob];
    if (st.done) return;
    const double sk = svec[(size_t)c.prob * ld + st.k] * sc[(size_t)c.prob * ld + st.k];
    const uint64_t off = probs[c.prob].off;
    for (uint64_t i = c.begin + threadIdx.x; i < c.end; i += blockDim.x) y[off + i] += sk * (double)v[off + i];
}

// A cluster whose last Lanczos vector has been added needs no further one.
__global__ void k_bregen_mark(BCtl* ctl, const int* kfin, uint32_t n) {
    const uint32_t p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n || ctl[p].done) return;
    if (ctl[p].k + 1 >= kfin[p]) ctl[p].done = 1;
}

// q_{k+1} from w = H q_k with the stored alpha_k, beta_k and scales: the run's
// recurrence, so the vectors are the run's bit for bit.
template <typename T>
__global__ __launch_bounds__(kRed) void k_bregen_update(const BChunk* ch, const BProb* probs, const BCtl* ctl,
                                                        const double* alpha, const double* beta, const double* sc,
                                                        int ld, T* w, const T* q, const T* qp) {
    const BChunk c = ch[blockIdx.x];
    const BCtl st = ctl[c.prob];
    if (st.done) return;
    const size_t row = (size_t)c.prob * ld;
    const double a = sc[row + st.k], b = alpha[row + st.k] * a;
    const double cc = st.k > 0 ? beta[row + st.k] * sc[row + st.k - 1] : 0.0;
    const uint64_t off = probs[c.prob].off;
    for (uint64_t i = c.begin + threadIdx.x; i < c.end; i += blockDim.x)
        w[off + i] = lanczos_recurrence<T>(w[off + i], T(0), q[off + i], qp[off + i], a, b, cc);
}

__global__ void k_bregen_next(BCtl* ctl, uint32_t n) {
    const uint32_t p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n || ctl[p].done) return;
    ctl[p].k += 1;
}

// Every cluster that ran at least one step is live again.
__global__ void k_bregen_reopen(BCtl* ctl, const int* kfin, uint32_t n) {
    const uint32_t p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    ctl[p].k = 0;
    ctl[p].done = kfin[p] > 0 ? 0 : 1;
}

// out[p] = sum of the chunk partials of cluster p (sqrt when root).
__global__ __launch_bounds__(kRed) void k_bsum_out(const uint32_t* ch_begin, const double* partial, const BCtl* ctl,
                                                   double* out, int root) {
    __shared__ double red[kRed];
    const uint32_t p = blockIdx.x;
    if (ctl[p].done) return;
    double acc = 0.0;
    for (uint32_t c = ch_begin[p] + threadIdx.x; c < ch_begin[p + 1]; c += blockDim.x) acc += partial[c];
    acc = bsum(acc, red);
    if (threadIdx.x == 0) out[p] = root ? sqrt(acc) : acc;
}

// partial[c] = |hy - E_p y|^2 over chunk c.
__global__ __launch_bounds__(kRed) void k_bresid(const BChunk* ch, const BProb* probs, const BCtl* ctl,
                                                 const double* hy, const double* y, const double* E, double* partial) {
    __shared__ double red[kRed];
    const BChunk c = ch[blockIdx.x];
    if (ctl[c.prob].done) return;
    const double e = E[c.prob];
    const uint64_t off = probs[c.prob].off;
    double acc = 0.0;
    for (uint64_t i = c.begin + threadIdx.x; i < c.end; i += blockDim.x) {
        const double r = hy[off + i] - e * y[off + i];
        acc += r * r;
    }
    acc = bsum(acc, red);
    if (threadIdx.x == 0) partial[blockIdx.x] = acc;
}

size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

constexpr size_t kBatchLds = 159 * 1024;   // dynamic LDS limit: 160 KiB less the kernels' static words

template <typename T, int BLOCK>
pdz_status set_batch_lds() {
    PDZ_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_batch_hv<T, BLOCK>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)kBatchLds));
    PDZ_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_batch_rows<T, BLOCK>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)kBatchLds));
    return ok();
}

}  // namespace

pdz_status batch_prepare() {
    pdz_status st = set_batch_lds<double, 256>();
    if (st == PDZ_OK) st = set_batch_lds<double, 512>();
    if (st == PDZ_OK) st = set_batch_lds<double, 1024>();
    if (st == PDZ_OK) st = set_batch_lds<float, 256>();
    if (st == PDZ_OK) st = set_batch_lds<float, 512>();
    if (st == PDZ_OK) st = set_batch_lds<float, 1024>();
    return st;
}

}  // namespace pdz

using namespace pdz;

struct pdz_batch_s {
    int device = 0;
    int n = 0;
    std::vector<pdz_problem> problems;
    std::vector<uint64_t> offsets;   // n + 1, elements
    uint64_t total = 0;
    BProb* d_probs = nullptr;
    BTile* d_tiles = nullptr;        // tiles for the current plan
    uint32_t ntiles = 0;
    BChunk* d_chunks = nullptr;
    uint32_t* d_chunk_begin = nullptr;   // n + 1
    uint32_t nchunks = 0;
    uint32_t* d_tile_begin = nullptr;    // n first tiles, then n tile counts, for the current plan
    uint32_t nrows_tiles = 0;            // tiles of k_batch_rows, first in the list; the rest are k_batch_hv's
    uint64_t max_D_dn = 0;
    pdz_batch_plan plan{0, 0, 0, 0};
    pdz_batch_plan tiles_for{-1, -1, -1, -1};
};

namespace {

pdz_batch_plan resolve(const pdz_batch_s* b) {
    pdz_batch_plan p = b->plan;
    if (p.tile_elems == 0) p.tile_elems = 4096;
    // the fastest of the search space in FP64 on 32 mixed clusters (108 us; 256
    // threads and four groups per CU 118), within 5 % of it in FP32
    if (p.block == 0) p.block = 512;
    if (p.wgs_per_cu == 0) p.wgs_per_cu = 8;
    if (p.order == 0) p.order = 1;
    return p;
}

bool plan_ok(const pdz_batch_s* b, const pdz_batch_plan& p) {
    const bool te = p.tile_elems == 1024 || p.tile_elems == 2048 || p.tile_elems == 4096 || p.tile_elems == 8192;
    const bool bl = p.block == 256 || p.block == 512 || p.block == 1024;
    const bool wg = p.wgs_per_cu >= 1 && p.wgs_per_cu <= 8;
    const bool od = p.order == 1 || p.order == 2;
    // every tile must hold at least one full row in LDS for both precisions
    const bool fits = b->max_D_dn * 8 + kMaxCoef * 8 + 1024 <= 160 * 1024;
    return te && bl && wg && od && fits;
}

// Whether a cluster's tiles take the one-pass form (k_batch_rows): four rows in
// LDS in FP64, byte offsets of its elements in 32 bits, and rows of at least 33
// columns.  One product of a batch in us, one-pass form against k_batch_hv
// (FP64, FP32): 16 x (4x4 8+1, 16 columns) 183 / 82, 123 / 68; 512 x (ring of 8
// 4+2, 28 columns) 17.6 / 14.2, 13.4 / 12.0; 512 x (ring of 7 3+3, 35 columns)
// 10.7 / 10.5, 9.0 / 9.2; 256 x (3x3 4+2, 36 columns) 32 / 42, 22 / 28; and with
// the device work queue k_batch_hv once had, 2 x (5x3 6+6, 5005 columns)
// 1044 / 1820, 502 / 1420.
bool rows_form(const pdz_problem q) {
    return q->dn.D >= kRowsMinDn && q->D <= 0xFFFFFFFFull / 8 &&
           kMaxCoef * 8 + (q->dn.D + 1) * kBatchRV * 8 <= kBatchLds;
}

// Rows per tile of a cluster: about tile_elems elements, whole groups of
// kBatchRV rows in the one-pass form, no more than the LDS holds.
uint64_t tile_rows(const pdz_problem q, int tile_elems) {
    const uint64_t Dn = q->dn.D;
    uint64_t rows = (uint64_t)tile_elems / Dn;
    if (rows_form(q)) {
        rows = rows / kBatchRV * kBatchRV;
        return rows < kBatchRV ? kBatchRV : rows;
    }
    const uint64_t cap = (160 * 1024 - kMaxCoef * 8 - 1024) / 8;   // elements, FP64 worst case
    if (rows * Dn > cap) rows = cap / Dn;
    return rows < 1 ? 1 : rows;
}

// Most tiles of any plan (the smallest tiles).
size_t max_tiles(const pdz_batch_s* b) {
    size_t n = 0;
    for (const pdz_problem q : b->problems) {
        const uint64_t rows = tile_rows(q, 1024);
        n += (size_t)((q->up.D + rows - 1) / rows);
    }
    return n;
}

// Tiles: rows of each cluster in groups of about tile_elems elements, the
// one-pass form's first; order 1 = largest clusters first, 2 = cluster order.
pdz_status build_tiles(pdz_batch_s* b, const pdz_batch_plan& p) {
    if (b->d_tiles && b->tiles_for.tile_elems == p.tile_elems && b->tiles_for.order == p.order) return ok();
    std::vector<int> idx(b->n);
    std::iota(idx.begin(), idx.end(), 0);
    if (p.order == 1)
        std::stable_sort(idx.begin(), idx.end(), [&](int a, int c) { return b->problems[a]->D > b->problems[c]->D; });
    std::vector<BTile> tiles;
    std::vector<uint32_t> range(2 * (size_t)b->n);
    std::stable_partition(idx.begin(), idx.end(), [&](int i) { return rows_form(b->problems[i]); });
    uint32_t nrows_tiles = 0;
    for (int i : idx) {
        const pdz_problem q = b->problems[i];
        const uint64_t Du = q->up.D;
        const uint64_t rows = tile_rows(q, p.tile_elems);
        range[i] = (uint32_t)tiles.size();
        for (uint64_t u0 = 0; u0 < Du; u0 += rows) {
            BTile t;
            t.prob = (uint32_t)i;
            t.u0 = (uint32_t)u0;
            t.nrows = (uint32_t)((Du - u0) < rows ? (Du - u0) : rows);
            t.pad = 0;
            tiles.push_back(t);
        }
        range[b->n + i] = (uint32_t)tiles.size() - range[i];
        if (rows_form(q)) nrows_tiles = (uint32_t)tiles.size();
    }
    if (b->d_tiles) {
        PDZ_HIP(hipDeviceSynchronize());   // products in flight read the list
        (void)hipFree(b->d_tiles);
        b->d_tiles = nullptr;
    }
    PDZ_HIP(hipMalloc(&b->d_tiles, tiles.size() * sizeof(BTile)));
    PDZ_HIP(hipMemcpy(b->d_tiles, tiles.data(), tiles.size() * sizeof(BTile), hipMemcpyHostToDevice));
    PDZ_HIP(hipMemcpy(b->d_tile_begin, range.data(), range.size() * sizeof(uint32_t), hipMemcpyHostToDevice));
    b->ntiles = (uint32_t)tiles.size();
    b->nrows_tiles = nrows_tiles;
    b->tiles_for = p;
    return ok();
}

// dotp: NULL, or one partial sum of x . y per tile
template <typename T>
pdz_status batch_hv_launch(pdz_batch_s* b, const pdz_batch_plan& p, const T* x, T* y, hipStream_t s, const int* done,
                           int dstride, double* dotp) {
    DeviceCtx* ctx = nullptr;
    pdz_status st = device_ctx(&ctx);
    if (st != PDZ_OK) return st;
    size_t max_tile[2] = {0, 0};   // elements of a tile's LDS: k_batch_rows, k_batch_hv
    for (const pdz_problem q : b->problems) {
        const uint64_t rows = std::min<uint64_t>(tile_rows(q, p.tile_elems), q->up.D);
        if (rows_form(q))
            max_tile[0] = std::max(max_tile[0], (size_t)(rows + kBatchRV - 1) / kBatchRV * kBatchRV * (q->dn.D + 1));
        else
            max_tile[1] = std::max(max_tile[1], (size_t)rows * q->dn.D);
    }
    const auto launch = [&](auto kernel, int form, uint32_t t0, uint32_t n) {
        const dim3 grid(std::min<unsigned>((unsigned)(ctx->cu_count * p.wgs_per_cu), n)), block((unsigned)p.block);
        hipLaunchKernelGGL(kernel, grid, block, (kMaxCoef + max_tile[form]) * sizeof(T), s, b->d_probs, b->d_tiles + t0,
                           n, done, dstride, dotp ? dotp + t0 : nullptr, x, y);
    };
    const uint32_t nr = b->nrows_tiles, ng = b->ntiles - nr;
    if (nr > 0) {
        if (p.block == 1024) launch(k_batch_rows<T, 1024>, 0, 0, nr);
        else if (p.block == 512) launch(k_batch_rows<T, 512>, 0, 0, nr);
        else launch(k_batch_rows<T, 256>, 0, 0, nr);
    }
    if (ng > 0) {
        if (p.block == 1024) launch(k_batch_hv<T, 1024>, 1, nr, ng);
        else if (p.block == 512) launch(k_batch_hv<T, 512>, 1, nr, ng);
        else launch(k_batch_hv<T, 256>, 1, nr, ng);
    }
    PDZ_HIP(hipGetLastError());
    return ok();
}

pdz_status batch_hv_any(pdz_batch_s* b, pdz_dtype dt, const void* x, void* y, hipStream_t s, const int* done,
                        int dstride, double* dotp = nullptr) {
    const pdz_batch_plan p = resolve(b);
    pdz_status st = build_tiles(b, p);
    if (st != PDZ_OK) return st;
    if (dt == PDZ_F64)
        return batch_hv_launch<double>(b, p, static_cast<const double*>(x), static_cast<double*>(y), s, done,
                                       dstride, dotp);
    return batch_hv_launch<float>(b, p, static_cast<const float*>(x), static_cast<float*>(y), s, done, dstride,
                                  dotp);
}

struct BLayout {
    size_t vec = 0, buf[3] = {0, 0, 0}, alpha = 0, beta = 0, sc = 0, theta = 0, resid = 0, svec = 0, partial = 0,
           norms[2] = {0, 0}, dots = 0, ctl = 0, total = 0;
    size_t y = 0, hy = 0, kfin = 0, eref = 0;   // refinement (refine == 1)
    int ld = 0;
};

BLayout blayout(const pdz_batch_s* b, const pdz_lanczos_opts* o) {
    BLayout L;
    const size_t es = o->storage == PDZ_F64 ? 8 : 4;
    L.vec = al256(b->total * es);
    size_t off = 0;
    for (int i = 0; i < 3; ++i) {
        L.buf[i] = off;
        off += L.vec;
    }
    L.ld = o->max_iter + 8;
    const size_t per = (size_t)L.ld * b->n * 8;
    for (size_t* a : {&L.alpha, &L.beta, &L.sc, &L.theta, &L.resid, &L.svec}) {
        *a = off;
        off += al256(per);
    }
    for (size_t* a : {&L.partial, &L.norms[0], &L.norms[1]}) {
        *a = off;
        off += al256((size_t)b->nchunks * 8);
    }
    L.dots = off;
    off += al256(max_tiles(b) * 8);
    L.ctl = off;
    off += al256((size_t)b->n * sizeof(BCtl));
    if (o->refine) {
        L.y = off;
        off += al256(b->total * 8);
        L.hy = off;
        off += al256(b->total * 8);
        L.kfin = off;
        off += al256((size_t)b->n * sizeof(int));
        L.eref = off;
        off += al256((size_t)b->n * 2 * 8);
    }
    L.total = off;
    return L;
}

template <typename T>
pdz_status batch_lanczos_run(pdz_batch_s* b, const pdz_lanczos_opts* o, char* ws, const BLayout& L,
                             pdz_lanczos_result* res, hipStream_t s, uint32_t* err) {
    T* buf[3];
    for (int i = 0; i < 3; ++i) buf[i] = reinterpret_cast<T*>(ws + L.buf[i]);
    double* alpha = reinterpret_cast<double*>(ws + L.alpha);
    double* beta = reinterpret_cast<double*>(ws + L.beta);
    double* sc = reinterpret_cast<double*>(ws + L.sc);
    double* theta = reinterpret_cast<double*>(ws + L.theta);
    double* resid = reinterpret_cast<double*>(ws + L.resid);
    double* svec = reinterpret_cast<double*>(ws + L.svec);
    double* partial = reinterpret_cast<double*>(ws + L.partial);
    BCtl* ctl = reinterpret_cast<BCtl*>(ws + L.ctl);
    const int ld = L.ld;
    const dim3 nch(b->nchunks), np(b->n), blk(kRed), npg((b->n + 255) / 256), b256(256);
    const pdz_dtype dt = o->storage == PDZ_F64 ? PDZ_F64 : PDZ_F32;
    BStep bs;
    bs.tile_begin = b->d_tile_begin;
    bs.tile_count = b->d_tile_begin + b->n;
    bs.chunk_begin = b->d_chunk_begin;
    bs.dots = reinterpret_cast<double*>(ws + L.dots);
    for (int i = 0; i < 2; ++i) bs.norms[i] = reinterpret_cast<double*>(ws + L.norms[i]);
    bs.alpha = alpha;
    bs.beta = beta;
    bs.sc = sc;
    bs.ld = ld;
    bs.koff = 0;
    bs.kmax = o->max_iter;
    // start: q_0 = SplitMix64 vectors, sc_0 = 1 / |q_0| per cluster, q_{-1} = 0
    const auto start = [&]() {
        hipLaunchKernelGGL(k_bzero<T>, dim3(1024), blk, 0, s, b->total, buf[0], buf[2]);
        hipLaunchKernelGGL(k_bfill<T>, nch, blk, 0, s, b->d_chunks, b->d_probs, o->seed, buf[0]);
        hipLaunchKernelGGL(k_bdot<T>, nch, blk, 0, s, b->d_chunks, b->d_probs, ctl, buf[0], buf[0], partial);
        hipLaunchKernelGGL(k_bnorm0, np, blk, 0, s, b->d_chunk_begin, partial, ctl, sc, ld, err);
    };
    hipLaunchKernelGGL(k_clear_bits1, dim3(1), dim3(1), 0, s, err, kErrNonFinite);
    hipLaunchKernelGGL(k_binit, npg, b256, 0, s, ctl, beta, ld, (uint32_t)b->n);
    start();
    PDZ_HIP(hipGetLastError());
    const int* done = &ctl[0].done;
    const int dstride = (int)(sizeof(BCtl) / sizeof(int));
    int period = o->check_every;
    if (period % 3) period += 3 - period % 3;
    auto step = [&](T* q, T* qp, T* w, int koff) -> pdz_status {
        pdz_status st = batch_hv_any(b, dt, q, w, s, done, dstride, const_cast<double*>(bs.dots));
        if (st != PDZ_OK) return st;
        bs.koff = koff;
        hipLaunchKernelGGL(k_bupdate<T>, nch, blk, 0, s, b->d_chunks, b->d_probs, ctl, bs, w, q, qp);
        return ok();
    };
    auto end_block = [&](int steps) {
        hipLaunchKernelGGL(k_britz_block, dim3((unsigned)steps, (unsigned)b->n), dim3(kTriBlock), 0, s, ctl,
                           b->d_chunk_begin, bs.norms[0], bs.norms[1], alpha, beta, theta, resid, ld, o->max_iter);
        hipLaunchKernelGGL(k_britz_end, npg, b256, 0, s, ctl, (uint32_t)b->n, steps, alpha, beta, theta, resid, ld,
                           o->tol, o->max_iter, err);
    };
    auto enqueue = [&]() -> pdz_status {
        for (int t = 0; t < period; ++t) {
            const int a = t % 3;
            pdz_status st = step(buf[a], buf[(a + 2) % 3], buf[(a + 1) % 3], t % kRitzBlock);
            if (st != PDZ_OK) return st;
            if ((t + 1) % kRitzBlock == 0 || t + 1 == period) end_block(t % kRitzBlock + 1);
        }
        PDZ_HIP(hipGetLastError());
        return ok();
    };
    // tiles for the current plan must exist before capture (no allocation inside a graph)
    pdz_status st = build_tiles(b, resolve(b));
    if (st != PDZ_OK) return st;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    if (o->use_graph) {
        PDZ_HIP(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
        st = enqueue();
        hipGraph_t g2 = nullptr;
        hipError_t e = hipStreamEndCapture(s, &g2);
        if (st != PDZ_OK) {
            if (g2) (void)hipGraphDestroy(g2);
            return st;
        }
        if (e != hipSuccess) return hip_fail(e, "hipStreamEndCapture");
        graph = g2;
        e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
        if (e != hipSuccess) {
            (void)hipGraphDestroy(graph);
            return hip_fail(e, "hipGraphInstantiate");
        }
    }
    std::vector<BCtl> h(b->n);
    st = ok();
    for (int steps = 0; steps < o->max_iter; steps += period) {
        if (exec) {
            hipError_t e = hipGraphLaunch(exec, s);
            if (e != hipSuccess) {
                st = hip_fail(e, "hipGraphLaunch");
                break;
            }
        } else {
            st = enqueue();
            if (st != PDZ_OK) break;
        }
        hipError_t e = hipMemcpyAsync(h.data(), ctl, b->n * sizeof(BCtl), hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) {
            st = hip_fail(e, "batched Lanczos flags");
            break;
        }
        bool all = true;
        for (const BCtl& c : h) all = all && c.done;
        if (all) break;
    }
    if (exec) (void)hipGraphExecDestroy(exec);
    if (graph) (void)hipGraphDestroy(graph);
    if (st != PDZ_OK) return st;
    uint32_t word = 0;
    PDZ_HIP(hipMemcpyAsync(h.data(), ctl, b->n * sizeof(BCtl), hipMemcpyDeviceToHost, s));
    PDZ_HIP(hipMemcpyAsync(&word, err, sizeof(word), hipMemcpyDeviceToHost, s));
    PDZ_HIP(hipStreamSynchronize(s));
    if (word & kErrNonFinite) {
        hipLaunchKernelGGL(k_clear_bits1, dim3(1), dim3(1), 0, s, err, kErrNonFinite);
        (void)hipStreamSynchronize(s);
        return fail(PDZ_EINVAL, "non-finite Lanczos scalar (start vector or H)");
    }
    bool all_conv = true;
    int kmax = 0;
    for (int i = 0; i < b->n; ++i) {
        if (!(h[i].norm0 > 0.0) || !std::isfinite(h[i].norm0))
            return fail(PDZ_EINVAL, "a start vector has zero or non-finite norm");
        res[i].E0 = h[i].theta;
        res[i].resid_est = h[i].resid;
        res[i].E0_refined = h[i].theta;
        res[i].resid_refined = -1.0;
        res[i].iters = h[i].k;
        res[i].converged = h[i].converged;
        all_conv = all_conv && h[i].converged;
        kmax = std::max(kmax, h[i].k);
    }
    if (o->refine && kmax > 0) {
        // Ritz vector y_p = sum_j s_{p,j} sc_{p,j} q_{p,j} in FP64 from the regenerated
        // Lanczos vectors, normalised; its FP64 Rayleigh quotient and residual.
        double* y = reinterpret_cast<double*>(ws + L.y);
        double* hy = reinterpret_cast<double*>(ws + L.hy);
        int* kfin = reinterpret_cast<int*>(ws + L.kfin);
        double* eref = reinterpret_cast<double*>(ws + L.eref);
        hipLaunchKernelGGL(k_britz_vector, np, dim3(kTriBlock), 0, s, ctl, alpha, beta, svec, ld);
        hipLaunchKernelGGL(k_bregen_init, npg, b256, 0, s, ctl, kfin, (uint32_t)b->n);
        hipLaunchKernelGGL(k_bzero<double>, dim3(1024), blk, 0, s, b->total, y, hy);
        start();
        for (int j = 0; j < kmax; ++j) {
            const int a = j % 3;
            T* v = buf[a];
            T* vp = buf[(a + 2) % 3];
            T* w = buf[(a + 1) % 3];
            hipLaunchKernelGGL(k_baxpy_ritz<T>, nch, blk, 0, s, b->d_chunks, b->d_probs, ctl, svec, sc, ld, v, y);
            if (j + 1 >= kmax) break;
            hipLaunchKernelGGL(k_bregen_mark, npg, b256, 0, s, ctl, kfin, (uint32_t)b->n);
            st = batch_hv_any(b, dt, v, w, s, done, dstride);
            if (st != PDZ_OK) return st;
            hipLaunchKernelGGL(k_bregen_update<T>, nch, blk, 0, s, b->d_chunks, b->d_probs, ctl, alpha, beta, sc,
                               ld, w, v, vp);
            hipLaunchKernelGGL(k_bregen_next, npg, b256, 0, s, ctl, (uint32_t)b->n);
        }
        hipLaunchKernelGGL(k_bregen_reopen, npg, b256, 0, s, ctl, kfin, (uint32_t)b->n);
        hipLaunchKernelGGL(k_bdot<double>, nch, blk, 0, s, b->d_chunks, b->d_probs, ctl, y, y, partial);
        hipLaunchKernelGGL(k_bnorm0, np, blk, 0, s, b->d_chunk_begin, partial, ctl, (double*)nullptr, ld, err);
        hipLaunchKernelGGL(k_bscale, nch, blk, 0, s, b->d_chunks, b->d_probs, ctl, y);
        st = batch_hv_any(b, PDZ_F64, y, hy, s, done, dstride);
        if (st != PDZ_OK) return st;
        hipLaunchKernelGGL(k_bdot<double>, nch, blk, 0, s, b->d_chunks, b->d_probs, ctl, y, hy, partial);
        hipLaunchKernelGGL(k_bsum_out, np, blk, 0, s, b->d_chunk_begin, partial, ctl, eref, 0);
        hipLaunchKernelGGL(k_bresid, nch, blk, 0, s, b->d_chunks, b->d_probs, ctl, hy, y, eref, partial);
        hipLaunchKernelGGL(k_bsum_out, np, blk, 0, s, b->d_chunk_begin, partial, ctl, eref + b->n, 1);
        PDZ_HIP(hipGetLastError());
        std::vector<double> er(2 * (size_t)b->n);
        std::vector<int> kf(b->n);
        PDZ_HIP(hipMemcpyAsync(er.data(), eref, er.size() * 8, hipMemcpyDeviceToHost, s));
        PDZ_HIP(hipMemcpyAsync(kf.data(), kfin, kf.size() * sizeof(int), hipMemcpyDeviceToHost, s));
        PDZ_HIP(hipStreamSynchronize(s));
        for (int i = 0; i < b->n; ++i)
            if (kf[i] > 0) {
                res[i].E0_refined = er[i];
                res[i].resid_refined = er[b->n + i];
            }
        // leave the control blocks as the run ended
        PDZ_HIP(hipMemcpyAsync(ctl, h.data(), b->n * sizeof(BCtl), hipMemcpyHostToDevice, s));
        PDZ_HIP(hipStreamSynchronize(s));
    }
    return all_conv ? ok() : fail(PDZ_ENOCONV, "max_iter reached before every cluster met the tolerance");
}

}  // namespace

extern "C" {

pdz_status pdz_batch_create(const pdz_problem* problems, int32_t n, pdz_batch* out) {
    if (!out) return fail(PDZ_EINVAL, "out is NULL");
    *out = nullptr;
    if (n < 1 || !problems) return fail(PDZ_EINVAL, "need at least one problem");
    int dev = 0;
    PDZ_HIP(hipGetDevice(&dev));
    for (int i = 0; i < n; ++i) {
        if (!problems[i]) return fail(PDZ_EINVAL, "NULL problem in batch");
        if (problems[i]->device != dev) return fail(PDZ_EINVAL, "batch problems must live on the current device");
        if (problems[i]->hv_path != 0) return fail(PDZ_ERANGE, "batched H.v needs sector hop tables");
    }
    pdz_batch_s* b = new pdz_batch_s();
    b->device = dev;
    b->n = n;
    b->problems.assign(problems, problems + n);
    b->offsets.resize(n + 1);
    uint64_t off = 0;
    std::vector<BProb> hp(n);
    std::vector<BChunk> chunks;
    std::vector<uint32_t> cb(n + 1);
    for (int i = 0; i < n; ++i) {
        const pdz_problem q = problems[i];
        b->offsets[i] = off;
        hp[i].off = off;
        hp[i].D_up = q->up.D;
        hp[i].D_dn = q->dn.D;
        hp[i].U = q->U;
        hp[i].up_states = q->up.states;
        hp[i].dn_states = q->dn.states;
        hp[i].up_count = q->up.count;
        hp[i].dn_count = q->dn.count;
        hp[i].up_ell = q->up.ell;
        hp[i].dn_ell = q->dn.ell;
        hp[i].coef64 = q->d_coef64;
        hp[i].coef32 = q->d_coef32;
        hp[i].ncoef = (int)q->coef_host.size();
        hp[i].dn_max = q->dn.max_hops;
        b->max_D_dn = std::max<uint64_t>(b->max_D_dn, q->dn.D);
        cb[i] = (uint32_t)chunks.size();
        for (uint64_t s0 = 0; s0 < q->D; s0 += kChunk) {
            BChunk c;
            c.prob = (uint32_t)i;
            c.pad = 0;
            c.begin = s0;
            c.end = std::min<uint64_t>(q->D, s0 + kChunk);
            chunks.push_back(c);
        }
        off += (q->D + kAlign - 1) / kAlign * kAlign;
    }
    cb[n] = (uint32_t)chunks.size();
    b->offsets[n] = off;
    b->total = off;
    b->nchunks = (uint32_t)chunks.size();
    auto cleanup = [&](pdz_status code) {
        pdz_batch_destroy(b);
        return code;
    };
#define BCK(call)                                                   \
    do {                                                            \
        hipError_t e_ = (call);                                     \
        if (e_ != hipSuccess) return cleanup(hip_fail(e_, #call)); \
    } while (0)
    BCK(hipMalloc(&b->d_probs, n * sizeof(BProb)));
    BCK(hipMemcpy(b->d_probs, hp.data(), n * sizeof(BProb), hipMemcpyHostToDevice));
    BCK(hipMalloc(&b->d_chunks, chunks.size() * sizeof(BChunk)));
    BCK(hipMemcpy(b->d_chunks, chunks.data(), chunks.size() * sizeof(BChunk), hipMemcpyHostToDevice));
    BCK(hipMalloc(&b->d_chunk_begin, (n + 1) * sizeof(uint32_t)));
    BCK(hipMemcpy(b->d_chunk_begin, cb.data(), (n + 1) * sizeof(uint32_t), hipMemcpyHostToDevice));
    BCK(hipMalloc(&b->d_tile_begin, 2 * (size_t)n * sizeof(uint32_t)));
#undef BCK
    if (!plan_ok(b, resolve(b))) return cleanup(fail(PDZ_ERANGE, "a cluster row does not fit the batched kernel's LDS"));
    pdz_status st = build_tiles(b, resolve(b));
    if (st != PDZ_OK) return cleanup(st);
    *out = b;
    return ok();
}

pdz_status pdz_batch_destroy(pdz_batch b) {
    if (!b) return ok();
    int prev = 0;
    (void)hipGetDevice(&prev);
    (void)hipSetDevice(b->device);
    (void)hipDeviceSynchronize();
    if (b->d_probs) (void)hipFree(b->d_probs);
    if (b->d_tiles) (void)hipFree(b->d_tiles);
    if (b->d_chunks) (void)hipFree(b->d_chunks);
    if (b->d_chunk_begin) (void)hipFree(b->d_chunk_begin);
    if (b->d_tile_begin) (void)hipFree(b->d_tile_begin);
    (void)hipSetDevice(prev);
    delete b;
    return ok();
}

pdz_status pdz_batch_offsets(pdz_batch b, uint64_t* offsets) {
    if (!b || !offsets) return fail(PDZ_EINVAL, "NULL argument");
    for (int i = 0; i <= b->n; ++i) offsets[i] = b->offsets[i];
    return ok();
}

pdz_status pdz_batch_get_plan(pdz_batch b, pdz_batch_plan* out) {
    if (!b || !out) return fail(PDZ_EINVAL, "NULL argument");
    *out = resolve(b);
    return ok();
}

pdz_status pdz_batch_set_plan(pdz_batch b, const pdz_batch_plan* plan) {
    if (!b || !plan) return fail(PDZ_EINVAL, "NULL argument");
    pdz_batch_plan p = *plan;
    const pdz_batch_plan d = resolve(b);
    if (p.tile_elems == 0) p.tile_elems = d.tile_elems;
    if (p.block == 0) p.block = d.block;
    if (p.wgs_per_cu == 0) p.wgs_per_cu = d.wgs_per_cu;
    if (p.order == 0) p.order = d.order;
    if (!plan_ok(b, p)) return fail(PDZ_EINVAL, "batch plan out of range");
    pdz_status st = build_tiles(b, p);
    if (st != PDZ_OK) return st;
    b->plan = p;
    return ok();
}

pdz_status pdz_batch_hv(pdz_batch b, pdz_dtype dt, const void* x, void* y, void* stream) {
    if (!b) return fail(PDZ_EINVAL, "batch is NULL");
    if (dt != PDZ_F64 && dt != PDZ_F32) return fail(PDZ_EINVAL, "dtype must be PDZ_F64 or PDZ_F32");
    if (!x || !y) return fail(PDZ_EINVAL, "NULL vector");
    const size_t bytes = (size_t)b->total * (dt == PDZ_F64 ? 8 : 4);
    const char* xb = static_cast<const char*>(x);
    const char* yb = static_cast<const char*>(y);
    if (xb < yb + bytes && yb < xb + bytes) return fail(PDZ_EINVAL, "x and y overlap");
    return batch_hv_any(b, dt, x, y, (hipStream_t)stream, nullptr, 0);
}

pdz_status pdz_batch_tune(pdz_batch b, pdz_dtype dt, const void* x, void* y, int32_t reps, pdz_batch_trial* trials,
                          int32_t max_trials, int32_t* n_trials, pdz_batch_plan* best, void* stream) {
    if (!b || !x || !y) return fail(PDZ_EINVAL, "NULL argument");
    if (dt != PDZ_F64 && dt != PDZ_F32) return fail(PDZ_EINVAL, "dtype must be PDZ_F64 or PDZ_F32");
    if (reps < 1) return fail(PDZ_EINVAL, "reps must be >= 1");
    if (max_trials > 0 && !trials) return fail(PDZ_EINVAL, "trials is NULL");
    hipStream_t s = (hipStream_t)stream;
    const pdz_batch_plan saved = resolve(b);
    hipEvent_t e0 = nullptr, e1 = nullptr;
    PDZ_HIP(hipEventCreate(&e0));
    PDZ_HIP(hipEventCreate(&e1));
    double best_ms = 1e300;
    pdz_batch_plan bp = saved;
    int n = 0;
    pdz_status st = ok();
    const int tes[] = {1024, 2048, 4096, 8192};
    const int bls[] = {256, 512, 1024};
    const int wgs[] = {2, 4, 8};
    const int ods[] = {1, 2};
    for (int te : tes)
        for (int bl : bls)
            for (int wg : wgs)
                for (int od : ods) {
                    pdz_batch_plan c{te, bl, wg, od};
                    if (!plan_ok(b, c)) continue;
                    // prune: natural order only with the default tile size (largest-first wins by cost model)
                    if (od == 2 && te != 4096) continue;
                    st = pdz_batch_set_plan(b, &c);
                    if (st != PDZ_OK) break;
                    st = pdz_batch_hv(b, dt, x, y, stream);
                    if (st != PDZ_OK) break;
                    hipError_t e = hipEventRecord(e0, s);
                    for (int r = 0; r < reps && st == PDZ_OK; ++r) st = pdz_batch_hv(b, dt, x, y, stream);
                    if (st != PDZ_OK) break;
                    if (e == hipSuccess) e = hipEventRecord(e1, s);
                    if (e == hipSuccess) e = hipEventSynchronize(e1);
                    float ms = 0.f;
                    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
                    if (e != hipSuccess) {
                        st = hip_fail(e, "batch autotune timing");
                        break;
                    }
                    const double avg = (double)ms / reps;
                    if (n < max_trials) {
                        trials[n].plan = c;
                        trials[n].ms = avg;
                    }
                    ++n;
                    if (avg < best_ms) {
                        best_ms = avg;
                        bp = c;
                    }
                }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (st != PDZ_OK) {
        (void)pdz_batch_set_plan(b, &saved);
        return st;
    }
    st = pdz_batch_set_plan(b, &bp);
    if (st != PDZ_OK) return st;
    if (n_trials) *n_trials = n < max_trials ? n : max_trials;
    if (best) *best = bp;
    return ok();
}

pdz_status pdz_batch_lanczos_workspace_size(pdz_batch b, const pdz_lanczos_opts* o, size_t* bytes) {
    if (!b || !o || !bytes) return fail(PDZ_EINVAL, "NULL argument");
    if (o->max_iter < 1 || o->max_iter > kBatchMaxIter) return fail(PDZ_EINVAL, "max_iter must be in [1, 2000]");
    *bytes = blayout(b, o).total;
    return ok();
}

pdz_status pdz_batch_lanczos(pdz_batch b, const pdz_lanczos_opts* o, void* ws, size_t ws_bytes,
                             pdz_lanczos_result* results, void* stream) {
    const auto t0 = std::chrono::steady_clock::now();
    if (!b || !o || !results) return fail(PDZ_EINVAL, "NULL argument");
    if (o->max_iter < 1 || o->max_iter > kBatchMaxIter) return fail(PDZ_EINVAL, "max_iter must be in [1, 2000]");
    if (!(o->tol >= 0.0) || !std::isfinite(o->tol)) return fail(PDZ_EINVAL, "tol must be finite and >= 0");
    if (o->storage != PDZ_F64 && o->storage != PDZ_F32) return fail(PDZ_EINVAL, "storage must be F64 or F32");
    if (o->check_every < 1) return fail(PDZ_EINVAL, "check_every must be >= 1");
    if (o->reorth != 0) return fail(PDZ_EINVAL, "batched Lanczos runs the three-term recurrence (reorth must be 0)");
    if (o->refine != 0 && o->refine != 1) return fail(PDZ_EINVAL, "refine must be 0 or 1");
    if (o->keep_basis != 0) return fail(PDZ_EINVAL, "keep_basis is not offered for batches (refine regenerates)");
    const BLayout L = blayout(b, o);
    if (!ws || ws_bytes < L.total) return fail(PDZ_EINVAL, "workspace smaller than pdz_batch_lanczos_workspace_size");
    if (reinterpret_cast<uintptr_t>(ws) % 256) return fail(PDZ_EINVAL, "workspace must be 256-byte aligned");
    DeviceCtx* ctx = nullptr;
    pdz_status st = device_ctx(&ctx);
    if (st != PDZ_OK) return st;
    hipStream_t s = (hipStream_t)stream;
    hipStream_t own = nullptr;
    if (!s && o->use_graph) {
        PDZ_HIP(hipStreamCreateWithFlags(&own, hipStreamNonBlocking));
        PDZ_HIP(hipDeviceSynchronize());
        s = own;
    }
    std::memset(results, 0, sizeof(pdz_lanczos_result) * b->n);
    if (o->storage == PDZ_F64)
        st = batch_lanczos_run<double>(b, o, static_cast<char*>(ws), L, results, s, ctx->err);
    else
        st = batch_lanczos_run<float>(b, o, static_cast<char*>(ws), L, results, s, ctx->err);
    if (own) {
        (void)hipStreamSynchronize(own);
        (void)hipStreamDestroy(own);
    }
    const double secs = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    for (int i = 0; i < b->n; ++i) results[i].seconds = secs;
    return st;
}

}  // extern "C"
