// Learned Lanczos start vector: a 32 -> 128 -> 128 -> 2 tanh network on
// occupation strings, its training kernels and its inference over a basis.
//
// Parameters live in one vector (W1 128x32, b1, W2 128x128, b2, W3 2x128, b3;
// 20,994 values): FP32 master copy for Adam, BF16 copy for the kernels.
// Dense products run on the BF16 matrix cores (16x16x32, FP32 accumulation):
// one wave multiplies the weights by tiles of 16 states, the rows of weights
// dealt so that a layer's accumulators are the next layer's operands in
// place.  Stored activations are BF16.
//
// Training samples states with probability proportional to |psi|^2 using
// integer weights w_r = floor(2^32 psi_r^2 / max psi^2), an exact prefix sum
// and a SplitMix64 draw per sample, so the draws do not depend on summation
// order.
#include <cmath>
#include <mutex>
#include <vector>

#include "pdz_internal.h"

namespace pdz {
namespace {

constexpr int kIn = 32, kHid = 128, kOut = 2;
constexpr int kParams = kHid * kIn + kHid + kHid * kHid + kHid + kOut * kHid + kOut;   // 20,994
constexpr int oW1 = 0, oB1 = kHid * kIn, oW2 = oB1 + kHid, oB2 = oW2 + kHid * kHid, oW3 = oB2 + kHid,
              oB3 = oW3 + kOut * kHid;
static_assert(oB3 + kOut == kParams, "parameter layout");
constexpr int kLd1 = kIn + 8;    // padded LDS row of W1 (bf16 elements)
constexpr int kLd2 = kHid + 8;   // padded LDS row of W2 / W2^T / hidden tiles
constexpr int kLossBlocks = 64;
constexpr int kScanChunk = 8192;   // elements per block of the sampler prefix sum (32 per thread)

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
__device__ __forceinline__ uint16_t f2bf(float f) {   // round to nearest even
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ bf16x8 ld8(const uint16_t* p) {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(p));
}
__device__ __forceinline__ bf16x8 pack8(const uint16_t* v) {
    u32x4 u;
    u.x = v[0] | ((uint32_t)v[1] << 16);
    u.y = v[2] | ((uint32_t)v[3] << 16);
    u.z = v[4] | ((uint32_t)v[5] << 16);
    u.w = v[6] | ((uint32_t)v[7] << 16);
    return __builtin_bit_cast(bf16x8, u);
}
__device__ __forceinline__ f32x4 mma(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// tanh(x) = 1 - 2 / (exp(2x) + 1); saturates to +-1 for large |x|
__device__ __forceinline__ float tanh_fast(float x) {
    constexpr float k = 2.0f * 1.44269504088896340736f;   // exp(2x) = 2^(2x log2(e))
    return fmaf(-2.0f, __builtin_amdgcn_rcpf(__builtin_amdgcn_exp2f(k * x) + 1.0f), 1.0f);
}
// 8 features (+-1 in BF16) of one operand slot: bits [off, off + 8) of `bits`
__device__ __forceinline__ bf16x8 feature8(uint32_t bits) {
    uint16_t v[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) v[t] = ((bits >> t) & 1u) ? (uint16_t)0x3F80 : (uint16_t)0xBF80;
    return pack8(v);
}
// Source of the states of a forward pass.
struct StateSrc {
    const uint32_t* occ;        // list mode: occ[2s] up bits, occ[2s+1] down bits
    const uint32_t* up_states;  // basis mode: state s = r is (up_states[r / D_dn], dn_states[r % D_dn])
    const uint32_t* dn_states;
    uint64_t D_dn;
};
template <bool BASIS>
__device__ __forceinline__ void state_of(const StateSrc& S, uint64_t s, uint32_t* up, uint32_t* dn) {
    if (BASIS) {   // at most 16 sites: the basis has fewer than 2^32 states
        const uint32_t iu = (uint32_t)s / (uint32_t)S.D_dn;
        *up = S.up_states[iu];
        *dn = S.dn_states[(uint32_t)s - iu * (uint32_t)S.D_dn];
    } else {
        *up = S.occ[2 * s];
        *dn = S.occ[2 * s + 1];
    }
}

struct Act {                 // saved activations of a training forward pass (BF16)
    uint16_t* h1;            // n x 128, state major
    uint16_t* h1t;           // 128 x n
    uint16_t* h2;            // n x 128
};

// Weights as a wave's matrix operands read them, staged in LDS (padded rows)
// or held in registers.  Row r of the last layer's operand is row r mod 4 of
// W3 with two rows of zeros below it.
struct WLds {
    const uint16_t *w1, *w2, *w3;
    __device__ __forceinline__ bf16x8 l3(int q, int g, int c) const { return ld8(w3 + (c & 3) * kLd2 + 32 * q + 8 * g); }
    __device__ __forceinline__ bf16x8 l1(int, int u, int g) const { return ld8(w1 + u * kLd1 + 8 * g); }
    __device__ __forceinline__ bf16x8 l2(int, int k, int u, int g) const { return ld8(w2 + u * kLd2 + 32 * k + 8 * g); }
};
struct WReg {
    bf16x8 w1[8], w2[8][4], w3[4];
    __device__ __forceinline__ bf16x8 l3(int q, int, int) const { return w3[q]; }
    __device__ __forceinline__ bf16x8 l1(int i, int, int) const { return w1[i]; }
    __device__ __forceinline__ bf16x8 l2(int i, int k, int, int) const { return w2[i][k]; }
};

// Unit of row r in tile i of a hidden layer's operand order: tiles 2q and
// 2q + 1 give the lane group g of the accumulators the units 32q + 8g .. + 3
// and 32q + 8g + 4 .. + 7, that is the eight features 8g .. 8g + 7 of block q
// that the same lane has to bring to the next product.
__device__ __forceinline__ int tile_unit(int i, int r) { return 32 * (i >> 1) + 8 * (r >> 2) + 4 * (i & 1) + (r & 3); }

// tanh of eight pre-activations (two accumulators plus biases), BF16
__device__ __forceinline__ bf16x8 tanh8(f32x4 a, f32x4 b, f32x4 ba, f32x4 bb) {
    typedef float f32x8 __attribute__((ext_vector_type(8)));
    f32x8 v;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        v[t] = tanh_fast(a[t] + ba[t]);
        v[4 + t] = tanh_fast(b[t] + bb[t]);
    }
    return __builtin_convertvector(v, bf16x8);   // round to nearest even, two per instruction
}

// One wave, 16 S states from s0: the three layers.  Products are weights
// (rows: units) times states (columns), so a lane's accumulators hold four
// units of one state; the rows are dealt (tile_unit) so that two tiles leave
// a lane exactly the operand slot it feeds to the next layer, in the plain
// feature order: no exchange between lanes, no LDS round trip and no barrier
// between layers.  The last layer's two rows are in every group of four rows of
// its operand, so each lane group finds the outputs in its own rows and takes
// those of state tile g: with S = 4 lane l holds (o_0, o_1) of state s0 + l in
// the first two elements (S = 1: lanes 0..15, state s0 + l).  Each tile has an
// accumulator of its own: a state whose activations are not numbers stays alone.
template <bool ACT, int S, typename W>
__device__ __forceinline__ f32x4 mlp_layers(const W& w, const bf16x8 (&x)[S], const float* b1, const float* b2,
                                            int g, int c, uint64_t s0, uint64_t n, const Act& act,
                                            bool act_wide) {
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    bf16x8 h[S][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const bf16x8 wa = w.l1(2 * q, tile_unit(2 * q, c), g), wb = w.l1(2 * q + 1, tile_unit(2 * q + 1, c), g);
        const f32x4 ba = *reinterpret_cast<const f32x4*>(b1 + 32 * q + 8 * g);
        const f32x4 bb = *reinterpret_cast<const f32x4*>(b1 + 32 * q + 8 * g + 4);
#pragma unroll
        for (int s = 0; s < S; ++s) {
            h[s][q] = tanh8(mma(wa, x[s], zero), mma(wb, x[s], zero), ba, bb);
            const uint64_t st = s0 + 16 * s + c;
            if (ACT && act.h1 && st < n) {
                const u32x4 hv = __builtin_bit_cast(u32x4, h[s][q]);
                uint16_t* row = act.h1 + st * kHid + 32 * q + 8 * g;
                if (act_wide) *reinterpret_cast<u32x4*>(row) = hv;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const uint16_t hb = (uint16_t)((e & 1) ? (hv[e >> 1] >> 16) : (hv[e >> 1] & 0xFFFFu));
                    if (!act_wide) row[e] = hb;
                    act.h1t[(uint64_t)(32 * q + 8 * g + e) * n + st] = hb;
                }
            }
        }
    }
    f32x4 o[S];
#pragma unroll
    for (int s = 0; s < S; ++s) o[s] = zero;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (S > 1) asm volatile("" ::: "memory");   // the next block's weights are not read before this one is done
        f32x4 a[S], b[S];
#pragma unroll
        for (int s = 0; s < S; ++s) a[s] = b[s] = zero;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const bf16x8 wa = w.l2(2 * q, k, tile_unit(2 * q, c), g), wb = w.l2(2 * q + 1, k, tile_unit(2 * q + 1, c), g);
#pragma unroll
            for (int s = 0; s < S; ++s) {
                a[s] = mma(wa, h[s][k], a[s]);
                b[s] = mma(wb, h[s][k], b[s]);
            }
        }
        const f32x4 ba = *reinterpret_cast<const f32x4*>(b2 + 32 * q + 8 * g);
        const f32x4 bb = *reinterpret_cast<const f32x4*>(b2 + 32 * q + 8 * g + 4);
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const bf16x8 h2 = tanh8(a[s], b[s], ba, bb);
            const uint64_t st = s0 + 16 * s + c;
            if (ACT && act.h2 && st < n) {
                const u32x4 hv = __builtin_bit_cast(u32x4, h2);
                uint16_t* row = act.h2 + st * kHid + 32 * q + 8 * g;
                if (act_wide) *reinterpret_cast<u32x4*>(row) = hv;
                else
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        row[e] = (uint16_t)((e & 1) ? (hv[e >> 1] >> 16) : (hv[e >> 1] & 0xFFFFu));
            }
            o[s] = mma(w.l3(q, g, c), h2, o[s]);
        }
    }
    f32x4 own = o[0];
#pragma unroll
    for (int s = 1; s < S; ++s) own = g == s ? o[s] : own;
    return own;
}

// Features of a state whose up and down strings are packed as up | dn << 16:
// operand slot g holds sites 8g .. 8g + 7 of the 32.
__device__ __forceinline__ uint32_t pack_state(uint32_t up, uint32_t dn) { return (up & 0xFFFFu) | (dn << 16); }

__device__ __forceinline__ void write_out(float* out, uint64_t s, float o0, float o1) {
    out[2 * s] = o0;
    out[2 * s + 1] = o1;
}

// Forward pass over n states.  BASIS = false: outputs (n x 2) and, when
// act.h1 != NULL, the activations; BASIS = true (n < 2^32): the start vector
// v0[s] = sign * exp(min(o_0, 60)), sign = + for o_1 >= 0.
//
// Bound by the vector ALUs: 256 tanh a state, each five vector instructions,
// an exponential and a reciprocal.  A wave takes 64 states, so an operand of
// weights is read from LDS once for four products (40 KB of LDS reads per 64
// states; with 16 states a wave they would cost half as much as the ALU work).
// 1.31e8 states (4x4, 7 + 7): 19.2 ms with 16 states a wave, the hidden layer
// through LDS, scalar rounding to BF16 and the last layer on the vector ALUs;
// 9.6 ms with the last layer's four tiles in one accumulator behind masked
// weights, 9.4 ms so (576 TFLOP/s; the accumulators cost ten spilled registers).
constexpr int kFwdTiles = 4;             // state tiles of 16 per wave
constexpr int kFwdStates = 4 * 16 * kFwdTiles;   // states per work group and turn
template <typename T, bool BASIS>
__global__ __launch_bounds__(256, BASIS ? 3 : 2) void k_mlp_fwd(const uint16_t* __restrict__ prm, StateSrc src, uint64_t n,
                                                    float* __restrict__ out, Act act, int act_wide,
                                                    T* __restrict__ v0) {
    __shared__ __align__(16) uint16_t sW1[kHid * kLd1];
    __shared__ __align__(16) uint16_t sW2[kHid * kLd2];
    __shared__ __align__(16) uint16_t sW3[4 * kLd2];
    __shared__ __align__(16) uint16_t sF[256 * 8];   // the eight features of every byte of occupations
    __shared__ __align__(16) float sb1[kHid], sb2[kHid];
    const int tid = threadIdx.x;
    for (int i = tid; i < kHid * kIn; i += 256) sW1[(i / kIn) * kLd1 + (i % kIn)] = prm[oW1 + i];
    for (int i = tid; i < kHid * kHid; i += 256) sW2[(i / kHid) * kLd2 + (i % kHid)] = prm[oW2 + i];
    for (int i = tid; i < kHid; i += 256) {
        sb1[i] = bf2f(prm[oB1 + i]);
        sb2[i] = bf2f(prm[oB2 + i]);
    }
    for (int i = tid; i < 4 * kHid; i += 256) sW3[(i / kHid) * kLd2 + (i % kHid)] = i < kOut * kHid ? prm[oW3 + i] : 0;
    *reinterpret_cast<bf16x8*>(sF + 8 * tid) = feature8((uint32_t)tid);
    const int wave = tid >> 6, lane = tid & 63, g = lane >> 4, c = lane & 15;
    const float b30 = bf2f(prm[oB3]), b31 = bf2f(prm[oB3 + 1]);
    const WLds w{sW1, sW2, sW3};
    __syncthreads();
    for (uint64_t s0 = blockIdx.x * (uint64_t)kFwdStates + wave * (16 * kFwdTiles); s0 < n;
         s0 += (uint64_t)gridDim.x * kFwdStates) {
        const uint64_t own = s0 + lane, sa = own < n ? own : n - 1;
        uint32_t up, dn;
        state_of<BASIS>(src, sa, &up, &dn);
        const uint32_t occ = pack_state(up, dn);
        bf16x8 x[kFwdTiles];
#pragma unroll
        for (int s = 0; s < kFwdTiles; ++s)
            x[s] = ld8(sF + 8 * (((uint32_t)__shfl((int)occ, 16 * s + c) >> (8 * g)) & 255u));
        asm volatile("" ::: "memory");   // read the weights anew each turn: kept, they would not fit the registers
        const f32x4 o = mlp_layers<!BASIS, kFwdTiles>(w, x, sb1, sb2, g, c, s0, n, act, act_wide != 0);
        if (own < n) {
            const float o0 = o[0] + b30, o1 = o[1] + b31;
            if (BASIS) {
                const double a = exp((double)fminf(o0, 60.0f));
                v0[own] = (T)(o1 >= 0.0f ? a : -a);
            } else {
                write_out(out, own, o0, o1);
            }
        }
    }
}

// The same for a list of at most kFwdFew states, one wave per 16: at these
// sizes the time is latency, so a work group is one wave that holds the
// weights in registers (40 loads of 16 bytes a lane, all in flight at once,
// instead of staging them through LDS behind a barrier).  A training gradient
// of 4096 states took 74 us with the kernel above at 16 states a wave, 66 us
// with this one (nothing else changed).  Up to eight waves a CU, where the two
// meet (this one / the one above, us, without and with activations): 16,385
// states 8.2 / 11.3 and 11.8 / 15.4, 32,768 states 11.5 / 11.5 and 16.4 / 16.6,
// 40,000 states 16.0 / 11.7 and 21.2 / 18.4.  prm 16-byte aligned.
constexpr uint64_t kFwdFew = 32768;
__global__ __launch_bounds__(64) void k_mlp_fwd_few(const uint16_t* __restrict__ prm,
                                                    const uint32_t* __restrict__ occ, uint64_t n,
                                                    float* __restrict__ out, Act act, int act_wide) {
    __shared__ __align__(16) float sb1[kHid], sb2[kHid];
    const int lane = threadIdx.x, g = lane >> 4, c = lane & 15;
    const uint64_t s0 = blockIdx.x * 16ull, own = s0 + c, sa = own < n ? own : n - 1;
    const uint32_t st = pack_state(occ[2 * sa], occ[2 * sa + 1]);
    for (int i = lane; i < kHid; i += 64) {
        sb1[i] = bf2f(prm[oB1 + i]);
        sb2[i] = bf2f(prm[oB2 + i]);
    }
    WReg w;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int u = tile_unit(i, c);
        w.w1[i] = ld8(prm + oW1 + u * kIn + 8 * g);
#pragma unroll
        for (int k = 0; k < 4; ++k) w.w2[i][k] = ld8(prm + oW2 + u * kHid + 32 * k + 8 * g);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {   // rows of other tiles than the one there is stay zero
        const uint16_t none[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        w.w3[q] = c < kOut ? ld8(prm + oW3 + c * kHid + 32 * q + 8 * g) : pack8(none);
    }
    const bf16x8 x[1] = {feature8(st >> (8 * g))};
    __syncthreads();
    const f32x4 o = mlp_layers<true, 1>(w, x, sb1, sb2, g, c, s0, n, act, act_wide != 0);
    if (g == 0 && own < n) write_out(out, own, o[0] + bf2f(prm[oB3]), o[1] + bf2f(prm[oB3 + 1]));
}

// dout and the loss partial sums of one work group of BLOCK threads; with
// one work group (at most kLossOne states) partial is the loss itself.
constexpr uint64_t kLossOne = 8192;
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_mlp_loss(const float* __restrict__ out, const float* __restrict__ target,
                                                    uint64_t n, float* __restrict__ dout, double* partial,
                                                    double scale) {
    __shared__ double red[BLOCK / 64];
    double acc = 0.0;
    const float inv_n = 1.0f / (float)n;
    for (uint64_t s = blockIdx.x * (uint64_t)BLOCK + threadIdx.x; s < n; s += (uint64_t)gridDim.x * BLOCK) {
        const float a = out[2 * s], z = out[2 * s + 1];
        const float la = target[2 * s];
        const float y = target[2 * s + 1] > 0.0f ? 1.0f : 0.0f;
        const float d = a - la;
        const float sp = fmaxf(z, 0.0f) + log1pf(expf(-fabsf(z)));   // softplus(z)
        acc += (double)(d * d) + (double)sp - (double)(y * z);
        dout[2 * s] = 2.0f * d * inv_n;
        dout[2 * s + 1] = (1.0f / (1.0f + expf(-z)) - y) * inv_n;
    }
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) acc += __shfl_xor(acc, m);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = red[0];
        for (int i = 1; i < BLOCK / 64; ++i) t += red[i];
        partial[blockIdx.x] = t * scale;
    }
}

__global__ void k_sum_partials(const double* partial, int np, double scale, double* result) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        double s = 0.0;
        for (int i = 0; i < np; ++i) s += partial[i];
        *result = s * scale;
    }
}

// Backward over one slice of states per work group, in chunks of 64 states:
//   dz2 = (dout W3) (1 - h2^2), dz1 = (dz2 W2) (1 - h1^2)   (BF16, in LDS)
//   dW2 += dz2^T h1, dW1 += dz1^T x, b2 += dz2^T 1, b1 += dz1^T 1 on the matrix cores,
//   dW3 += dout^T h2, b3 += dout^T 1 in FP32.
// Wave w: states 16 (w & 3) .. + 15 of the chunk and half w >> 2 of the units
// for dz1; then the unit rows 16 w .. + 15 of the weight gradients, whose
// accumulators stay in registers over the chunks.  The slice's sums go to
// part[slice * kParams + k] (to grad itself when there is one slice).
//
// Bound by latency: at 4096 states a work group has one chunk, and its time is
// one round of loads, 16 + 40 products a wave and the stores of its partial
// gradient.  dz2 and dz1 never leave LDS; as kernels of their own (dz1, dz2
// through memory, then 16x16 gradient tiles with 16 dependent load rounds of
// 32 states each) these took 11 + 37 us at 4096 states; the whole gradient of
// 4096 states 66 us then, 30 us with this kernel and a one-launch loss.
constexpr int kBwdBlock = 512;
constexpr int kChunk = 64;             // states per chunk
constexpr int kMaxSlices = 256;        // one work group per CU
constexpr int kLdS = kChunk + 8;       // padded LDS row of a [unit][state] tile
__global__ __launch_bounds__(kBwdBlock) void k_mlp_bwd(const uint16_t* __restrict__ prm, int prm_wide,
                                                       const uint32_t* __restrict__ occ, uint64_t n, uint64_t slice_len,
                                                       Act act, const float* __restrict__ dout,
                                                       float* __restrict__ part) {
    __shared__ __align__(16) uint16_t sW2t[kHid * kLd2];   // sW2t[j][o] = W2[o][j]
    __shared__ __align__(16) uint16_t sZ2[kHid * kLdS], sZ1[kHid * kLdS], sH1[kHid * kLdS];
    __shared__ float sW3[kOut * kHid];
    __shared__ float sD[kChunk * kOut];
    __shared__ __align__(16) uint32_t sOcc[kChunk];
    __shared__ float sR[3][kHid * kOut];
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63, g = lane >> 4, c = lane & 15;
    const uint64_t b0 = blockIdx.x * slice_len;
    const uint64_t b1 = b0 + slice_len < n ? b0 + slice_len : n;
    // W2 transposed: a wave reads eight columns of 64 rows at a time
    for (int i = tid; i < kHid * kHid / 8; i += kBwdBlock) {
        const int o = i & (kHid - 1), j0 = 8 * (i >> 7);
        uint16_t v[8];
        if (prm_wide) {
            const u32x4 u = *reinterpret_cast<const u32x4*>(prm + oW2 + o * kHid + j0);
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = (uint16_t)((e & 1) ? (u[e >> 1] >> 16) : (u[e >> 1] & 0xFFFFu));
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = prm[oW2 + o * kHid + j0 + e];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) sW2t[(j0 + e) * kLd2 + o] = v[e];
    }
    if (tid < kOut * kHid) sW3[tid] = bf2f(prm[oW3 + tid]);
    const uint16_t one8[8] = {0x3F80, 0x3F80, 0x3F80, 0x3F80, 0x3F80, 0x3F80, 0x3F80, 0x3F80};   // BF16 1.0
    const bf16x8 ones = pack8(one8);
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 g2[8], g1[2], gb2 = zero, gb1 = zero;
#pragma unroll
    for (int t = 0; t < 8; ++t) g2[t] = zero;
    g1[0] = g1[1] = zero;
    float w30 = 0.f, w31 = 0.f, e0 = 0.f, e1 = 0.f;
    const int tile = wave & 3, half = wave >> 2;
    for (uint64_t s0 = b0; s0 < b1; s0 += kChunk) {   // b0, b1, n: multiples of 32
        if (s0 != b0) __syncthreads();   // the tiles of the chunk before are read
        // h1^T of the chunk: eight states per 16-byte load; states past the slice are zeros
        for (int i = tid; i < kHid * kChunk / 8; i += kBwdBlock) {
            const int j = i >> 3, sl = 8 * (i & 7);
            u32x4 v = {0u, 0u, 0u, 0u};
            if (s0 + sl < b1) v = *reinterpret_cast<const u32x4*>(act.h1t + (uint64_t)j * n + s0 + sl);
            *reinterpret_cast<u32x4*>(sH1 + j * kLdS + sl) = v;
        }
        if (tid < kChunk) {
            const uint64_t s = s0 + tid;
            const bool in = s < b1;
            sOcc[tid] = in ? pack_state(occ[2 * s], occ[2 * s + 1]) : 0u;
            const float d0 = in ? dout[2 * s] : 0.f, d1 = in ? dout[2 * s + 1] : 0.f;
            sD[2 * tid] = d0;
            sD[2 * tid + 1] = d1;
            e0 += d0;
            e1 += d1;
        }
        u32x4 hv[4];
        {
            const uint64_t s = s0 + 16 * tile + c;
#pragma unroll
            for (int kc = 0; kc < 4; ++kc)
                hv[kc] = s < b1 ? *reinterpret_cast<const u32x4*>(act.h2 + s * kHid + 32 * kc + 8 * g)
                                : u32x4{0u, 0u, 0u, 0u};
        }
        __syncthreads();
        // dz2 of state 16 tile + c, units 32kc + 8g + t, in operand layout
        bf16x8 A[4];
        const float d0 = sD[2 * (16 * tile + c)], d1 = sD[2 * (16 * tile + c) + 1];
#pragma unroll
        for (int kc = 0; kc < 4; ++kc) {
            const int o0 = 32 * kc + 8 * g;
            uint16_t v[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const uint32_t w = hv[kc][t >> 1];
                const float h2 = bf2f((uint16_t)((t & 1) ? (w >> 16) : (w & 0xFFFFu)));
                v[t] = f2bf((d0 * sW3[o0 + t] + d1 * sW3[kHid + o0 + t]) * (1.0f - h2 * h2));
            }
            if ((kc >> 1) == half)   // the two waves of a tile store one half each
#pragma unroll
                for (int t = 0; t < 8; ++t) sZ2[(o0 + t) * kLdS + 16 * tile + c] = v[t];
            A[kc] = pack8(v);
        }
        // dh1 = dz2 W2; accumulator rows: states 16 tile + 4g + t, column: unit j
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) {
            const int j = 64 * half + 16 * ct + c;
            f32x4 acc = zero;
#pragma unroll
            for (int kc = 0; kc < 4; ++kc) acc = mma(A[kc], ld8(sW2t + j * kLd2 + 32 * kc + 8 * g), acc);
            const uint2 h1w = *reinterpret_cast<const uint2*>(sH1 + j * kLdS + 16 * tile + 4 * g);
            uint16_t o[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const uint32_t w = (t < 2) ? h1w.x : h1w.y;
                const float h1 = bf2f((uint16_t)((t & 1) ? (w >> 16) : (w & 0xFFFFu)));
                o[t] = f2bf(acc[t] * (1.0f - h1 * h1));
            }
            uint2 st;
            st.x = o[0] | ((uint32_t)o[1] << 16);
            st.y = o[2] | ((uint32_t)o[3] << 16);
            *reinterpret_cast<uint2*>(sZ1 + j * kLdS + 16 * tile + 4 * g) = st;
        }
        // W3: unit tid mod 128, the chunk's states 16 (tid / 128) .. + 15
        {
            const int j = tid & (kHid - 1), q = tid >> 7;
            float h[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const uint64_t s = s0 + 16 * q + u;
                h[u] = s < b1 ? bf2f(act.h2[s * kHid + j]) : 0.f;
            }
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                w30 += sD[2 * (16 * q + u)] * h[u];
                w31 += sD[2 * (16 * q + u) + 1] * h[u];
            }
        }
        __syncthreads();
        // weight gradients of unit rows 16 wave + c over the chunk's states
#pragma unroll
        for (int k = 0; k < kChunk; k += 32) {
            const bf16x8 a2 = ld8(sZ2 + (16 * wave + c) * kLdS + k + 8 * g);
#pragma unroll
            for (int jt = 0; jt < 8; ++jt) g2[jt] = mma(a2, ld8(sH1 + (16 * jt + c) * kLdS + k + 8 * g), g2[jt]);
            gb2 = mma(a2, ones, gb2);
            const bf16x8 a1 = ld8(sZ1 + (16 * wave + c) * kLdS + k + 8 * g);
            const u32x4 oa = *reinterpret_cast<const u32x4*>(sOcc + k + 8 * g);
            const u32x4 ob = *reinterpret_cast<const u32x4*>(sOcc + k + 8 * g + 4);
#pragma unroll
            for (int it = 0; it < 2; ++it) {   // feature i = 16 it + c of states k + 8g + e: +1 where its bit is set
                u32x4 f;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t lo = e < 2 ? oa[2 * e] : ob[2 * e - 4], hi = e < 2 ? oa[2 * e + 1] : ob[2 * e - 3];
                    f[e] = 0xBF80BF80u ^ (((lo >> (16 * it + c)) & 1u) << 15) ^ (((hi >> (16 * it + c)) & 1u) << 31);
                }
                g1[it] = mma(a1, __builtin_bit_cast(bf16x8, f), g1[it]);
            }
            gb1 = mma(a1, ones, gb1);
        }
    }
    float* P = part + (size_t)blockIdx.x * kParams;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int o = 16 * wave + 4 * g + t;
#pragma unroll
        for (int jt = 0; jt < 8; ++jt) P[oW2 + o * kHid + 16 * jt + c] = g2[jt][t];
        P[oW1 + o * kIn + c] = g1[0][t];
        P[oW1 + o * kIn + 16 + c] = g1[1][t];
        if (c == 0) {   // every column of gb holds the row sums
            P[oB2 + o] = gb2[t];
            P[oB1 + o] = gb1[t];
        }
    }
    if (tid >= kHid) {
        sR[(tid >> 7) - 1][tid & (kHid - 1)] = w30;
        sR[(tid >> 7) - 1][kHid + (tid & (kHid - 1))] = w31;
    }
    __syncthreads();
    if (tid < kHid) {
        P[oW3 + tid] = ((w30 + sR[0][tid]) + sR[1][tid]) + sR[2][tid];
        P[oW3 + kHid + tid] = ((w31 + sR[0][kHid + tid]) + sR[1][kHid + tid]) + sR[2][kHid + tid];
    }
    if (wave == 0) {
#pragma unroll
        for (int m = 32; m > 0; m >>= 1) {
            e0 += __shfl_xor(e0, m);
            e1 += __shfl_xor(e1, m);
        }
        if (lane == 0) {
            P[oB3] = e0;
            P[oB3 + 1] = e1;
        }
    }
}

// Sum of the slices, one wave per 64 parameters and every fourth slice, the
// four sums combined in a fixed order.
__global__ __launch_bounds__(256) void k_mlp_grad_reduce(const float* __restrict__ part, int slices,
                                                         float* __restrict__ grad) {
    __shared__ float red[3][64];
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int k = blockIdx.x * 64 + lane;
    float s = 0.f;
    if (k < kParams) {
#pragma unroll 16
        for (int i = q; i < slices; i += 4) s += part[(size_t)i * kParams + k];
    }
    if (q > 0) red[q - 1][lane] = s;
    __syncthreads();
    if (q == 0 && k < kParams) grad[k] = ((s + red[0][lane]) + red[1][lane]) + red[2][lane];
}

__global__ __launch_bounds__(256) void k_adam(float* __restrict__ w, uint16_t* __restrict__ wb,
                                              const float* __restrict__ grad, float* __restrict__ m,
                                              float* __restrict__ v, uint64_t count, float lr, float b1, float b2,
                                              float eps, float c1, float c2) {
    const uint64_t k = blockIdx.x * 256ull + threadIdx.x;
    if (k >= count) return;
    const float gk = grad[k];
    const float mk = b1 * m[k] + (1.0f - b1) * gk;
    const float vk = b2 * v[k] + (1.0f - b2) * gk * gk;
    m[k] = mk;
    v[k] = vk;
    const float wk = w[k] - lr * (mk / c1) / (sqrtf(vk / c2) + eps);
    w[k] = wk;
    wb[k] = f2bf(wk);
}

__global__ __launch_bounds__(256) void k_to_bf16(const float* __restrict__ w, uint16_t* __restrict__ wb,
                                                 uint64_t count) {
    const uint64_t k = blockIdx.x * 256ull + threadIdx.x;
    if (k < count) wb[k] = f2bf(w[k]);
}

// ------------------------------------------------------------------ sampler

__device__ __forceinline__ uint64_t qweight(double p, double m) {
    return (uint64_t)floor(p * p / m * 4294967296.0);
}

__global__ __launch_bounds__(256) void k_max_sq(const double* __restrict__ psi, uint64_t D, double* partial) {
    __shared__ double red[256];
    double mx = 0.0;
    for (uint64_t i = blockIdx.x * 256ull + threadIdx.x; i < D; i += (uint64_t)gridDim.x * 256)
        mx = fmax(mx, psi[i] * psi[i]);
    red[threadIdx.x] = mx;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (threadIdx.x < st) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + st]);
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

__global__ void k_max_final(const double* partial, int np, double* result) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        double m = 0.0;
        for (int i = 0; i < np; ++i) m = fmax(m, partial[i]);
        *result = m;
    }
}

// sums[b] = sum of the weights of chunk b
__global__ __launch_bounds__(256) void k_chunk_sums(const double* __restrict__ psi, uint64_t D, const double* mx,
                                                    uint64_t* sums) {
    __shared__ uint64_t red[256];
    const double m = *mx;
    const uint64_t c0 = (uint64_t)blockIdx.x * kScanChunk;
    uint64_t acc = 0;
    for (uint64_t i = c0 + threadIdx.x; i < c0 + kScanChunk && i < D; i += 256) acc += qweight(psi[i], m);
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) sums[blockIdx.x] = red[0];
}

// exclusive scan of the chunk sums in place (one block), total in *total
__global__ __launch_bounds__(256) void k_scan_sums(uint64_t* sums, uint64_t nchunks, uint64_t* total) {
    __shared__ uint64_t sh[256];
    uint64_t carry = 0;
    for (uint64_t base = 0; base < nchunks; base += 256) {
        const uint64_t i = base + threadIdx.x;
        const uint64_t v = i < nchunks ? sums[i] : 0;
        sh[threadIdx.x] = v;
        __syncthreads();
        for (int off = 1; off < 256; off <<= 1) {   // inclusive Hillis-Steele scan
            const uint64_t add = threadIdx.x >= off ? sh[threadIdx.x - off] : 0;
            __syncthreads();
            sh[threadIdx.x] += add;
            __syncthreads();
        }
        if (i < nchunks) sums[i] = carry + sh[threadIdx.x] - v;
        carry += sh[255];
        __syncthreads();
    }
    if (threadIdx.x == 0) *total = carry;
}

// prefix[r] = inclusive prefix sum of the weights; 32 consecutive elements per thread
__global__ __launch_bounds__(256) void k_chunk_scan(const double* __restrict__ psi, uint64_t D, const double* mx,
                                                    const uint64_t* offs, uint64_t* __restrict__ prefix) {
    __shared__ uint64_t sh[256];
    const double m = *mx;
    const uint64_t c0 = (uint64_t)blockIdx.x * kScanChunk + (uint64_t)threadIdx.x * 32;
    uint64_t w[32];
    uint64_t tot = 0;
#pragma unroll
    for (int q = 0; q < 32; ++q) {
        const uint64_t i = c0 + q;
        w[q] = i < D ? qweight(psi[i], m) : 0;
        tot += w[q];
    }
    sh[threadIdx.x] = tot;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
        const uint64_t add = threadIdx.x >= off ? sh[threadIdx.x - off] : 0;
        __syncthreads();
        sh[threadIdx.x] += add;
        __syncthreads();
    }
    uint64_t run = offs[blockIdx.x] + sh[threadIdx.x] - tot;
#pragma unroll
    for (int q = 0; q < 32; ++q) {
        const uint64_t i = c0 + q;
        run += w[q];
        if (i < D) prefix[i] = run;
    }
}

__device__ __forceinline__ uint64_t splitmix_u64(uint64_t seed, uint64_t k) {
    uint64_t z = seed + (k + 1ull) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__global__ __launch_bounds__(256) void k_sample(const double* __restrict__ psi, const uint64_t* __restrict__ prefix,
                                                uint64_t D, const uint32_t* __restrict__ up_states,
                                                const uint32_t* __restrict__ dn_states, uint64_t D_dn, uint64_t seed,
                                                uint64_t first, uint64_t count, float gauge,
                                                uint32_t* __restrict__ occ, float* __restrict__ target,
                                                uint32_t* __restrict__ idx) {
    const uint64_t j = blockIdx.x * 256ull + threadIdx.x;
    if (j >= count) return;
    const uint64_t W = prefix[D - 1];
    const uint64_t t = __umul64hi(splitmix_u64(seed, first + j), W);
    uint64_t lo = 0, hi = D - 1;   // prefix[hi] = W > t
    while (lo < hi) {
        const uint64_t mid = lo + (hi - lo) / 2;
        if (prefix[mid] > t)
            hi = mid;
        else
            lo = mid + 1;
    }
    const uint64_t r = lo;
    const uint64_t iu = r / D_dn;
    occ[2 * j] = up_states[iu];
    occ[2 * j + 1] = dn_states[r - iu * D_dn];
    const double p = psi[r];
    target[2 * j] = (float)log(fabs(p));
    target[2 * j + 1] = (p * gauge > 0.0) ? 1.0f : -1.0f;
    if (idx) idx[j] = (uint32_t)r;
}

// ----------------------------------------------------------------- vectors

template <typename T>
__global__ __launch_bounds__(256) void k_vdot(const T* __restrict__ a, const T* __restrict__ b, uint64_t n,
                                              double* partial) {
    __shared__ double red[256];
    double acc = 0.0;
    for (uint64_t i = blockIdx.x * 256ull + threadIdx.x; i < n; i += (uint64_t)gridDim.x * 256)
        acc += (double)a[i] * (double)b[i];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

struct MlpWs {
    size_t part = 0, loss = 0, total = 0;
    int slices = 0;
    uint64_t slice_len = 0;   // states per slice, a multiple of kChunk
};
MlpWs mlp_ws(uint64_t n) {
    MlpWs w;
    const uint64_t chunks = (n + kChunk - 1) / kChunk;
    const uint64_t per = (chunks + kMaxSlices - 1) / kMaxSlices;   // chunks per slice
    w.slice_len = per * kChunk;
    w.slices = per ? (int)((chunks + per - 1) / per) : 0;
    size_t off = 0;
    w.part = off;
    off += al256((size_t)w.slices * kParams * 4);
    w.loss = off;
    off += al256(kLossBlocks * 8);
    w.total = off;
    return w;
}

struct SampWs {
    size_t prefix = 0, sums = 0, mx = 0, total = 0;
    uint64_t nchunks = 0;
};
SampWs samp_ws(uint64_t D) {
    SampWs w;
    w.nchunks = (D + kScanChunk - 1) / kScanChunk;
    size_t off = 0;
    w.prefix = off;
    off += al256((size_t)D * 8);
    w.sums = off;
    off += al256((size_t)(w.nchunks + 1) * 8);
    w.mx = off;
    off += al256(1024 * 8 + 8);
    w.total = off;
    return w;
}

// Work groups of the forward pass: as many as are resident, so that each walks the
// same number of turns.  Three a CU fit in the basis form (168 registers, 50 KB of
// LDS), two in the list form (244 registers): with three, list passes of 200,000,
// 262,144 and 400,000 states took 30.1, 31.3 and 46.5 us, with two 27.9, 28.8, 43.9.
int fwd_grid(uint64_t n, int per_cu) {
    DeviceCtx* ctx = nullptr;
    const int cu = (device_ctx(&ctx) == PDZ_OK && ctx) ? ctx->cu_count : 256;
    const uint64_t groups = (n + kFwdStates - 1) / kFwdStates;
    const uint64_t g = (uint64_t)cu * per_cu;
    return (int)(groups < g ? groups : g);
}

Act act_views(void* act, uint64_t n) {
    Act a;
    uint16_t* base = static_cast<uint16_t*>(act);
    a.h1 = base;
    a.h1t = base ? base + (size_t)n * kHid : nullptr;
    a.h2 = base ? base + 2 * (size_t)n * kHid : nullptr;
    return a;
}

}  // namespace
}  // namespace pdz

using namespace pdz;

namespace {

// Partial sums of pdz_dot_noalloc: one array per device, held until the
// process ends.  Host code reaches it only through the address
// hipGetSymbolAddress returns on each device (dot_scratch_ptr).
constexpr int kDotPartials = 1024;
static __device__ __align__(256) double scratch[kDotPartials];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {};

// Address of this device's array (the current device), looked up once per device.
pdz_status dot_scratch_ptr(double** out) {
    int dev = -1;
    PDZ_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(PDZ_EDEVICE, "device index outside the supported range");
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        PDZ_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) return fail(PDZ_EDEVICE, "no device address for the dot-product scratch array");
        g_scratch_ptr[dev] = static_cast<double*>(ptr);
    }
    *out = g_scratch_ptr[dev];
    return ok();
}

}  // namespace

extern "C" {

int32_t pdz_mlp_param_count(void) { return kParams; }

pdz_status pdz_mlp_init(float* params, uint16_t* params_bf16, uint64_t seed) {
    if (!params || !params_bf16) return fail(PDZ_EINVAL, "NULL argument");
    // weights uniform in +-1/sqrt(fan_in) from SplitMix64 output k of `seed`, biases zero
    std::vector<float> h(kParams, 0.0f);
    auto uni = [&](uint64_t k) {
        uint64_t z = seed + (k + 1ull) * 0x9E3779B97F4A7C15ull;
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        z = z ^ (z >> 31);
        return 2.0 * ((double)(z >> 11) * 0x1.0p-53) - 1.0;
    };
    for (int k = oW1; k < oB1; ++k) h[k] = (float)(uni(k) / std::sqrt((double)kIn));
    for (int k = oW2; k < oB2; ++k) h[k] = (float)(uni(k) / std::sqrt((double)kHid));
    for (int k = oW3; k < oB3; ++k) h[k] = (float)(uni(k) / std::sqrt((double)kHid));
    PDZ_HIP(hipMemcpy(params, h.data(), kParams * sizeof(float), hipMemcpyHostToDevice));
    hipLaunchKernelGGL(k_to_bf16, dim3((kParams + 255) / 256), dim3(256), 0, 0, params, params_bf16,
                       (uint64_t)kParams);
    PDZ_HIP(hipGetLastError());
    PDZ_HIP(hipDeviceSynchronize());
    return ok();
}

pdz_status pdz_mlp_to_bf16(const float* params, uint16_t* params_bf16, void* stream) {
    if (!params || !params_bf16) return fail(PDZ_EINVAL, "NULL argument");
    hipLaunchKernelGGL(k_to_bf16, dim3((kParams + 255) / 256), dim3(256), 0, (hipStream_t)stream, params,
                       params_bf16, (uint64_t)kParams);
    PDZ_HIP(hipGetLastError());
    return ok();
}

pdz_status pdz_mlp_forward(const uint16_t* params_bf16, const uint32_t* occ, uint64_t n, float* out, void* act,
                           void* stream) {
    if (!params_bf16 || !out || (n > 0 && !occ)) return fail(PDZ_EINVAL, "NULL argument");
    if (n == 0) return ok();
    if (n > (1ull << 32)) return fail(PDZ_ERANGE, "at most 2^32 states per call");
    StateSrc src{occ, nullptr, nullptr, 1};
    const Act a = act_views(act, n);
    const int act_wide = reinterpret_cast<uintptr_t>(act) % 16 == 0;   // 16-byte stores of the activations
    if (n <= kFwdFew && reinterpret_cast<uintptr_t>(params_bf16) % 16 == 0)
        hipLaunchKernelGGL(k_mlp_fwd_few, dim3((unsigned)((n + 15) / 16)), dim3(64), 0, (hipStream_t)stream,
                           params_bf16, occ, n, out, a, act_wide);
    else
        hipLaunchKernelGGL((k_mlp_fwd<float, false>), dim3(fwd_grid(n, 2)), dim3(256), 0, (hipStream_t)stream,
                           params_bf16, src, n, out, a, act_wide, (float*)nullptr);
    PDZ_HIP(hipGetLastError());
    return ok();
}

pdz_status pdz_mlp_workspace_size(uint64_t n, size_t* bytes) {
    if (!bytes) return fail(PDZ_EINVAL, "NULL argument");
    *bytes = mlp_ws(n).total;
    return ok();
}

pdz_status pdz_mlp_loss(const float* out, const float* target, uint64_t n, float* dout, double* loss, void* ws,
                        size_t ws_bytes, void* stream) {
    if (!out || !target || !dout || !loss || !ws) return fail(PDZ_EINVAL, "NULL argument");
    if (n == 0) return fail(PDZ_EINVAL, "empty batch");
    const MlpWs w = mlp_ws(n);
    if (ws_bytes < w.total) return fail(PDZ_EINVAL, "workspace smaller than pdz_mlp_workspace_size");
    double* part = reinterpret_cast<double*>(static_cast<char*>(ws) + w.loss);
    hipStream_t s = (hipStream_t)stream;
    // one launch while a work group has at most eight states a thread (the sum over work groups is a launch of its own)
    if (n <= kLossOne) {
        hipLaunchKernelGGL(k_mlp_loss<1024>, dim3(1), dim3(1024), 0, s, out, target, n, dout, loss, 1.0 / (double)n);
    } else {
        hipLaunchKernelGGL(k_mlp_loss<256>, dim3(kLossBlocks), dim3(256), 0, s, out, target, n, dout, part, 1.0);
        hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(64), 0, s, part, kLossBlocks, 1.0 / (double)n, loss);
    }
    PDZ_HIP(hipGetLastError());
    return ok();
}

pdz_status pdz_mlp_backward(const uint16_t* params_bf16, const uint32_t* occ, uint64_t n, const void* act,
                            const float* dout, float* grad, void* ws, size_t ws_bytes, void* stream) {
    if (!params_bf16 || !occ || !act || !dout || !grad || !ws) return fail(PDZ_EINVAL, "NULL argument");
    if (n == 0 || n % 32 != 0) return fail(PDZ_EINVAL, "the batch size must be a positive multiple of 32");
    if (n > (1ull << 24)) return fail(PDZ_ERANGE, "at most 2^24 states per training batch");
    const MlpWs w = mlp_ws(n);
    if (ws_bytes < w.total) return fail(PDZ_EINVAL, "workspace smaller than pdz_mlp_workspace_size");
    if (reinterpret_cast<uintptr_t>(ws) % 256 || reinterpret_cast<uintptr_t>(act) % 16)
        return fail(PDZ_EINVAL, "workspace must be 256-byte aligned and activations 16-byte aligned");
    char* base = static_cast<char*>(ws);
    float* part = reinterpret_cast<float*>(base + w.part);
    const Act a = act_views(const_cast<void*>(act), n);
    hipStream_t s = (hipStream_t)stream;
    const int prm_wide = reinterpret_cast<uintptr_t>(params_bf16) % 16 == 0;
    float* sums = w.slices == 1 ? grad : part;
    hipLaunchKernelGGL(k_mlp_bwd, dim3((unsigned)w.slices), dim3(kBwdBlock), 0, s, params_bf16, prm_wide, occ, n,
                       w.slice_len, a, dout, sums);
    if (w.slices > 1)
        hipLaunchKernelGGL(k_mlp_grad_reduce, dim3((kParams + 63) / 64), dim3(256), 0, s, part, w.slices, grad);
    PDZ_HIP(hipGetLastError());
    return ok();
}

pdz_status pdz_adam_step(float* params, uint16_t* params_bf16, const float* grad, float* m, float* v, uint64_t count,
                         float lr, float beta1, float beta2, float eps, int32_t step, void* stream) {
    if (!params || !params_bf16 || !grad || !m || !v) return fail(PDZ_EINVAL, "NULL argument");
    if (step < 1) return fail(PDZ_EINVAL, "step counts from 1");
    if (!(beta1 >= 0.f && beta1 < 1.f && beta2 >= 0.f && beta2 < 1.f && eps >= 0.f && std::isfinite(lr)))
        return fail(PDZ_EINVAL, "Adam hyper-parameters out of range");
    if (count == 0) return ok();
    const float c1 = (float)(1.0 - std::pow((double)beta1, step));
    const float c2 = (float)(1.0 - std::pow((double)beta2, step));
    hipLaunchKernelGGL(k_adam, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, (hipStream_t)stream, params,
                       params_bf16, grad, m, v, count, lr, beta1, beta2, eps, c1, c2);
    PDZ_HIP(hipGetLastError());
    return ok();
}

pdz_status pdz_sampler_workspace_size(pdz_problem p, size_t* bytes) {
    if (!p || !bytes) return fail(PDZ_EINVAL, "NULL argument");
    *bytes = samp_ws(p->D).total;
    return ok();
}

pdz_status pdz_sampler_prepare(pdz_problem p, const double* psi, void* ws, size_t ws_bytes, void* stream) {
    if (!p || !psi || !ws) return fail(PDZ_EINVAL, "NULL argument");
    const SampWs w = samp_ws(p->D);
    if (ws_bytes < w.total) return fail(PDZ_EINVAL, "workspace smaller than pdz_sampler_workspace_size");
    if (reinterpret_cast<uintptr_t>(ws) % 256) return fail(PDZ_EINVAL, "workspace must be 256-byte aligned");
    char* base = static_cast<char*>(ws);
    uint64_t* prefix = reinterpret_cast<uint64_t*>(base + w.prefix);
    uint64_t* sums = reinterpret_cast<uint64_t*>(base + w.sums);
    double* mx = reinterpret_cast<double*>(base + w.mx);   // [0] max, [1..1024] partials
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(k_max_sq, dim3(1024), dim3(256), 0, s, psi, p->D, mx + 1);
    hipLaunchKernelGGL(k_max_final, dim3(1), dim3(64), 0, s, mx + 1, 1024, mx);
    hipLaunchKernelGGL(k_chunk_sums, dim3((unsigned)w.nchunks), dim3(256), 0, s, psi, p->D, mx, sums);
    hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(256), 0, s, sums, w.nchunks, sums + w.nchunks);
    hipLaunchKernelGGL(k_chunk_scan, dim3((unsigned)w.nchunks), dim3(256), 0, s, psi, p->D, mx, sums, prefix);
    PDZ_HIP(hipGetLastError());
    return ok();
}

pdz_status pdz_sample(pdz_problem p, const double* psi, const void* ws, size_t ws_bytes, uint64_t seed,
                      uint64_t first, uint64_t count, double gauge, uint32_t* occ, float* target, uint32_t* idx,
                      void* stream) {
    if (!p || !psi || !ws || (count > 0 && (!occ || !target))) return fail(PDZ_EINVAL, "NULL argument");
    if (!(gauge == 1.0 || gauge == -1.0)) return fail(PDZ_EINVAL, "gauge must be +1 or -1");
    const SampWs w = samp_ws(p->D);
    if (ws_bytes < w.total) return fail(PDZ_EINVAL, "workspace smaller than pdz_sampler_workspace_size");
    if (count == 0) return ok();
    const uint64_t* prefix = reinterpret_cast<const uint64_t*>(static_cast<const char*>(ws) + w.prefix);
    hipLaunchKernelGGL(k_sample, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, (hipStream_t)stream, psi,
                       prefix, p->D, p->up.states, p->dn.states, p->dn.D, seed, first, count, (float)gauge, occ,
                       target, idx);
    PDZ_HIP(hipGetLastError());
    return ok();
}

pdz_status pdz_start_vector(pdz_problem p, const uint16_t* params_bf16, pdz_dtype dt, void* v0, void* stream) {
    if (!p || !params_bf16 || !v0) return fail(PDZ_EINVAL, "NULL argument");
    if (dt != PDZ_F64 && dt != PDZ_F32) return fail(PDZ_EINVAL, "dtype must be PDZ_F64 or PDZ_F32");
    if (p->N > 16) return fail(PDZ_ERANGE, "the network reads 16 sites per spin");
    StateSrc src{nullptr, p->up.states, p->dn.states, p->dn.D};
    const Act none = act_views(nullptr, 0);
    hipStream_t s = (hipStream_t)stream;
    if (dt == PDZ_F64)
        hipLaunchKernelGGL((k_mlp_fwd<double, true>), dim3(fwd_grid(p->D, 3)), dim3(256), 0, s, params_bf16, src, p->D,
                           (float*)nullptr, none, 0, static_cast<double*>(v0));
    else
        hipLaunchKernelGGL((k_mlp_fwd<float, true>), dim3(fwd_grid(p->D, 3)), dim3(256), 0, s, params_bf16, src, p->D,
                           (float*)nullptr, none, 0, static_cast<float*>(v0));
    PDZ_HIP(hipGetLastError());
    return ok();
}

pdz_status pdz_dot(pdz_dtype dt, const void* a, const void* b, uint64_t n, double* result, void* stream) {
    if (!a || !b || !result) return fail(PDZ_EINVAL, "NULL argument");
    if (dt != PDZ_F64 && dt != PDZ_F32) return fail(PDZ_EINVAL, "dtype must be PDZ_F64 or PDZ_F32");
    hipStream_t s = (hipStream_t)stream;
    double* d = nullptr;
    PDZ_HIP(hipMallocAsync((void**)&d, 1025 * sizeof(double), s));
    if (dt == PDZ_F64)
        hipLaunchKernelGGL(k_vdot<double>, dim3(1024), dim3(256), 0, s, static_cast<const double*>(a),
                           static_cast<const double*>(b), n, d + 1);
    else
        hipLaunchKernelGGL(k_vdot<float>, dim3(1024), dim3(256), 0, s, static_cast<const float*>(a),
                           static_cast<const float*>(b), n, d + 1);
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(64), 0, s, d + 1, 1024, 1.0, d);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(result, d, sizeof(double), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    (void)hipFreeAsync(d, s);
    (void)hipStreamSynchronize(s);
    if (e != hipSuccess) return hip_fail(e, "pdz_dot");
    return ok();
}

pdz_status pdz_dot_noalloc(pdz_dtype dt, const void* a, const void* b, uint64_t n, double* result, void* stream) {
    if (!a || !b || !result) return fail(PDZ_EINVAL, "NULL argument");
    if (dt != PDZ_F64 && dt != PDZ_F32) return fail(PDZ_EINVAL, "dtype must be PDZ_F64 or PDZ_F32");
    double* part = nullptr;
    pdz_status st = dot_scratch_ptr(&part);
    if (st != PDZ_OK) return st;
    hipStream_t s = (hipStream_t)stream;
    // every one of the kDotPartials work groups writes its partial sum, so
    // nothing of the previous call's contents is read
    if (dt == PDZ_F64)
        hipLaunchKernelGGL(k_vdot<double>, dim3(kDotPartials), dim3(256), 0, s, static_cast<const double*>(a),
                           static_cast<const double*>(b), n, part);
    else
        hipLaunchKernelGGL(k_vdot<float>, dim3(kDotPartials), dim3(256), 0, s, static_cast<const float*>(a),
                           static_cast<const float*>(b), n, part);
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(64), 0, s, part, kDotPartials, 1.0, result);
    PDZ_HIP(hipGetLastError());
    return ok();
}

}  // extern "C"
