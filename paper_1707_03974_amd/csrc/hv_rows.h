// H.v over short rows (fewer than 1024 down states), whole in one pass: the
// tile of one work group, shared by the single-problem and the batched kernel.
//
// A tile is a few rows u0 .. u0 + nrows - 1 of X.  They are staged in LDS in
// groups of RV rows, element d of a group's rows side by side, so one read of
// RV elements gathers a hop target for all RV rows.  A wave takes 64 columns of
// one row group at a time; each lane owns one column:
//   diagonal;
//   down hops: a table entry and its amplitude serve RV rows;
//   up hops: the rows' hop lists are the same for every lane, so lane l loads
//     one entry of one row's list (RV lists of 64 / RV slots in one load),
//     and each hop's source row and amplitude are broadcast to scalar
//     registers: per hop and row one coalesced load and one multiply-add.
// Every element is summed by one lane: diagonal, down hops, up hops, each in
// table order, with the roundings of the two-pass H.v (k_hv.hip), so both give
// the same bits.
//
// Bound by latency on one cluster (a wave's chain is stage, entries, gathers,
// up loads) and by the LDS gathers and L2 reads of the up hops on many.
#pragma once

#include <type_traits>

#include "pdz_internal.h"

namespace pdz {

template <typename T>
struct RowsProb {
    uint64_t D_up, D_dn;
    uint64_t pitch;               // elements from one row of x and y to the next
    const uint32_t* up_states;
    const uint32_t* dn_states;
    const uint8_t* up_count;
    const uint8_t* dn_count;
    const uint32_t* up_ell;       // 32-bit hop tables, slot major
    const uint32_t* dn_ell;
    T U;
    int dn_max;                   // most hops out of a down state
};

constexpr int kRowsHops = 8;   // hops whose loads are in flight together
constexpr uint64_t kRowsMinDn = 33;   // a shorter row leaves half of every wave idle or more

__device__ __forceinline__ float rows_readlane(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ double rows_readlane(double v, int l) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                            __builtin_amdgcn_readlane(__double2loint(v), l));
}
// x at byte offset voff (per lane) + soff (scalar): one instruction, no address arithmetic
__device__ __forceinline__ float rows_load(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, float) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}
__device__ __forceinline__ double rows_load(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, double) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}

// Up hops of slots s .. s + NB - 1 of the loaded lists (lane row * HS + slot:
// byte offset of the source row, amplitude): every row's loads, then the
// multiply-adds in order.  left[r]: hops row r still has from slot s on; a slot
// past them holds the row itself and is loaded but not added.  ALL: none is.
template <typename T, int RV, int NB, bool ALL>
__device__ __forceinline__ void rows_up_batch(T (&acc)[RV], const int (&left)[RV], int s, uint32_t off, T amp,
                                              __amdgpu_buffer_rsrc_t x, uint32_t dbytes) {
    constexpr int HS = 64 / RV;
    T v[RV][NB];
#pragma unroll
    for (int r = 0; r < RV; ++r)
#pragma unroll
        for (int j = 0; j < NB; ++j)
            v[r][j] = rows_load(x, dbytes, (uint32_t)__builtin_amdgcn_readlane((int)off, r * HS + s + j), T(0));
    if (!ALL) {   // every load is issued before the first branch
#pragma unroll
        for (int r = 0; r < RV; ++r)
#pragma unroll
            for (int j = 0; j < NB; ++j) asm volatile("" : "+v"(v[r][j]));
    }
#pragma unroll
    for (int r = 0; r < RV; ++r)
#pragma unroll
        for (int j = 0; j < NB; ++j)
            if (ALL || j < left[r]) acc[r] = fma(rows_readlane(amp, r * HS + s + j), v[r][j], acc[r]);
}

// One tile of BLOCK threads; coef: the amplitudes in LDS; lds: room for
// ceil(nrows / RV) * (D_dn + 1) groups of RV elements.  x, y: first element of
// the problem's vectors; D_up * pitch * sizeof(T) < 2^32.  Returns the lane's
// part of the tile's x . y (FP64).
template <typename T, int RV, int BLOCK>
__device__ __forceinline__ double rows_tile(const RowsProb<T>& p, uint32_t u0, uint32_t nrows, const T* coef,
                                            unsigned char* lds, const T* __restrict__ x, T* __restrict__ y) {
    constexpr int HS = 64 / RV;
    typedef T vec __attribute__((ext_vector_type(RV)));
    vec* rows = reinterpret_cast<vec*>(lds);
    const uint32_t D_dn = (uint32_t)p.D_dn, pitch = (uint32_t)p.pitch, D_up = (uint32_t)p.D_up;
    const uint32_t ng = (nrows + RV - 1) / RV, gpitch = D_dn + 1;
    const int lane = threadIdx.x & 63;
    const uint32_t nch = (D_dn + 63) / 64, items = ng * nch;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<T*>(x), 0, (int)(D_up * pitch * (uint32_t)sizeof(T)), 0x00020000);
    // stage: rows past the tile's last are zeros; group element D_dn is -0.0,
    // which a hop slot past a column's count adds with amplitude 1: no change
    for (uint32_t it = wave; it < items; it += BLOCK / 64) {
        const uint32_t g = ng == 1 ? 0u : it / nch, d = (it - g * nch) * 64 + lane;
        if (d < D_dn) {
            vec v;
#pragma unroll
            for (int r = 0; r < RV; ++r)
                v[r] = g * RV + r < nrows ? x[(u0 + g * RV + r) * pitch + d] : (T)0;
            rows[g * gpitch + d] = v;
        }
    }
    for (uint32_t g = threadIdx.x; g < ng; g += BLOCK) rows[g * gpitch + D_dn] = (vec)(T)(-0.0);
    __syncthreads();
    double dsum = 0.0;
    for (uint32_t it = wave; it < items; it += BLOCK / 64) {
        const uint32_t g = ng == 1 ? 0u : it / nch, d = (it - g * nch) * 64 + lane;
        const bool on = d < D_dn;
        const uint32_t dc = on ? d : D_dn - 1;
        const uint32_t ug = u0 + g * RV;
        const int nr = (int)min((uint32_t)RV, nrows - g * RV);
        // the rows' up-hop lists: lane l holds slot l % HS of row l / HS
        const uint32_t lr = min(ug + (uint32_t)(lane / HS), ug + (uint32_t)nr - 1);
        const int lcnt = lane / HS < nr ? (int)p.up_count[lr] : 0;
        const uint32_t lpu = p.up_states[lr];
        const uint32_t pd = p.dn_states[dc];
        const int cd = on ? (int)p.dn_count[dc] : 0;
        auto list = [&](int slot0, uint32_t* off, T* amp) {
            const int h = slot0 + lane % HS;
            *off = lr * pitch * (uint32_t)sizeof(T);
            *amp = (T)0;
            if (h < lcnt) {
                const uint32_t e = p.up_ell[(uint64_t)h * D_up + lr];
                *off = (e & kTargetMask) * pitch * (uint32_t)sizeof(T);
                *amp = coef[e >> kTargetBits];
            }
        };
        uint32_t off;
        T amp;
        list(0, &off, &amp);
        int cnt[RV];
#pragma unroll
        for (int r = 0; r < RV; ++r) cnt[r] = __builtin_amdgcn_readlane(lcnt, r * HS);
        // diagonal
        const vec* grp = rows + g * gpitch;
        const vec own = grp[dc];
        T acc[RV];
#pragma unroll
        for (int r = 0; r < RV; ++r) {
            const uint32_t pu = (uint32_t)__builtin_amdgcn_readlane((int)lpu, r * HS);
            acc[r] = p.U * (T)__builtin_popcount(pu & pd) * own[r];
            // keep the roundings of the two-pass H.v: no term is contracted with the next kind
            asm volatile("" : "+v"(acc[r]));
        }
        // down hops: kRowsHops table entries, then their gathers, then the multiply-adds
        const int cmax = p.dn_max;
        const auto down = [&](int h, auto all) {
            constexpr bool ALL = decltype(all)::value;
            uint32_t e[kRowsHops];
            T c[kRowsHops];
            vec v[kRowsHops];
#pragma unroll
            for (int j = 0; j < kRowsHops; ++j)   // past the table's last slot: that slot again, not used
                e[j] = (p.dn_ell + (uint64_t)(ALL ? h + j : min(h + j, cmax - 1)) * D_dn)[dc];
#pragma unroll
            for (int j = 0; j < kRowsHops; ++j) {
                const bool in = ALL || h + j < cd;
                c[j] = coef[in ? e[j] >> kTargetBits : 0u];
                v[j] = grp[in ? e[j] & kTargetMask : D_dn];
                if (!ALL) c[j] = in ? c[j] : (T)1;
            }
#pragma unroll
            for (int j = 0; j < kRowsHops; ++j)
#pragma unroll
                for (int r = 0; r < RV; ++r) acc[r] = fma(c[j], v[j][r], acc[r]);
        };
        int h = 0;
        while (h + kRowsHops <= cmax && __all(!on || h + kRowsHops <= cd)) {
            down(h, std::true_type{});
            h += kRowsHops;
        }
        for (; __any(h < cd); h += kRowsHops) down(h, std::false_type{});
#pragma unroll
        for (int r = 0; r < RV; ++r) asm volatile("" : "+v"(acc[r]));
        // up hops
        const uint32_t db = dc * (uint32_t)sizeof(T);
        int least = cnt[0], most = cnt[0];
#pragma unroll
        for (int r = 1; r < RV; ++r) {
            least = min(least, cnt[r]);
            most = max(most, cnt[r]);
        }
        for (int s0 = 0; s0 < most; s0 += HS) {
            if (s0 > 0) list(s0, &off, &amp);
            int s = 0, left[RV];
            for (; s + kRowsHops <= min(least - s0, HS); s += kRowsHops)
                rows_up_batch<T, RV, kRowsHops, true>(acc, left, s, off, amp, xr, db);
            const int end = min(most - s0, HS);
            while (s < end) {
#pragma unroll
                for (int r = 0; r < RV; ++r) left[r] = cnt[r] - s0 - s;
                if (end - s > kRowsHops / 2) {
                    rows_up_batch<T, RV, kRowsHops, false>(acc, left, s, off, amp, xr, db);
                    s += kRowsHops;
                } else {
                    rows_up_batch<T, RV, kRowsHops / 2, false>(acc, left, s, off, amp, xr, db);
                    s += kRowsHops / 2;
                }
            }
        }
        if (on) {
#pragma unroll
            for (int r = 0; r < RV; ++r)
                if (r < nr) {
                    y[(ug + r) * pitch + d] = acc[r];
                    dsum += (double)own[r] * (double)acc[r];
                }
        }
    }
    return dsum;
}

}  // namespace pdz
