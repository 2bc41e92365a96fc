// Per-lane state of the rescaled Legendre recurrence shared by the temperature and the
// polarization kernels: mu_l = A_lm z mu_{l-1} - mu_{l-2}, lambda_lm = c_lm mu_lm, started
// at the block of l that holds each (m, ring pair)'s first non-negligible value.
#pragma once

#include "mfwf_internal.h"

namespace mfwf {

static constexpr int kW = 64;  // wavefront

__device__ __forceinline__ int wave_min_uniform(int v) {
    for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o));
    return __builtin_amdgcn_readfirstlane(v);
}
__device__ __forceinline__ int wave_max_uniform(int v) {
    for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o));
    return __builtin_amdgcn_readfirstlane(v);
}

// A row of one m is walked in blocks of kLegBlock values of l from l = m.  A pair enters it at
// the block that holds its first l with |lambda_lm| >= 2^-100, from the state
// (mu_{l0-1}, mu_{l0-2}) at that block's first value l0 (0, -mu_m at l0 = m, where A_lm = 0), so
// a start is a load of two registers between blocks and no value of l inside a block tests
// for one: with a test and four selects at every l the blocks that can hold a start cost 9
// vector instructions per (l, pair) instead of 4.
static constexpr int kLegBlock = 16;

template <int P>
struct PairState {
    double z[P], u1[P], u2[P];  // mu_{l-1}, mu_{l-2}
    double2 ent[P];             // state at the pair's first block
    int kb[P];                  // its first block
    int klo, khi;               // wave-uniform: smallest first block, largest one of the row's

    __device__ __forceinline__ void load(int m, int g, int npair, int nblk,
                                         const double *__restrict__ zp,
                                         const int *__restrict__ kstart,
                                         const double2 *__restrict__ entry) {
        int mylo = nblk, myhi = -1;
#pragma unroll
        for (int k = 0; k < P; k++) {
            const int p = g * kW * P + k * kW + (int)threadIdx.x;
            const bool valid = p < npair;
            z[k] = valid ? zp[p] : 0.0;
            kb[k] = valid ? kstart[(long)m * npair + p] : nblk;
            ent[k] = valid ? entry[(long)m * npair + p] : make_double2(0.0, 0.0);
            u1[k] = 0.0;
            u2[k] = 0.0;
            mylo = min(mylo, kb[k]);
            if (kb[k] < nblk) myhi = max(myhi, kb[k]);
        }
        klo = wave_min_uniform(mylo);
        khi = wave_max_uniform(myhi);
    }

    // at the start of block k: the pairs whose first block it is take their state
    __device__ __forceinline__ void enter(int blk) {
        if (blk > khi) return;  // uniform
#pragma unroll
        for (int k = 0; k < P; k++)
            if (kb[k] == blk) {
                u1[k] = ent[k].x;
                u2[k] = ent[k].y;
            }
    }

    // mu_l for every pair (0 before the pair's first block)
    __device__ __forceinline__ void step(double A, double (&cur)[P]) {
#pragma unroll
        for (int k = 0; k < P; k++) {
            const double v = fma(A, z[k] * u1[k], -u2[k]);
            u2[k] = u1[k];
            u1[k] = v;
            cur[k] = v;
        }
    }
};

// Workgroup L of an FP64 Legendre launch of ngrp pair groups x nmi rows (or row pairs).
// Workgroup L runs on XCD L mod 8; every XCD takes whole chunks of 8 adjacent m (a 128-byte
// line of a ring's coefficients, so that a line meets in one L2) from all pair groups, the
// equatorial groups (whose pairs start first and carry the most values of l) before the
// polar ones.  With the group as the fastest index instead, 8 groups put all rows of one
// group on one XCD and the equatorial one finished last by a third.
struct LegItem {
    int g, mi;
};
__host__ __device__ __forceinline__ int leg_items_per_group(int nmi) { return (((nmi + 7) / 8 + 7) / 8) * 8; }
__device__ __forceinline__ LegItem leg_item(int ngrp, int nmi) {
    const int L = blockIdx.x, x = L & 7, s = L >> 3, w = leg_items_per_group(nmi);
    const int q = s / w, t = s - q * w;
    return LegItem{ngrp - 1 - q, ((t >> 3) * 8 + x) * 8 + (t & 7)};
}
static inline dim3 leg_grid(int ngrp, int nmi, int nb) {
    return dim3(8 * leg_items_per_group(nmi) * ngrp, nb);
}

// (x, y) of every lane after exchanging lanes 32..63 of x with lanes 0..31 of y (SWAP32),
// or the odd 16-lane rows of x with the even rows of y (v_permlane{32,16}_swap, one 32-bit
// half at a time): x + y then holds x summed over lanes L and L + 32 (L + 16) in the lower
// lanes (even rows) and y summed over L - 32 (L - 16) and L in the upper lanes (odd rows).
template <bool SWAP32>
__device__ __forceinline__ double swap_add(double x, double y) {
    const unsigned long long a = __double_as_longlong(x), b = __double_as_longlong(y);
    const unsigned alo = (unsigned)a, ahi = (unsigned)(a >> 32), blo = (unsigned)b, bhi = (unsigned)(b >> 32);
    unsigned xl, yl, xh, yh;
    if constexpr (SWAP32) {
        const auto l = __builtin_amdgcn_permlane32_swap(alo, blo, false, false);
        const auto h = __builtin_amdgcn_permlane32_swap(ahi, bhi, false, false);
        xl = l[0], yl = l[1], xh = h[0], yh = h[1];
    } else {
        const auto l = __builtin_amdgcn_permlane16_swap(alo, blo, false, false);
        const auto h = __builtin_amdgcn_permlane16_swap(ahi, bhi, false, false);
        xl = l[0], yl = l[1], xh = h[0], yh = h[1];
    }
    return __longlong_as_double(((unsigned long long)xh << 32) | xl) +
           __longlong_as_double(((unsigned long long)yh << 32) | yl);
}

}  // namespace mfwf
