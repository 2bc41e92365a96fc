// Legendre steps of the SHT, FP64 on the vector ALUs (Sect. 3 names the transforms as the
// cost driver, O(nside lmax^2)).
//
//   synthesis  F_{N/S,r}(m) = E_r(m) +/- O_r(m),
//              E = sum_{l+m even} lambda_lm(z_r) s_lm,   O = sum_{l+m odd} lambda_lm(z_r) s_lm
//   analysis   a_lm = sum_pairs lambda_lm(z_r) (G_N + (-1)^{l+m} G_S)_r(m)
//
// lambda_lm(-z) = (-1)^{l+m} lambda_lm(z), so one recurrence serves the north and south
// ring of a pair.  The orthonormal recurrence
//     lambda_l = alpha_lm z lambda_{l-1} - beta_lm lambda_{l-2}
// is run in the rescaled form lambda_l = c_lm mu_l with c_l = beta_l c_{l-2}
// (c_m = c_{m+1} = 1), which turns it into
//     mu_l = A_lm z mu_{l-1} - mu_{l-2},   A_lm = alpha_lm c_{l-1} / c_l,
// two FP64 operations per (l, ring pair) instead of three.  The synthesis reads the
// c-scaled coefficients c_lm s_lm and the analysis returns sum mu_l X, which the harmonic
// kernel multiplies by c_lm.  Each (m, pair) contributes from the block of kLegBlock values of l
// that holds the first |lambda_lm| >= 2^-100, from a host-computed recurrence state entering
// the block; earlier blocks are below 2^-100 and are dropped, and a pair carries mu = 0 (no
// contribution) before its start.
//
// What bounds both kernels is FP64 issue (about 5 cycles per wave instruction): four to six
// instructions per (l, pair), in the analysis plus the lane reduction.  With starts tested
// once a block and equal work per XCD, synthesis / analysis of one map went from 123 / 188 to
// 100 / 138 us at nside 512, lmax 1024, and from 711 / 1114 to 515 / 829 us at nside 1024.
//
// Work split: one 64-lane wave per (pair group g, m) or (pair group g, m and lmax - m);
// lane L handles ring pairs g*64*P + k*64 + L, k < P (adjacent lanes = adjacent latitudes, so
// first blocks are close).  Two rows per wave balance the triangle (every wave walks lmax + 2
// values of l), one row per wave gives twice the waves where there are few.
// The l loop is wave-uniform: its bounds come through readfirstlane, so it runs on the
// scalar unit and A_lm and the coefficients of each l are scalar loads.  Blocks of kLegBlock
// values of l start at l = m, so the even/odd split is fixed at compile time inside a block
// and pairs start between blocks.  The analysis reduces over the wave's lanes once per block
// (fixed order, deterministic).
#include <type_traits>

#include "leg_core.h"

namespace mfwf {

// ---------------------------------------------------------------------------------------
// Synthesis
// ---------------------------------------------------------------------------------------
template <int P>
struct SynthAcc {
    double Er[P], Ei[P], Or[P], Oi[P];
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int k = 0; k < P; k++) Er[k] = Ei[k] = Or[k] = Oi[k] = 0.0;
    }
    template <bool ODD>
    __device__ __forceinline__ void add(const double (&cur)[P], double2 a) {
#pragma unroll
        for (int k = 0; k < P; k++) {
            if (ODD) {
                Or[k] = fma(cur[k], a.x, Or[k]);
                Oi[k] = fma(cur[k], a.y, Oi[k]);
            } else {
                Er[k] = fma(cur[k], a.x, Er[k]);
                Ei[k] = fma(cur[k], a.y, Ei[k]);
            }
        }
    }
};

template <int P, int U>
__device__ __forceinline__ void synth_one_m(int m, int g, const double2 *__restrict__ alm,
                                            const double *__restrict__ Atab,
                                            const long *__restrict__ mofs,
                                            const int *__restrict__ kstart,
                                            const double2 *__restrict__ entry,
                                            const double *__restrict__ zp,
                                            double2 *__restrict__ phase, int lmax, int npair,
                                            int nring, int nm) {
    PairState<P> st;
    const int nblk = (lmax - m + kLegBlock) / kLegBlock;
    st.load(m, g, npair, nblk, zp, kstart, entry);
    const long off = mofs[m];
    const double *Am = Atab + off;
    const double2 *am = alm + off;
    SynthAcc<P> acc;
    acc.zero();
    const int nl = lmax - m + 1;  // values of l, from r = l - m = 0
    int r = st.klo * kLegBlock;
    for (; r + kLegBlock <= nl; r += kLegBlock) {
        st.enter(r / kLegBlock);
#pragma unroll
        for (int h = 0; h < kLegBlock; h += U) {
            double A[U];
            double2 a[U];
#pragma unroll
            for (int u = 0; u < U; u++) {
                A[u] = Am[r + h + u];
                a[u] = am[r + h + u];
            }
#pragma unroll
            for (int u = 0; u < U; u++) {
                double cur[P];
                st.step(A[u], cur);
                if (u & 1) acc.template add<true>(cur, a[u]);
                else acc.template add<false>(cur, a[u]);
            }
        }
    }
    if (r < nl) st.enter(r / kLegBlock);
    for (; r < nl; r++) {  // the last, partial block
        double cur[P];
        st.step(Am[r], cur);
        if (r & 1) acc.template add<true>(cur, am[r]);
        else acc.template add<false>(cur, am[r]);
    }
#pragma unroll
    for (int k = 0; k < P; k++) {
        const int p = g * kW * P + k * kW + (int)threadIdx.x;
        if (p >= npair) continue;
        const int rN = p, rS = nring - 1 - p;
        double2 *out = phase + m;  // ring-Fourier layout [map][ring][m]
        out[(long)rN * nm] = make_double2(acc.Er[k] + acc.Or[k], acc.Ei[k] + acc.Oi[k]);
        if (rS != rN)
            out[(long)rS * nm] = make_double2(acc.Er[k] - acc.Or[k], acc.Ei[k] - acc.Oi[k]);
    }
}

// ROWS: values of m per wave (2: m and lmax - m)
template <int P, int U, int ROWS>
__global__ void __launch_bounds__(kW)
k_leg_synth(const double2 *__restrict__ alm, long nalm, const double *__restrict__ Atab,
            const long *__restrict__ mofs, const int *__restrict__ kstart,
            const double2 *__restrict__ entry, const double *__restrict__ zp,
            double2 *__restrict__ phase, int lmax, int npair, int nring, int nm, int ngrp) {
    const int nmi = ROWS == 2 ? (lmax + 2) / 2 : nm;
    const LegItem it = leg_item(ngrp, nmi);
    if (it.mi >= nmi) return;
    const int b = blockIdx.y;
    const int npass = (ROWS == 2 && lmax - it.mi > it.mi) ? 2 : 1;
    for (int pass = 0; pass < npass; pass++)
        synth_one_m<P, U>(pass == 0 ? it.mi : lmax - it.mi, it.g, alm + (long)b * nalm, Atab, mofs,
                          kstart, entry, zp, phase + (long)b * nm * nring, lmax, npair, nring, nm);
}

// ---------------------------------------------------------------------------------------
// Analysis
// ---------------------------------------------------------------------------------------
static constexpr int kAnaV = 2 * kLegBlock;  // doubles reduced per lane per block (re, im)
static constexpr int kAnaQ = kAnaV / 4;      // doubles per lane after the two lane swaps
// LDS slot of a lane's reduced values: 8 doubles of padding after every 8 lanes put the
// eight (row, half) groups that read at once on four different bank quarters
__device__ __forceinline__ int ana_slot(int lane) { return (lane + (lane >> 3)) * kAnaQ; }
static constexpr int kAnaLds = (kW + kW / 8) * kAnaQ;

// the block's values summed over the wave's 64 lanes: two lane swaps halve the values a lane
// holds twice (the 16-lane row r = L / 16 then holds values Q r .. Q r + Q - 1, each summed over
// four lanes), then through LDS lane L sums value L / 2 over half L % 2 of its row
__device__ __forceinline__ double ana_reduce(double (&acc)[kAnaV], double *red) {
#pragma unroll
    for (int i = 0; i < kAnaV / 2; i++) acc[i] = swap_add<true>(acc[i], acc[i + kAnaV / 2]);
#pragma unroll
    for (int i = 0; i < kAnaQ; i++) acc[i] = swap_add<false>(acc[i], acc[i + kAnaQ]);
    double *w = red + ana_slot(threadIdx.x);
#pragma unroll
    for (int i = 0; i < kAnaQ; i += 2)
        *reinterpret_cast<double2 *>(w + i) = make_double2(acc[i], acc[i + 1]);
    __syncthreads();
    const int v = threadIdx.x >> 1, h = threadIdx.x & 1, r = v / kAnaQ, j = v - kAnaQ * r;
    const double *x = red + ana_slot(16 * r + 8 * h) + j;
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < 8; q++) s += x[q * kAnaQ];
    s += __shfl_xor(s, 1);
    __syncthreads();
    return s;
}

template <int P>
__device__ __forceinline__ void analysis_one_m(int m, int g, const double2 *__restrict__ phase,
                                               int nring, int nm, const double *__restrict__ Atab,
                                               const long *__restrict__ mofs,
                                               const int *__restrict__ kstart,
                                               const double2 *__restrict__ entry,
                                               const double *__restrict__ zp,
                                               double2 *__restrict__ apart, int lmax, int npair,
                                               double *red) {
    PairState<P> st;
    const int nl = lmax - m + 1, nblk = (nl + kLegBlock - 1) / kLegBlock;
    st.load(m, g, npair, nblk, zp, kstart, entry);
    const long off = mofs[m];
    const double *Am = Atab + off;
    double2 *out = apart + off;
    // X_even = G_N + G_S (l + m even), X_odd = G_N - G_S; the equator ring counts once.
    double2 X[2][P];
#pragma unroll
    for (int k = 0; k < P; k++) {
        const int p = g * kW * P + k * kW + (int)threadIdx.x;
        const bool valid = p < npair;
        const int rN = p, rS = nring - 1 - p;
        const double2 *G = phase + m;  // [ring][m]
        const double2 gN = valid ? G[(long)rN * nm] : make_double2(0.0, 0.0);
        const double2 gS = (valid && rS != rN) ? G[(long)rS * nm] : make_double2(0.0, 0.0);
        X[0][k] = make_double2(gN.x + gS.x, gN.y + gS.y);
        X[1][k] = make_double2(gN.x - gS.x, gN.y - gS.y);
    }
    // values of l before the group's first block receive no contribution
    for (int r = threadIdx.x; r < min(st.klo * kLegBlock, nl); r += kW) out[r] = make_double2(0.0, 0.0);
    for (int blk = st.klo; blk < nblk; blk++) {
        const int r0 = blk * kLegBlock;
        st.enter(blk);
        double acc[kAnaV];
        auto row = [&](int c, double A) __attribute__((always_inline)) {
            double cur[P];
            st.step(A, cur);
            double x = 0.0, y = 0.0;
#pragma unroll
            for (int k = 0; k < P; k++) {
                const double2 q = X[c & 1][k];
                x = k ? fma(cur[k], q.x, x) : cur[k] * q.x;
                y = k ? fma(cur[k], q.y, y) : cur[k] * q.y;
            }
            acc[2 * c] = x;
            acc[2 * c + 1] = y;
        };
        if (r0 + kLegBlock <= nl) {
            double A[kLegBlock];
#pragma unroll
            for (int c = 0; c < kLegBlock; c++) A[c] = Am[r0 + c];
#pragma unroll
            for (int c = 0; c < kLegBlock; c++) row(c, A[c]);
        } else {
#pragma unroll
            for (int c = 0; c < kLegBlock; c++) {
                acc[2 * c] = acc[2 * c + 1] = 0.0;
                if (r0 + c < nl) row(c, Am[r0 + c]);
            }
        }
        const double s = ana_reduce(acc, red);
        // lane 2 v holds value v = 2 c + (0 re, 1 im): the block's coefficients in order
        const int v = threadIdx.x >> 1;
        if ((threadIdx.x & 1) == 0 && r0 + (v >> 1) < nl) reinterpret_cast<double *>(out + r0)[v] = s;
    }
}

template <int P, int ROWS>
__global__ void __launch_bounds__(kW)
k_leg_analysis(const double2 *__restrict__ phase, int nring, int nm,
               const double *__restrict__ Atab, const long *__restrict__ mofs,
               const int *__restrict__ kstart, const double2 *__restrict__ entry,
               const double *__restrict__ zp, double2 *__restrict__ apart, long nalm, int lmax,
               int npair, int ngrp) {
    __shared__ __align__(16) double red[kAnaLds];
    const int nmi = ROWS == 2 ? (lmax + 2) / 2 : nm;
    const LegItem it = leg_item(ngrp, nmi);
    if (it.mi >= nmi) return;
    const int b = blockIdx.y;
    const int npass = (ROWS == 2 && lmax - it.mi > it.mi) ? 2 : 1;
    for (int pass = 0; pass < npass; pass++)
        analysis_one_m<P>(pass == 0 ? it.mi : lmax - it.mi, it.g, phase + (long)b * nm * nring, nring,
                          nm, Atab, mofs, kstart, entry, zp,
                          apart + ((long)it.g * gridDim.y + b) * nalm, lmax, npair, red);
}

// ---------------------------------------------------------------------------------------
// Variant tables: index = tuning choice stored in the plan.
// ---------------------------------------------------------------------------------------
using SynthFn = void (*)(const double2 *, long, const double *, const long *, const int *,
                         const double2 *, const double *, double2 *, int, int, int, int, int);
using AnaFn = void (*)(const double2 *, int, int, const double *, const long *, const int *,
                       const double2 *, const double *, double2 *, long, int, int, int);

struct LegVariant {
    int pairs, rows;  // ring pairs per lane, values of m per wave
};
static const SynthFn kSynth[] = {
    k_leg_synth<1, 8, 2>, k_leg_synth<2, 8, 2>, k_leg_synth<4, 8, 2>,
    k_leg_synth<1, 8, 1>, k_leg_synth<2, 8, 1>, k_leg_synth<4, 8, 1>,
    k_leg_synth<1, 4, 1>, k_leg_synth<2, 4, 1>, k_leg_synth<4, 4, 1>,
};
static const LegVariant kSynthVar[] = {{1, 2}, {2, 2}, {4, 2}, {1, 1}, {2, 1}, {4, 1}, {1, 1}, {2, 1}, {4, 1}};
static const AnaFn kAna[] = {
    k_leg_analysis<1, 2>, k_leg_analysis<2, 2>, k_leg_analysis<4, 2>,
    k_leg_analysis<1, 1>, k_leg_analysis<2, 1>, k_leg_analysis<4, 1>,
};
static const LegVariant kAnaVar[] = {{1, 2}, {2, 2}, {4, 2}, {1, 1}, {2, 1}, {4, 1}};

int leg_synth_variants() { return (int)(sizeof(kSynth) / sizeof(kSynth[0])); }
int leg_analysis_variants() { return (int)(sizeof(kAna) / sizeof(kAna[0])); }
int leg_synth_pairs_per_lane(int v) { return kSynthVar[v].pairs; }
int leg_analysis_pairs_per_lane(int v) { return kAnaVar[v].pairs; }

static int groups(int npair, int P) { return (npair + 64 * P - 1) / (64 * P); }

int launch_leg_synth(const Plan &p, const double2 *alm_scaled, double2 *phase, int nb) {
    const LegVariant v = kSynthVar[p.synth_variant];
    const int ngrp = groups(p.npair, v.pairs);
    hipLaunchKernelGGL(kSynth[p.synth_variant], leg_grid(ngrp, v.rows == 2 ? (p.lmax + 2) / 2 : p.nm, nb),
                       dim3(kW), 0, p.stream, alm_scaled, p.nalm, p.d_A, p.d_mofs, p.d_kstart,
                       p.d_entry, p.d_z, phase, p.lmax, p.npair, p.nring, p.nm, ngrp);
    MFWF_HIP(hipGetLastError());
    return MFWF_OK;
}

int launch_leg_analysis(const Plan &p, const double2 *phase, double2 *apart, int nb) {
    const LegVariant v = kAnaVar[p.ana_variant];
    const int ngrp = groups(p.npair, v.pairs);
    hipLaunchKernelGGL(kAna[p.ana_variant], leg_grid(ngrp, v.rows == 2 ? (p.lmax + 2) / 2 : p.nm, nb),
                       dim3(kW), 0, p.stream, phase, p.nring, p.nm, p.d_A, p.d_mofs, p.d_kstart,
                       p.d_entry, p.d_z, apart, p.nalm, p.lmax, p.npair, ngrp);
    MFWF_HIP(hipGetLastError());
    return MFWF_OK;
}

}  // namespace mfwf
