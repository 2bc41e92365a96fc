// Batched FP32 path: many right-hand sides share one plan and the Legendre steps become
// dense contractions on the matrix cores (MFMA), the GPU form of the transforms that
// Sect. 3 names as the cost driver.
//
// For one m, with columns c = (map, re/im) of all maps in the batch:
//   synthesis  E[p][c] = sum_{l+m even} lambda_lm(z_p) s'[l][c],  O likewise over odd l+m,
//              F_N = E + O, F_S = E - O                      ([pairs x L] x [L x cols])
//   analysis   a[l][c] = sum_p lambda_lm(z_p) X_{(l+m) mod 2}[p][c],
//              X_0 = G_N + G_S, X_1 = G_N - G_S              ([L x pairs] x [pairs x cols])
// lambda_lm is tabulated once per plan in FP32 (computed from the FP64 recurrence from each
// pair's entry state, zero below its first block), as rows [m][pair][l - m] padded to 128
// values of l and 128 pairs.  The FP32 products run as sums of bf16 piece products on the
// matrix cores, accumulated in FP32; the
// ring-Fourier array ([ring][m][cols]) and the coefficients ([alm][cols]) are FP32 with the
// maps innermost, so tiles of columns are contiguous.  Maps, the pixel update and every
// diagnostic stay FP64.  The ring FFTs are the FP64 transforms of the per-map path with
// FP32 per-map output rows, regrouped into the column layout by LDS-tiled transposes.
#include <algorithm>
#include <type_traits>

#include "col_scale.h"
#include "fft_core.h"
#include "leg_core.h"

namespace mfwf {

typedef float floatx16 __attribute__((ext_vector_type(16)));
// Native 4-vectors for the prefetch registers: copies of the HIP float4 struct into LDS are
// aggregate copies that keep the source array in scratch memory.
typedef float floatx4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------------------
// lambda table: one lane per ring pair, one workgroup per (pair tile of 64, m).
// ---------------------------------------------------------------------------------------
__global__ void __launch_bounds__(64)
k_lam_table(const double *__restrict__ Atab, const double *__restrict__ ctab,
            const long *__restrict__ mofs, const int *__restrict__ kstart,
            const double2 *__restrict__ entry, const double *__restrict__ zp,
            const long *__restrict__ loff, const int *__restrict__ Lp, float *__restrict__ lam,
            int lmax, int npair) {
    const int p = blockIdx.x * 64 + threadIdx.x, m = blockIdx.y;
    const int L = Lp[m];
    float *row = lam + loff[m] + (long)p * L;
    const long off = mofs[m] - m;
    if (p >= npair) {
        for (int r = 0; r < L; r++) row[r] = 0.f;
        return;
    }
    const int r0 = kLegBlock * kstart[(long)m * npair + p];  // first row of the pair's first block
    const double2 st = entry[(long)m * npair + p];
    const double z = zp[p];
    double u1 = st.x, u2 = st.y;
    for (int r = 0; r < L; r++) {
        const int l = m + r;
        float v = 0.f;
        if (l <= lmax && r >= r0) {
            const double mu = fma(Atab[off + l] * z, u1, -u2);
            u2 = u1;
            u1 = mu;
            v = (float)(ctab[off + l] * mu);  // lambda = c mu
        }
        row[r] = v;
    }
}

// ---------------------------------------------------------------------------------------
// lambda rows generated inside the GEMMs (temperature batched form): instead of reading
// the FP32 table the GEMMs run the FP64 recurrence of k_lam_table themselves, 16 rows at a
// time, from its state at the start of every 16-row segment of a row, tabulated once per
// plan (16 bytes per 16 table entries: a quarter of the table's size, and the only
// per-(m, pair, l) data the GEMMs read).  The arithmetic and its order are k_lam_table's,
// so the generated values equal the table's bit for bit.
// ---------------------------------------------------------------------------------------
// lck[(segoff[m] + s) Rp + p] = (mu_{l-1}, mu_{l-2}) entering row l = m + 16 s of pair p,
// zero before the pair's first block (and for the padding pairs): the zero state stays zero
static_assert(kLegBlock == 16, "the segments are the blocks that pairs start at");
__global__ void __launch_bounds__(64)
k_lam_ckpt(const double *__restrict__ Atab, const long *__restrict__ mofs,
           const int *__restrict__ kstart, const double2 *__restrict__ entry,
           const double *__restrict__ zp, const int *__restrict__ Lp,
           const long *__restrict__ segoff, double2 *__restrict__ lck, int lmax, int npair,
           int Rp) {
    const int p = blockIdx.x * 64 + threadIdx.x, m = blockIdx.y;
    const int L = Lp[m];
    double2 *out = lck + segoff[m] * Rp + p;
    if (p >= npair) {
        for (int r = 0; r < L; r += 16) out[(long)(r / 16) * Rp] = make_double2(0.0, 0.0);
        return;
    }
    const long off = mofs[m] - m;
    const int r0 = kLegBlock * kstart[(long)m * npair + p];
    const double2 st = entry[(long)m * npair + p];
    const double z = zp[p];
    double u1 = 0.0, u2 = 0.0;
    for (int r = 0; r < L; r++) {
        if (r == r0) {
            u1 = st.x;
            u2 = st.y;
        }
        if ((r & 15) == 0) out[(long)(r / 16) * Rp] = make_double2(u1, u2);
        const int l = m + r;
        if (l <= lmax && r >= r0) {
            const double mu = fma(Atab[off + l] * z, u1, -u2);
            u2 = u1;
            u1 = mu;
        }
    }
}

// Rows l0 .. l0 + 15 of one pair from the segment state st = (u1, u2): the steps of
// k_lam_table; A(r), c(r) give the coefficients A_lm, c_lm of row l0 + r (c = 0 past lmax);
// sink(q, v4) receives rows 4 q .. 4 q + 3 as they are ready.
template <typename FA, typename FC, typename FS>
__device__ __forceinline__ void lam_rows16(double2 st, double z, FA A, FC c, FS sink) {
    double u1 = st.x, u2 = st.y;
#pragma unroll
    for (int q = 0; q < 4; q++) {
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int r = 4 * q + i;
            const double mu = fma(A(r) * z, u1, -u2);
            u2 = u1;
            u1 = mu;
            v[i] = (float)(c(r) * mu);
            // the rounded value, as the table holds it: without this the compiler rounds the
            // product straight to a narrower type where the value is split
            asm("" : "+v"(v[i]));
        }
        sink(q, v);
    }
}

// what a GEMM needs to generate its lambda rows
struct LamGen {
    const double2 *lck;    // segment states (k_lam_ckpt)
    const long *segoff;    // [nm] first segment of each m
    const double *z;       // [npair]
    const double *A, *c;   // [nalm]
};

// The column scales (col_scale.h) of the maps of a solve, or of the coefficients a transform reads:
// grid (map, group of components, part), 5 us a call.  Two groups: n0 and n1 values per map (T; E
// and B), the second's scale to [Bp + b]; both: one group, to both.  cl: the values are C^-1/2 x
// (mode 2 of k_alm_to_cols).
__global__ void __launch_bounds__(256)
k_unit_scale(ColScale *__restrict__ scale, ColScaleSearch *__restrict__ search, int n) {
    for (int i = threadIdx.x; i < n; i += 256) {
        scale[i] = kUnitScale;
        search[i] = ColScaleSearch{0, 0};
    }
}

__global__ void __launch_bounds__(256)
k_col_scale(const double *__restrict__ x, long stride, long n0, long n1, double factor,
            const double *__restrict__ cl, const int *__restrict__ lofi, int both, int Bp,
            ColScale *scale, ColScaleSearch *search) {
    __shared__ int flag;
    const int b = blockIdx.x, g = blockIdx.y;
    const double *v = x + b * stride + (g ? n0 : 0);
    find_col_scale<256>(g ? n1 : n0, blockIdx.z, gridDim.z, &flag, search + g * Bp + b, scale + g * Bp + b,
                        both ? scale + Bp + b : nullptr, [&](long i) {
        double f = factor;
        if (cl) {
            const double C = cl[lofi[i >> 1]];
            f = C > 0.0 ? 1.0 / sqrt(C) : 0.0;
        }
        return f * v[i];
    });
}

// ---------------------------------------------------------------------------------------
// Layout changes between the per-map ring-Fourier rows of the ring transforms,
// [map][ring][m] (FP32 complex), and the contraction layout [m][ring][C2] with columns 2b
// (re) and 2b + 1 (im) of map b.  One workgroup moves a tile of 64 values of m x 64 maps
// of one ring through LDS, so that both sides read and write 512-byte rows.  Each thread
// issues all of its 16 loads before it stores any of them (clamped in-range addresses, values
// selected), so that a workgroup has its whole tile in flight at once.
// ---------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
k_rows_to_cols(const float2 *__restrict__ phf, float *__restrict__ ph32, int nring, int nm,
               int rs, int nb, int Bp, int C2, const ColScale *__restrict__ scale) {
    __shared__ float2 tile[64][64 + 1];  // [map][m]
    const int ring = blockIdx.x, m0 = 64 * blockIdx.y, b0 = 64 * blockIdx.z;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // maps b0 + w + 4 u
    float sc[16];
#pragma unroll
    for (int u = 0; u < 16; u++) sc[u] = scale[min(b0 + w + 4 * u, nb - 1)].s32;
    float2 v[16];
#pragma unroll
    for (int u = 0; u < 16; u++) {
        const int e = threadIdx.x + 256 * u, bb = e >> 6, mm = e & 63, b = b0 + bb, m = m0 + mm;
        const float2 x = phf[((long)min(b, nb - 1) * nring + ring) * rs + min(m, nm - 1)];
        v[u] = (b < nb && m < nm) ? x : make_float2(0.f, 0.f);
    }
#pragma unroll
    for (int u = 0; u < 16; u++) {
        const int e = threadIdx.x + 256 * u;
        tile[e >> 6][e & 63] = make_float2(sc[u] * v[u].x, sc[u] * v[u].y);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 16; u++) {
        const int e = threadIdx.x + 256 * u, mm = e >> 6, bb = e & 63, b = b0 + bb, m = m0 + mm;
        if (b < Bp && m < nm)
            *reinterpret_cast<float2 *>(ph32 + ((long)m * nring + ring) * C2 + 2 * b) = tile[bb][mm];
    }
}

// map b's two columns (2b, 2b + 1) of every (m, ring) row of the columns [m][ring][C2] set
// to zero: a map whose chained iterations start from s = 0
__global__ void __launch_bounds__(256)
k_zero_map_cols(float *__restrict__ ph32, long nrows, int C2, int b) {
    for (long i = blockIdx.x * 256L + threadIdx.x; i < nrows; i += (long)gridDim.x * 256)
        *reinterpret_cast<float2 *>(ph32 + i * C2 + 2 * b) = make_float2(0.f, 0.f);
}

__global__ void __launch_bounds__(256)
k_cols_to_rows(const float *__restrict__ ph32, float2 *__restrict__ phf, int nring, int nm,
               int rs, int nb, int C2, const ColScale *__restrict__ scale) {
    __shared__ float2 tile[64][64 + 1];  // [m][map]
    const int ring = blockIdx.x, m0 = 64 * blockIdx.y, b0 = 64 * blockIdx.z;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // maps b0 + w + 4 u
    float sc[16];
#pragma unroll
    for (int u = 0; u < 16; u++) sc[u] = scale[min(b0 + w + 4 * u, nb - 1)].inv32;
    float2 v[16];
#pragma unroll
    for (int u = 0; u < 16; u++) {
        const int e = threadIdx.x + 256 * u, mm = e >> 6, bb = e & 63, b = b0 + bb, m = m0 + mm;
        const float2 x = *reinterpret_cast<const float2 *>(
            ph32 + ((long)min(m, nm - 1) * nring + ring) * C2 + 2 * min(b, nb - 1));
        v[u] = (b < nb && m < nm) ? x : make_float2(0.f, 0.f);
    }
#pragma unroll
    for (int u = 0; u < 16; u++) {
        const int e = threadIdx.x + 256 * u;
        tile[e >> 6][e & 63] = v[u];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 16; u++) {
        const int e = threadIdx.x + 256 * u, bb = e >> 6, mm = e & 63, b = b0 + bb, m = m0 + mm;
        const float2 x = tile[mm][bb];
        if (b < nb && m < nm)
            phf[((long)b * nring + ring) * rs + m] = make_float2(sc[u] * x.x, sc[u] * x.y);
    }
}

// ---------------------------------------------------------------------------------------
// MFMA GEMMs.  Both contractions run per parity q of l + m: C_q[128][CT] += A_q[128][k] B_q[k][CT]
// with A = lambda (analysis: rows = values of l of parity q, k = ring pairs; synthesis: rows
// = ring pairs, k = values of l of parity q) and B the FP32 columns.
//
// FP32 products on the bf16 matrix cores: every FP32 operand is the sum of three bf16 pieces, each
// the nearest to what the ones before leave (exact above 2^-110, where the column scales keep
// the values that count, and up to the largest finite bf16).  Of the nine piece products the
// six large ones (hi hi, hi mid, mid hi, mid mid, hi lo, lo hi) are accumulated in FP32; the other
// three are at most 2^-24 of the product, the rounding of an FP32 product, and 2^-27.5 in the rms
// (mid is at most 2^-8 of the value, lo 2^-17).  On this card random
// data runs v_mfma_f32_32x32x16_bf16 at 1.67 PFLOP/s, so six of them take the time of 278
// TFLOP/s, where v_mfma_f32_32x32x2_f32 reaches 117-142; and one rounding per 16 values of k
// instead of one per 2 makes the sums more exact, not less.  The sums of 16 values of k start
// from zero and are then added to the running sum (one long chain of FP32 additions over all
// rings would round several times more).
//
// Measured against the FP32 matrix instructions (us, analysis / synthesis): nside 512, 64 maps
// 1304 / 1163 -> 985 / 1123; nside 256, 64 maps 230 / 203 -> 191 / 201; nside 128, 4 maps
// 30 / 19 -> 20 / 18; nside 512, T, Q, U, 32 maps 3324 / 3112 -> 2514 / 2959; transforms with
// generated lambda, nside 2048, lmax 4096, 4 maps 49500 / 44500 -> 37100 / 30000.  What is left at
// nside 512: the table is 2.1 GB (0.43 ms at a copy's rate), the six products 0.5 ms, and the
// splits, which share the issue slots with them, about as much again.
//
// Workgroup i of a launch is dispatched to XCD i mod 8.  Each XCD takes its tiles from its
// own list, so that all tiles of one m, which read the same ring-Fourier (analysis) or
// coefficient (synthesis) block, run on one XCD and share its L2 instead of fetching the
// block from HBM once per XCD; the lists are balanced by the number of active K chunks.
//
// Pipeline: stages of 16 values of k per parity through two LDS buffers, one barrier per
// stage; during a stage's products the next stage is split into its pieces and written to
// the other buffer, and the loads of the stage after that are in flight.  Consecutive lanes
// load consecutive addresses (with two rows interleaved over the lanes the vector L1 took
// four times as many accesses and was the kernels' limit).  The pieces lie in LDS as
// [buffer][parity][piece][k / 4][row][4 k], rows padded, so that the splits' writes and the
// operands' reads (two 8-byte planes each) meet no bank twice.  v_mfma_f32_32x32x16_bf16 operands: A[i][k] in lane
// i + 32 (k / 8), element k % 8, B[k][j] likewise in lane j + 32 (k / 8); accumulator register r
// of lane L holds D[8 (r/4) + 4 (L/32) + r%4][L%32].
// ---------------------------------------------------------------------------------------
// Tile of workgroup bid: XCD x = bid mod 8 works through its own list tab[x][*] of tiles
// (balanced by work on the host, tiles of one m adjacent); columns groups innermost.
struct XcdTile {
    int item, cg;
};
__device__ __forceinline__ XcdTile xcd_tile(const int *__restrict__ tab, int per_xcd, int ncg) {
    const int x = blockIdx.x & 7, s = blockIdx.x >> 3;
    const int k = s / ncg;
    XcdTile r;
    r.cg = s - k * ncg;
    r.item = (k < per_xcd) ? tab[x * per_xcd + k] : -1;
    return r;
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// (hi, mid, lo) bf16 pieces of four floats, four per 8 bytes
struct Split4 {
    uint2 p[3];
};
__device__ __forceinline__ unsigned pack_bf16(float x, float y) {
    const bf16x2 v = {(__bf16)x, (__bf16)y};  // one v_cvt_pk_bf16_f32, round to nearest even
    return __builtin_bit_cast(unsigned, v);
}
__device__ __forceinline__ Split4 split4(float v0, float v1, float v2, float v3) {
    Split4 s;
#pragma unroll
    for (int q = 0; q < 3; q++) {
        const unsigned a = pack_bf16(v0, v1), b = pack_bf16(v2, v3);
        s.p[q] = make_uint2(a, b);
        if (q < 2) {  // the remainders, exact
            v0 -= __uint_as_float(a << 16);
            v1 -= __uint_as_float(a & 0xffff0000u);
            v2 -= __uint_as_float(b << 16);
            v3 -= __uint_as_float(b & 0xffff0000u);
        }
    }
    return s;
}

// the same of two floats, each piece in the halves of one register
__device__ __forceinline__ void split2(float v0, float v1, unsigned (&p)[3]) {
#pragma unroll
    for (int q = 0; q < 3; q++) {
        p[q] = pack_bf16(v0, v1);
        if (q < 2) {
            v0 -= __uint_as_float(p[q] << 16);
            v1 -= __uint_as_float(p[q] & 0xffff0000u);
        }
    }
}

static constexpr int kRows = 128;       // rows per parity of a tile
static constexpr int kAnaL = 2 * kRows; // values of l per analysis tile
// Columns of a tile: 128 (eight waves of 64 rows x 64 columns), 64 (four such waves) or 32
// (eight waves of 32 rows x 32 columns).  A wider tile splits and stages lambda fewer times; a
// narrower one leaves more workgroups, and the eight small waves hide each other's latency
// where a CU holds one or two workgroups (nside 128, 4 maps: analysis 26 -> 19 us against four
// waves of 64 x 32; the 64-column tile cut the same way needs more than 128 registers, loses
// its second workgroup per CU and goes from 202 to 290 us at nside 256, 64 maps).  Every output
// column sees the same operations with any tile.
template <int CT>
struct Tile {
    static constexpr int NTH = CT == 64 ? 256 : 512;   // threads
    static constexpr int NCT = CT == 32 ? 1 : 2;       // 32-column tiles per wave
    static constexpr int NRT = CT == 32 ? 1 : 2;       // 32-row tiles per wave
    static constexpr int NA = 4 * kRows / NTH;         // staging tasks per thread, A and B
    static constexpr bool B1 = CT == 32;               // a staging task of B: one k of both parities, else four
    static constexpr int NB = B1 ? NTH : 4 * CT;       // staging tasks of B
    static constexpr int NBV = B1 ? 2 : 8;             // values of such a task
    static constexpr int A_EL = 2 * 3 * 4 * (kRows + 8) * 4, B_EL = 2 * 3 * 4 * (CT + 8) * 4;  // bf16 per buffer
};
// bf16 offset of (parity, piece, k4 = k / 4, row) in a buffer of `rows` rows
__device__ __forceinline__ int piece_at(int par, int pc, int k4, int row, int rows) {
    return (((par * 3 + pc) * 4 + k4) * (rows + 8) + row) * 4;
}
// write a task's four values of k to a buffer
__device__ __forceinline__ void put_split(unsigned short *buf, int par, int k4, int row, int rows,
                                          const Split4 &s) {
#pragma unroll
    for (int q = 0; q < 3; q++)
        *reinterpret_cast<uint2 *>(buf + piece_at(par, q, k4, row, rows)) = s.p[q];
}
// write one value of k of both parities (v0 to parity par, v1 to the other)
__device__ __forceinline__ void put_split1(unsigned short *buf, int par, int k, int row, int rows,
                                           float v0, float v1) {
    unsigned x[3];
    split2(v0, v1, x);
#pragma unroll
    for (int q = 0; q < 3; q++) {
        buf[piece_at(par, q, k >> 2, row, rows) + (k & 3)] = (unsigned short)x[q];
        buf[piece_at(par ^ 1, q, k >> 2, row, rows) + (k & 3)] = (unsigned short)(x[q] >> 16);
    }
}
// a lane's operand: k = 8 kg .. 8 kg + 7 of one row
__device__ __forceinline__ bf16x8 get_operand(const unsigned short *buf, int par, int pc, int kg, int row, int rows) {
    const uint2 a = *reinterpret_cast<const uint2 *>(buf + piece_at(par, pc, 2 * kg, row, rows));
    const uint2 b = *reinterpret_cast<const uint2 *>(buf + piece_at(par, pc, 2 * kg + 1, row, rows));
    return __builtin_bit_cast(bf16x8, make_uint4(a.x, a.y, b.x, b.y));
}

// A wave's products of one stage, its 64 rows x 32 NCT columns of parity par, summed from zero,
// small piece products first
template <int CT>
__device__ __forceinline__ void stage_products(const unsigned short *A, const unsigned short *B, int par,
                                               int row0, int col0, floatx16 (&part)[Tile<CT>::NRT][Tile<CT>::NCT]) {
    constexpr int NCT = Tile<CT>::NCT, NRT = Tile<CT>::NRT;
    const int lane = threadIdx.x & 63, i = lane & 31, kg = lane >> 5;
    bf16x8 a[NRT][3];
#pragma unroll
    for (int q = 0; q < 3; q++)
#pragma unroll
        for (int t = 0; t < NRT; t++) a[t][q] = get_operand(A, par, q, kg, row0 + 32 * t + i, kRows);
    constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
    for (int c = 0; c < NCT; c++) {
        bf16x8 b[3];
#pragma unroll
        for (int q = 0; q < 3; q++) b[q] = get_operand(B, par, q, kg, col0 + 32 * c + i, CT);
#pragma unroll
        for (int p = 0; p < 6; p++)
#pragma unroll
            for (int t = 0; t < NRT; t++) {
                const floatx16 z = {};
                part[t][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[t][pa[p]], b[pb[p]], p == 0 ? z : part[t][c], 0, 0, 0);
            }
    }
}
// the stage's sums added to (NEG: taken from) the running sums, once the stage's splitting
// has covered the products' latency
template <bool NEG, int NRT, int NCT>
__device__ __forceinline__ void stage_add(float (&acc)[NRT][NCT][16], const floatx16 (&part)[NRT][NCT]) {
#pragma unroll
    for (int t = 0; t < NRT; t++)
#pragma unroll
        for (int c = 0; c < NCT; c++)
#pragma unroll
            for (int r = 0; r < 16; r++) {
                acc[t][c][r] += NEG ? -part[t][c][r] : part[t][c][r];
                // the addition stays here: sunk to the next use, it would hold two column
                // tiles' partial sums in registers through the next stage, and spill
                if constexpr (NCT > 1) asm volatile("" : "+v"(acc[t][c][r]));
            }
}
// 4-byte load at a uniform base plus a 32-bit byte offset per lane
__device__ __forceinline__ float ld_off(const float *base, unsigned byte) {
    return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(base) + byte);
}

// The matrix cores bring the terms of one v_mfma_f32_32x32x16_bf16 to the largest one's
// exponent by rounding towards minus infinity one bit below its last (measured: a small C
// under a product loses 0.25 ulp of the sum on average, whatever the signs; the FP32 form
// rounds to nearest).  Left alone, every sum comes out low: the mean error of an analysis is -0.24 of
// its rms at nside 64 and -0.33 at nside 512, the same in every iteration, and it adds up in the
// modes that converge slowly (nside 512, two maps, 300 iterations: 2.2e-6).  So its sign
// alternates: the stages of both contractions alternate between sums and negated sums, and in
// the synthesis, whose terms fall off with l, so do the rings, whose alternating error has no
// large-scale part.  The mean is then 0.003-0.03 of the rms and the error after 300 iterations 1.6e-6
// (1.7e-6 with the FP32 instructions; after 100 6.6e-7-7.6e-7 against 7.3e-7).
// Rounding the leading piece at random, so that the pieces differ from one iteration to the
// next, changes neither the mean nor the errors, and lets the products left out reach 2^-23.6.
__device__ __forceinline__ float row_sign(int row) { return row & 1 ? -1.f : 1.f; }

// analysis: tile = (m, 256 values of l, CT columns); K loop over active chunks of 32 ring
// pairs (two stages).  Wave w: parity w & 1, rows 64 rh .. +63 of that parity, columns 64 ch ..
// Output: raw sums a (if a_out) and/or the Wiener-filtered coefficients
// s = scale_s C_l / (C_l + lto) a (if s_out), rows [alm][C2].  Even l + m rows contract
// G_N + G_S and odd rows G_N - G_S (a table with lambda's mirror symmetry); flip swaps the
// two, for a table that is odd where lambda is even (the spin-2 F-).
// GEN: lambda from the segment states instead of the table, through an FP32 slab in LDS.
template <int CT, bool GEN>
__global__ void __launch_bounds__(Tile<CT>::NTH, 2)
k_gemm_analysis(const float *__restrict__ lam, LamGen gen, const long *__restrict__ loff,
                const int *__restrict__ Lp, const int *__restrict__ minls32,
                const int2 *__restrict__ items, const int *__restrict__ tab, int per_xcd,
                const float *__restrict__ ph32, const long *__restrict__ mofs,
                const double *__restrict__ cl, float *__restrict__ a_out,
                float *__restrict__ s_out, double scale_s, double lto, int lmax, int npair,
                int Rp, int nring, int nm, int C2, int ncols, int ncg,
                const double *__restrict__ tau_b, double lto_per_tau, int flip,
                const float *__restrict__ zrow) {
    using T = Tile<CT>;
    constexpr int NTH = T::NTH, NCT = T::NCT, NRT = T::NRT, NA = T::NA, RW = 32 * NRT;
    __shared__ __align__(16) unsigned short sA[2][T::A_EL], sB[2][T::B_EL];
    __shared__ double sF[kAnaL];  // filter factors of the tile's rows
    __shared__ float sL[GEN ? 2 : 1][GEN ? 16 : 1][GEN ? kAnaL + 4 : 1];  // generated lambda [pair][l]
    __shared__ double sAc[2][GEN ? kAnaL : 1];                            // A_lm, c_lm of the rows
    const XcdTile xt = xcd_tile(tab, per_xcd, ncg);
    if (xt.item < 0) return;
    const int2 it = items[xt.item];
    const int m = it.x, t0 = kAnaL * it.y, cg = xt.cg;  // rows l = m + t0 + ..
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int par = w & 1, rh = CT == 128 ? w >> 2 : w >> 1, ch = CT == 128 ? (w >> 1) & 1 : 0;
    const int L = Lp[m];
    const int nchunk = (npair + 31) / 32;
    const int *ms = minls32 + m * (Rp / 32);
    const int lhi = min(m + t0 + kAnaL - 1, lmax);          // last l of the tile
    const int lhi_w = min(m + t0 + 2 * RW * (rh + 1) - 1, lmax);  // last l of this wave's rows
    // a wave whose rows all lie past lmax, or whose columns lie past the batch, does no products
    const bool wave_on = CT * cg + 64 * ch < ncols && m + t0 + 2 * RW * rh <= lmax;
    // The first active chunk of the tile and of this wave's rows (ring pairs start at smaller l
    // towards the equator), 64 chunks looked at together: one by one, every skipped chunk
    // costs a memory latency before the first load
    int pc = nchunk, pw = nchunk;
    for (int q = 0; q < nchunk && pw == nchunk; q += 64) {
        const int v = q + lane < nchunk ? ms[q + lane] : lmax + 1;
        const unsigned long long any = __ballot(v <= lhi), own = __ballot(wave_on && v <= lhi_w);
        if (pc == nchunk && any) pc = q + __builtin_ctzll(any);
        if (own) pw = q + __builtin_ctzll(own);
    }
    const long base = mofs[m] - m;
    if (s_out && !tau_b)
        for (int r = threadIdx.x; r < kAnaL; r += NTH) {
            const double C = m + t0 + r <= lmax ? cl[m + t0 + r] : 0.0;
            sF[r] = C > 0.0 ? C / (C + lto) * scale_s : 0.0;
        }
    if constexpr (GEN)
        for (int r = threadIdx.x; r < kAnaL; r += NTH) {
            const int l = min(m + t0 + r, lmax);
            sAc[0][r] = gen.A[base + l];
            sAc[1][r] = m + t0 + r <= lmax ? gen.c[base + l] : 0.0;
        }
    // staging tasks of a stage: A: (l, l + 1; four ring pairs k4), B: (column; four ring pairs)
    // register sets of loads in flight: two stages ahead, one where two would not fit
    constexpr int NS = CT == 64 && !GEN ? 1 : 2;
    constexpr bool COMPACT = CT == 32 && !GEN;
    float ra[GEN ? 1 : NS][NA][8], rb[NS][T::NBV];
    const int bcol = threadIdx.x % CT, bk4 = threadIdx.x / CT;  // B1: bk4 is k itself
    const bool b_on = NTH <= T::NB || (int)threadIdx.x < T::NB;
    // addresses = a uniform base per load + one byte offset per thread.  What is loaded for rows
    // past the table, columns past the batch and padding pairs is valid data that never reaches
    // an output: those rows and columns are not stored, padding pairs have lambda = 0.
    const int col = min(CT * cg + bcol, ncols - 1);
    const unsigned noff = 4 * (4 * bk4 * C2 + col), soff = 4 * (4 * (3 - bk4) * C2 + col);
    unsigned aoff[NA];
#pragma unroll
    for (int u = 0; u < NA; u++) {
        const int e = threadIdx.x + NTH * u, row = e & (kRows - 1), k4 = e / kRows;
        aoff[u] = 4 * (4 * k4 * L + (t0 + 2 * row < L ? 2 * row : 0));
    }
    const float *lrow = GEN ? nullptr : lam + loff[m] + t0;
    const float *gN = ph32 + (long)m * nring * C2, *gS = gN + (long)(nring - 1) * C2;
    // GEN: task (pair, 16-row segment): 16 x 16 tasks, lanes over the pairs (the rows'
    // coefficients are then broadcast reads)
    const int gp = threadIdx.x & 15, gs = (threadIdx.x >> 4) & 15;
    const bool gen_on = GEN && threadIdx.x < 256;
    double2 gst = make_double2(0.0, 0.0);
    double gz = 0.0;
    auto load = [&](int p0, int set_) __attribute__((always_inline)) {  // pairs p0 .. p0 + 15
        const int set = set_ & (NS - 1);
        if constexpr (GEN) {
            if (gen_on) {
                // segments past the row's (rows that are not stored) repeat its last one
                const int seg = min(t0 / 16 + gs, L / 16 - 1);
                gst = gen.lck[(gen.segoff[m] + seg) * (long)Rp + p0 + gp];
                gz = gen.z[min(p0 + gp, npair - 1)];
            }
        } else {
#pragma unroll
            for (int u = 0; u < NA; u++) {
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    const char *q = reinterpret_cast<const char *>(lrow + (long)(p0 + j) * L);
                    const float2 v = *reinterpret_cast<const float2 *>(q + aoff[u]);
                    ra[set][u][2 * j] = v.x;
                    ra[set][u][2 * j + 1] = v.y;
                }
            }
        }
        if constexpr (T::B1) {
            const int p = min(p0 + bk4, npair - 1);
            rb[set][0] = ld_off(gN, 4 * (p * C2 + col));
            rb[set][1] = ld_off(gN, 4 * ((nring - 1 - p) * C2 + col));
        } else if (b_on) {
            if (p0 + 16 < npair) {
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    rb[set][j] = ld_off(gN + (long)(p0 + j) * C2, noff);
                    // south rings run backwards: pair p0 + 4 bk4 + j from the base of p0 + 12 + j
                    rb[set][4 + j] = ld_off(gS - (long)(p0 + 12 + j) * C2, soff);
                }
            } else {  // the equator, whose ring counts once, and what may follow it
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    const int p = p0 + 4 * bk4 + j, pq = min(p, npair - 1);
                    rb[set][j] = gN[(long)pq * C2 + col];
                    rb[set][4 + j] = *(p < npair - 1 ? gS + (col - (long)pq * C2) : zrow + col);
                }
            }
        }
    };
    auto gen_rows = [&](int buf) __attribute__((always_inline)) {
        if constexpr (GEN)
            if (gen_on)
                lam_rows16(gst, gz, [&](int r) { return sAc[0][16 * gs + r]; }, [&](int r) { return sAc[1][16 * gs + r]; },
                           [&](int q, const float (&v)[4]) {
                               *reinterpret_cast<floatx4 *>(&sL[buf][gp][16 * gs + 4 * q]) =
                                   floatx4{v[0], v[1], v[2], v[3]};
                           });
    };
    // split the stage data of register set `set` (GEN: of slab buffer `set`) into LDS buffer `buf`
    // (a chunk's second half is contracted negated)
    auto split = [&](int p0, int set_, int buf) __attribute__((always_inline)) {  // of pairs p0 ..
        const int set = GEN ? set_ : set_ & (NS - 1);
#pragma unroll
        for (int u = 0; u < NA; u++) {
            const int e = threadIdx.x + NTH * u, row = e & (kRows - 1), k4 = e / kRows;
            float v[8];
#pragma unroll
            for (int j = 0; j < 4; j++) {
                if constexpr (GEN) {
                    const float2 x = *reinterpret_cast<const float2 *>(&sL[set][4 * k4 + j][2 * row]);
                    v[2 * j] = x.x;
                    v[2 * j + 1] = x.y;
                } else {
                    v[2 * j] = ra[set][u][2 * j];
                    v[2 * j + 1] = ra[set][u][2 * j + 1];
                }
            }
            put_split(sA[buf], 0, k4, row, kRows, split4(v[0], v[2], v[4], v[6]));
            put_split(sA[buf], 1, k4, row, kRows, split4(v[1], v[3], v[5], v[7]));
        }
        if constexpr (T::B1) {
            float n = rb[set][0], v = p0 + bk4 < npair - 1 ? rb[set][1] : 0.f;  // the equator counts once
            if (buf) n = -n, v = -v;
            put_split1(sB[buf], flip, bk4, bcol, CT, n + v, n - v);
        } else if (b_on) {
            float ps[4], df[4];
#pragma unroll
            for (int j = 0; j < 4; j++) {
                ps[j] = buf ? -rb[set][j] - rb[set][4 + j] : rb[set][j] + rb[set][4 + j];
                df[j] = buf ? rb[set][4 + j] - rb[set][j] : rb[set][j] - rb[set][4 + j];
            }
            put_split(sB[buf], flip, bk4, bcol, CT, split4(ps[0], ps[1], ps[2], ps[3]));
            put_split(sB[buf], flip ^ 1, bk4, bcol, CT, split4(df[0], df[1], df[2], df[3]));
        }
    };
    float acc[NRT][NCT][16];
#pragma unroll
    for (int t = 0; t < NRT; t++)
#pragma unroll
        for (int c = 0; c < NCT; c++)
#pragma unroll
            for (int r = 0; r < 16; r++) acc[t][c][r] = 0.f;
    // The chunks from the first active one on.  stage (chunk, h): pairs 32 chunk + 16 h ..;
    // register set and buffers h.
    pc = __builtin_amdgcn_readfirstlane(pc);
    pw = __builtin_amdgcn_readfirstlane(max(pw, pc));
    const int last = nchunk - 1;
    if constexpr (COMPACT) {
        // Small launches run few rounds, and fetching the instructions weighs on them (27 KB
        // of straight code with separate rounds, 10 KB here; a solve's iteration at nside 16
        // with 4 maps 78 -> 71 us): one copy of the round, whose first split is the prologue's;
        // every wave does the products of all the tile's chunks, and the second stage's sums
        // are taken off after the next split.
        floatx16 part[NRT][NCT] = {};
        if (pc < nchunk) {
            load(32 * pc, 0);
            load(32 * pc + 16, 1);
        }
#pragma unroll 1
        for (; pc < nchunk; pc++) {
            split(32 * pc, 0, 0);
            load(32 * min(pc + 1, last), 0);
            stage_add<true>(acc, part);
            __syncthreads();
            stage_products<CT>(sA[0], sB[0], par, RW * rh, 64 * ch, part);
            split(32 * pc + 16, 1, 1);
            load(32 * min(pc + 1, last) + 16, 1);
            stage_add<false>(acc, part);
            __syncthreads();
            stage_products<CT>(sA[1], sB[1], par, RW * rh, 64 * ch, part);
        }
        stage_add<true>(acc, part);
    } else {
    if (pc < nchunk) {
        if constexpr (GEN) {
            __syncthreads();  // sAc
            load(32 * pc, 0);
            gen_rows(0);
            load(32 * pc + 16, 1);
            gen_rows(1);
            __syncthreads();
            split(32 * pc, 0, 0);
        } else {
            load(32 * pc, 0);
            if (NS == 2) load(32 * pc + 16, 1);
            split(32 * pc, 0, 0);
            if (NS == 2) load(32 * min(pc + 1, last), 0);
            else load(32 * pc + 16, 1);
        }
        __syncthreads();
    }
    // One chunk; on: with products.  Loads are issued in every round (the last ones repeat the
    // last chunk) and on one path, so that the waits for one register set leave the other in
    // flight, and a stage is one stretch of code in which the next stage's splitting fills
    // the time of its products.
    auto round = [&](auto on) __attribute__((always_inline)) {
        // first stage: products of buffer 0; the chunk's second half to buffer 1, and its
        // registers take the next chunk's second half
        auto refill1 = [&]() __attribute__((always_inline)) {
            split(32 * pc + 16, 1, 1);
            if (!GEN) load(32 * min(pc + 1, last) + (NS == 2 ? 16 : 0), 1);
        };
        if (GEN) load(32 * min(pc + 1, last), 0);
        floatx16 part[NRT][NCT];
        if constexpr (on()) stage_products<CT>(sA[0], sB[0], par, RW * rh, 64 * ch, part);
        refill1();
        if constexpr (on()) stage_add<false>(acc, part);
        gen_rows(0);
        __syncthreads();
        // second stage: products of buffer 1; the next chunk's first half to buffer 0
        auto refill0 = [&]() __attribute__((always_inline)) {
            split(32 * min(pc + 1, last), 0, 0);
            if (!GEN) load(NS == 2 ? 32 * min(pc + 2, last) : 32 * min(pc + 1, last) + 16, 0);
        };
        if (GEN) load(32 * min(pc + 1, last) + 16, 1);
        if constexpr (on()) stage_products<CT>(sA[1], sB[1], par, RW * rh, 64 * ch, part);
        refill0();
        if constexpr (on()) stage_add<true>(acc, part);
        gen_rows(1);
        __syncthreads();
        pc++;
    };
    while (pc < pw) round(std::false_type{});
    while (pc < nchunk) round(std::true_type{});
    }
    if (!wave_on) return;
    // for each register, lanes 0..31 and 32..63 hold 32 columns of two rows (rows 4 apart):
    // whole 128-byte lines, at a uniform base plus one offset per lane
    const int rhu = __builtin_amdgcn_readfirstlane(rh), paru = __builtin_amdgcn_readfirstlane(par);
    const int hi4 = 4 * (lane >> 5);
#pragma unroll
    for (int c = 0; c < NCT; c++) {
        const int oc = CT * cg + 64 * ch + 32 * c + (lane & 31);
        if (oc - (lane & 31) >= ncols) continue;
        const double lt = tau_b ? lto_per_tau * tau_b[oc >> 1] : lto;  // per-map tau (serving slots)
        const unsigned lane_off = 2 * hi4 * C2 + oc;
#pragma unroll
        for (int t = 0; t < NRT; t++)
#pragma unroll
            for (int r = 0; r < 16; r++) {
                const int row0 = 2 * (RW * rhu + 32 * t + 8 * (r >> 2) + (r & 3)) + paru;  // of lane 0
                const int row = row0 + 2 * hi4, l = m + t0 + row;
                if (l > lmax) continue;
                const long at = (base + m + t0 + row0) * C2;
                const float v = acc[t][c][r];
                if (a_out) (a_out + at)[lane_off] = v;
                if (s_out) {
                    double f;
                    if (tau_b) {
                        const double C = cl[l];
                        f = C > 0.0 ? C / (C + lt) * scale_s : 0.0;
                    } else {
                        f = sF[row];
                    }
                    (s_out + at)[lane_off] = (float)(f * v);
                }
            }
    }
}

// synthesis: tile = (m, 128 ring pairs, CT columns); K loop over chunks of 64 values of l (32
// of each parity, two stages).  Wave w: parity w & 1, pairs 64 rh .. +63, columns 64 ch ..
// The waves of the two parities swap their sums through LDS: the even one stores the north
// rings E + O, the odd one the south rings E - O (lambda's mirror symmetry), or O - E with
// flip (the spin-2 F-).
// ONCE: the table's loads are streaming loads (launch rule: synthesis_once).
// GEN: lambda is generated from the segment states by four waves, chains of sixteen steps in
// double precision, which bound the kernel: 32 columns take at most 128 registers, so that two
// workgroups of a CU hide each other's chains (nside 2048, lmax 4096, sht_inv, ms with one / two:
// 4 maps 49.9 / 30.1, 16 maps 57.9 / 38.2).  64 columns cut the same way spill.
template <int CT, bool GEN, bool ONCE>
__global__ void __launch_bounds__(Tile<CT>::NTH, CT == 32 ? 4 : 2)
k_gemm_synthesis(const float *__restrict__ lam, LamGen gen, const long *__restrict__ loff,
                 const int *__restrict__ Lp, const int *__restrict__ minls32,
                 const int2 *__restrict__ items, const int *__restrict__ tab, int per_xcd,
                 const float *__restrict__ s32, const long *__restrict__ mofs,
                 float *__restrict__ ph32, int lmax, int npair, int Rp, int nring, int nm,
                 int C2, int ncols, int ncg, int flip, int comb) {
    using T = Tile<CT>;
    constexpr int NTH = T::NTH, NCT = T::NCT, NRT = T::NRT, NA = T::NA, NW = NTH / 64, RW = 32 * NRT;
    __shared__ __align__(16) unsigned short sA[2][T::A_EL], sB[2][T::B_EL];
    const XcdTile xt = xcd_tile(tab, per_xcd, ncg);
    if (xt.item < 0) return;
    const int2 it = items[xt.item];
    const int m = it.x, q0 = kRows * it.y, cg = xt.cg;  // ring pairs q0 ..
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int par = w & 1, rh = CT == 128 ? w >> 2 : w >> 1, ch = CT == 128 ? (w >> 1) & 1 : 0;
    const int L = Lp[m], Lm = lmax - m + 1;
    const int *ms = minls32 + m * (Rp / 32) + q0 / 32;
    const int ls_wave = min(ms[NRT * rh], ms[NRT * rh + NRT - 1]);
    const int ls_tile = min(min(ms[0], ms[1]), min(ms[2], ms[3]));
    const bool wave_on = CT * cg + 64 * ch < ncols;
    const long base = mofs[m];
    // staging tasks of a stage: A: (pair; four values of l), two per thread of 512; B: (column;
    // eight values of l, four of each parity)
    // register sets of loads in flight: two stages ahead, one where two would not fit
    constexpr int NS = CT == 64 && !GEN ? 1 : 2;
    constexpr bool COMPACT = CT == 32 && !GEN;
    floatx4 ra[GEN ? 1 : NS][GEN ? 1 : 2 * NA];
    float rb[NS][T::NBV];
    const int bcol = threadIdx.x % CT, bk4 = threadIdx.x / CT;  // B1: bk4 is k itself
    const bool b_on = NTH <= T::NB || (int)threadIdx.x < T::NB;
    const int col = min(CT * cg + bcol, ncols - 1);  // columns past the batch are not stored
    const unsigned boff = 4 * (8 * bk4 * C2 + col);  // bytes
    const int al = threadIdx.x & 7, arow = threadIdx.x >> 3;  // eight lanes read 32 values of l of a pair
    const unsigned aoff = 4 * (arow * L + 4 * al);
    const float rsgn = row_sign(GEN ? threadIdx.x & (kRows - 1) : arow);  // the same for all of a thread's rows
    const float *lrow = GEN ? nullptr : lam + loff[m] + (long)q0 * L;
    // GEN: task (pair, 16 values of l = k / 8 group of both parities): threads 0..255; the
    // coefficients are the same for the whole wave (scalar loads)
    const int gp = threadIdx.x & (kRows - 1), gk = __builtin_amdgcn_readfirstlane(threadIdx.x >> 7);
    const bool gen_on = GEN && threadIdx.x < 256;
    double2 gst[2] = {};
    const double gz = gen_on ? gen.z[min(q0 + gp, npair - 1)] : 0.0;
    auto load = [&](int r0, int set_) __attribute__((always_inline)) {  // l = m + r0 .. m + r0 + 31
        const int set = set_ & (NS - 1);
        if constexpr (GEN) {
            if (gen_on) gst[set] = gen.lck[(gen.segoff[m] + r0 / 16 + gk) * (long)Rp + q0 + gp];
        } else {
#pragma unroll
            for (int u = 0; u < 2 * NA; u++) {
                const char *x = reinterpret_cast<const char *>(lrow + (long)(u * (NTH / 8)) * L + r0);
                const floatx4 *q = reinterpret_cast<const floatx4 *>(x + aoff);
                if constexpr (ONCE) ra[set][u] = __builtin_nontemporal_load(q);
                else ra[set][u] = *q;
            }
        }
        if constexpr (T::B1) {  // past lmax: valid data, times lambda = 0
#pragma unroll
            for (int j = 0; j < 2; j++)
                rb[set][j] = ld_off(s32 + base * C2, 4 * (min(r0 + 2 * bk4 + j, Lm - 1) * C2 + col));
        } else if (b_on) {
            if (r0 + 32 <= Lm) {
#pragma unroll
                for (int j = 0; j < 8; j++) rb[set][j] = ld_off(s32 + (base + r0 + j) * C2, boff);
            } else {  // past lmax: valid data, times lambda = 0
#pragma unroll
                for (int j = 0; j < 8; j++)
                    rb[set][j] = s32[(base + min(r0 + 8 * bk4 + j, Lm - 1)) * C2 + col];
            }
        }
    };
    auto split = [&](int r0, int set_, int buf) __attribute__((always_inline)) {
        const int set = set_ & (NS - 1);
        if constexpr (GEN) {
            if (gen_on) {
                const int l0 = m + r0 + 16 * gk;
                const long aoff = base - m;
                float v[16];
                lam_rows16(gst[set], gz, [&](int r) { return gen.A[aoff + min(l0 + r, lmax)]; },
                           [&](int r) { return l0 + r <= lmax ? gen.c[aoff + l0 + r] : 0.0; },
                           [&](int q, const float (&x)[4]) {
#pragma unroll
                               for (int i = 0; i < 4; i++) v[4 * q + i] = (buf ? -rsgn : rsgn) * x[i];
                           });
#pragma unroll
                for (int h = 0; h < 2; h++)
#pragma unroll
                    for (int q = 0; q < 2; q++)
                        put_split(sA[buf], q, 2 * gk + h, gp, kRows,
                                  split4(v[8 * h + q], v[8 * h + 2 + q], v[8 * h + 4 + q], v[8 * h + 6 + q]));
            }
        } else {
#pragma unroll
            for (int u = 0; u < 2 * NA; u++) {
                // l = 4 al .. 4 al + 3: k = 2 al, 2 al + 1 of each parity
                const floatx4 v = (buf ? -rsgn : rsgn) * ra[set][u];
                const Split4 x = split4(v[0], v[2], v[1], v[3]);  // .x even pair, .y odd pair
#pragma unroll
                for (int q = 0; q < 3; q++) {
                    unsigned short *o = sA[buf] + piece_at(0, q, al >> 1, arow + u * (NTH / 8), kRows) + 2 * (al & 1);
                    *reinterpret_cast<unsigned *>(o) = x.p[q].x;
                    *reinterpret_cast<unsigned *>(o + piece_at(1, 0, 0, 0, kRows)) = x.p[q].y;
                }
            }
        }
        if constexpr (T::B1) {
            put_split1(sB[buf], 0, bk4, bcol, CT, rb[set][0], rb[set][1]);
        } else if (b_on) {
            const float *v = rb[set];
            put_split(sB[buf], 0, bk4, bcol, CT, split4(v[0], v[2], v[4], v[6]));
            put_split(sB[buf], 1, bk4, bcol, CT, split4(v[1], v[3], v[5], v[7]));
        }
    };
    float acc[NRT][NCT][16];
#pragma unroll
    for (int t = 0; t < NRT; t++)
#pragma unroll
        for (int c = 0; c < NCT; c++)
#pragma unroll
            for (int r = 0; r < 16; r++) acc[t][c][r] = 0.f;
    int rc = max(0, ls_tile - m) / 64;  // first chunk with a nonzero lambda
    const int nrc = (Lm + 63) / 64;
    rc = __builtin_amdgcn_readfirstlane(rc);
    if constexpr (COMPACT) {  // one copy of the round, as in the analysis
        floatx16 part[NRT][NCT] = {};
        if (rc < nrc) {
            load(64 * rc, 0);
            load(64 * rc + 32, 1);
        }
#pragma unroll 1
        for (; rc < nrc; rc++) {
            const int rl = 64 * min(rc + 1, nrc - 1);
            split(64 * rc, 0, 0);
            load(rl, 0);
            stage_add<true>(acc, part);
            __syncthreads();
            stage_products<CT>(sA[0], sB[0], par, RW * rh, 64 * ch, part);
            split(64 * rc + 32, 1, 1);
            load(rl + 32, 1);
            stage_add<false>(acc, part);
            __syncthreads();
            stage_products<CT>(sA[1], sB[1], par, RW * rh, 64 * ch, part);
        }
        stage_add<true>(acc, part);
        __syncthreads();
    } else {
    if (rc < nrc) {
        load(64 * rc, 0);
        if (NS == 2) load(64 * rc + 32, 1);
        split(64 * rc, 0, 0);
        if (NS == 2) load(64 * min(rc + 1, nrc - 1), 0);
        else load(64 * rc + 32, 1);
        __syncthreads();
    }
    auto round = [&](auto on) __attribute__((always_inline)) {  // one chunk, as in the analysis
        const int rl = 64 * min(rc + 1, nrc - 1), rm = 64 * min(rc + 2, nrc - 1);
        auto refill1 = [&]() __attribute__((always_inline)) {
            split(64 * rc + 32, 1, 1);
            if (NS == 2) load(rl + 32, 1);
            else load(rl, 0);
        };
        floatx16 part[NRT][NCT];
        if constexpr (on()) stage_products<CT>(sA[0], sB[0], par, RW * rh, 64 * ch, part);
        refill1();
        if constexpr (on()) stage_add<false>(acc, part);
        __syncthreads();
        auto refill0 = [&]() __attribute__((always_inline)) {
            split(rl, 0, 0);
            if (NS == 2) load(rm, 0);
            else load(rl + 32, 1);
        };
        if constexpr (on()) stage_products<CT>(sA[1], sB[1], par, RW * rh, 64 * ch, part);
        refill0();
        if constexpr (on()) stage_add<true>(acc, part);
        __syncthreads();
        rc++;
    };
    // the wave's first chunk
    const int rw = __builtin_amdgcn_readfirstlane(wave_on ? min(max(0, ls_wave - m) / 64, nrc) : nrc);
    while (rc < rw) round(std::false_type{});
    while (rc < nrc) round(std::true_type{});
    }
    // Swap with the wave of the other parity, 32 pairs x 32 columns at a time, in register
    // order; each register then holds 32 columns of two rings (pairs 4 apart): whole 128-byte
    // lines, at a uniform base plus one offset per lane.
    float *ex = reinterpret_cast<float *>(&sA[0][0]);
    static_assert(sizeof(sA) >= NW * 1024 * sizeof(float), "epilogue exchange");
    const int rhu = __builtin_amdgcn_readfirstlane(rh), paru = __builtin_amdgcn_readfirstlane(par);
    const int hi4 = 4 * (lane >> 5);
    const bool whole = q0 + kRows < npair;  // every pair exists and none is the equator
#pragma unroll
    for (int c = 0; c < NCT; c++) {
#pragma unroll
        for (int t = 0; t < NRT; t++) {
            if (c + t) __syncthreads();
#pragma unroll
            for (int r = 0; r < 16; r++) ex[(w * 16 + r) * 64 + lane] = acc[t][c][r];
            __syncthreads();
            const int oc = CT * cg + 64 * ch + 32 * c + (lane & 31);
            if (oc - (lane & 31) >= ncols) continue;  // uniform per wave, after the barriers of this tile
            const int p0 = q0 + RW * rhu + 32 * t;
            // row of register r: pair p0 + 8 (r / 4) + r % 4 + hi4; south rings run backwards
            float *out0 = ph32 + ((long)m * nring + (paru ? nring - 1 - p0 - 4 : p0)) * C2;
            const unsigned lane_off = (paru ? 4 - hi4 : hi4) * C2 + oc;
            const long step = paru ? -(long)C2 : (long)C2;
            float v[16];
#pragma unroll
            for (int r = 0; r < 16; r++) {
                const float o = ex[((w ^ 1) * 16 + r) * 64 + lane], x = acc[t][c][r];
                // even wave: x = E, o = O; odd wave: x = O, o = E
                v[r] = (paru == 0 ? x + o : (flip ? x - o : o - x)) * row_sign(r);  // the row's parity is r's
            }
            auto at = [&](int r) { return out0 + (8 * (r >> 2) + (r & 3)) * step; };
            auto in = [&](int r) {
                const int p = p0 + 8 * (r >> 2) + (r & 3) + hi4;
                return p < npair - paru;  // the equator once (pair npair - 1 has no south ring)
            };
            if (comb) {
                // spin 2: v = R' = F- x s_EB of one map (E re, E im, B re, B im) and out holds
                // P' = F+ x s_EB: Q = -(P'_E + i R'_B), U = -(P'_B - i R'_E) over P'
                const int k = lane & 3;
                float P[16];
#pragma unroll
                for (int r = 0; r < 16; r++) P[r] = whole || in(r) ? at(r)[lane_off] : 0.f;
#pragma unroll
                for (int r = 0; r < 16; r++) {
                    const float x4 = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(
                        __builtin_bit_cast(int, v[r]), 0x1b, 0xf, 0xf, false));  // quad reversed
                    v[r] = ((k == 0 || k == 3) ? x4 : -x4) - P[r];
                }
            }
            if (whole) {
#pragma unroll
                for (int r = 0; r < 16; r++) at(r)[lane_off] = v[r];
            } else {
#pragma unroll
                for (int r = 0; r < 16; r++)
                    if (in(r)) at(r)[lane_off] = v[r];
            }
        }
    }
}

// ---------------------------------------------------------------------------------------
// Conversions between the FP32 rows [alm][C2] and the FP64 per-map alm layout
// [map][nalm] complex, through LDS-transposed tiles.
// ---------------------------------------------------------------------------------------
// alm FP64 [nb][nalm] (complex) -> x32 [nalm][C2] FP32, times f(l) (mode: 3 copy, 2 C^-1/2)
__global__ void __launch_bounds__(256)
k_alm_to_cols(const double2 *__restrict__ alm, float *__restrict__ x32,
              const double *__restrict__ cl, const int *__restrict__ lofi, long nalm, int nb,
              int C2, int mode, const ColScale *__restrict__ scale) {
    __shared__ float tile[64][65];  // [alm within tile][col within tile]
    const long i0 = (long)blockIdx.x * 64;
    const int c0 = blockIdx.y * 64;  // columns c0 .. c0+63 = maps c0/2 .. c0/2+31
    const int ii = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long ic = min(i0 + ii, nalm - 1);
    double f = 1.0;
    if (mode == 2) {
        const double C = cl[lofi[ic]];
        f = C > 0.0 ? 1.0 / sqrt(C) : 0.0;
    }
    double2 v[8];
#pragma unroll
    for (int u = 0; u < 8; u++) {  // clamped, so that all loads are in flight together
        const int b = min(c0 / 2 + w + 4 * u, nb - 1);
        const double fs = f * scale[b].s;
        const double2 x = alm[(long)b * nalm + ic];
        v[u] = make_double2(fs * x.x, fs * x.y);
    }
#pragma unroll
    for (int u = 0; u < 8; u++) {
        const int bb = w + 4 * u;
        const bool on = i0 + ii < nalm && c0 / 2 + bb < nb;
        tile[ii][2 * bb] = on ? (float)v[u].x : 0.f;
        tile[ii][2 * bb + 1] = on ? (float)v[u].y : 0.f;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 64 * 64; e += 256) {
        const int ii = e >> 6, cc = e & 63;
        const long i = i0 + ii;
        if (i < nalm && c0 + cc < C2) x32[i * C2 + c0 + cc] = tile[ii][cc];
    }
}

// x32 [nalm][C2] FP32 -> alm FP64 [nb][nalm], times f (mode 1: Omega; mode 3: 1)
__global__ void __launch_bounds__(256)
k_cols_to_alm(const float *__restrict__ x32, double2 *__restrict__ alm, long nalm, int nb, int C2,
              double scale, const ColScale *__restrict__ cscale) {
    __shared__ float tile[64][65];
    const long i0 = (long)blockIdx.x * 64;
    const int c0 = blockIdx.y * 64;
    for (int e = threadIdx.x; e < 64 * 64; e += 256) {
        const int ii = e >> 6, cc = e & 63;
        const long i = i0 + ii;
        tile[ii][cc] = (i < nalm && c0 + cc < C2) ? x32[i * C2 + c0 + cc] : 0.f;
    }
    const int ii = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double f[8];
#pragma unroll
    for (int u = 0; u < 8; u++) f[u] = scale * cscale[min(c0 / 2 + w + 4 * u, nb - 1)].inv;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 8; u++) {
        const int bb = w + 4 * u, b = c0 / 2 + bb;
        if (i0 + ii < nalm && b < nb)
            alm[(long)b * nalm + i0 + ii] = make_double2(f[u] * tile[ii][2 * bb], f[u] * tile[ii][2 * bb + 1]);
    }
}

// ---------------------------------------------------------------------------------------
// launch wrappers
// ---------------------------------------------------------------------------------------
int launch_lam_table(const Plan &p) {
    hipLaunchKernelGGL(k_lam_table, dim3(p.Rp / 64, p.nm), dim3(64), 0, p.stream, p.d_A, p.d_c,
                       p.d_mofs, p.d_kstart, p.d_entry, p.d_z, p.d_loff, p.d_Lp, p.d_lam, p.lmax,
                       p.npair);
    MFWF_HIP(hipGetLastError());
    return MFWF_OK;
}

int launch_lam_ckpt(const Plan &p) {
    hipLaunchKernelGGL(k_lam_ckpt, dim3(p.Rp / 64, p.nm), dim3(64), 0, p.stream, p.d_A, p.d_mofs,
                       p.d_kstart, p.d_entry, p.d_z, p.d_Lp, p.d_segoff, p.d_lck, p.lmax, p.npair,
                       p.Rp);
    MFWF_HIP(hipGetLastError());
    return MFWF_OK;
}

static int col_scale(const Plan &p, const double *x, long stride, long n0, long n1, double factor,
                     const double *cl, int both, int b0, int nb) {
    hipLaunchKernelGGL(k_col_scale, dim3(nb, n1 > 0 ? 2 : 1, col_scale_parts(n0)), dim3(256), 0, p.stream, x,
                       stride, n0, n1, factor, cl, p.d_lofi, both, p.Bp, p.d_cscale + b0, p.d_csearch + b0);
    MFWF_HIP(hipGetLastError());
    return MFWF_OK;
}

int launch_unit_scale(const Plan &p) {
    hipLaunchKernelGGL(k_unit_scale, dim3(1), dim3(256), 0, p.stream, p.d_cscale, p.d_csearch,
                       p.spin == 2 ? 2 * p.Bp : p.Bp);
    MFWF_HIP(hipGetLastError());
    return MFWF_OK;
}

// of the coefficients a transform reads (n = 2 nalm doubles a component), per map T and, spin 2, E
// and B
int launch_col_scale(const Plan &p, const double *x, long n, int mode, int nb) {
    return col_scale(p, x, p.ncomp * n, n, (p.ncomp - 1) * n, 1.0, mode == kHarmInvSqrtC ? p.d_cl : nullptr,
                     0, 0, nb);
}

// of the source rho of a solve's maps b0 .. b0 + nb - 1: the iterates are of the size of tau rho and
// above (tau M <= 1).  The components of T, Q, U mix in the update and share a scale.
int launch_col_scale_rho(const Plan &p, const double *rho, double tau, int b0, int nb) {
    return col_scale(p, rho, p.ncomp * p.npix, p.ncomp * p.npix, 0, tau, nullptr, p.spin == 2, b0, nb);
}

int launch_rows_to_cols(const Plan &p, int nb) {
    hipLaunchKernelGGL(k_rows_to_cols, dim3(p.nring, (p.nm + 63) / 64, (p.Bp + 63) / 64), dim3(256), 0,
                       p.stream, p.d_phf, p.d_ph32, p.nring, p.nm, p.nm32, nb, p.Bp, p.C2, p.d_cscale);
    MFWF_HIP(hipGetLastError());
    return MFWF_OK;
}

int launch_zero_map_cols(const Plan &p, int b) {
    const long nrows = (long)p.nm * p.nring;
    hipLaunchKernelGGL(k_zero_map_cols, dim3((unsigned)std::min<long>((nrows + 255) / 256, 4096)), dim3(256),
                       0, p.stream, p.d_ph32, nrows, p.C2, b);
    MFWF_HIP(hipGetLastError());
    return MFWF_OK;
}

int launch_cols_to_rows(const Plan &p, int nb) {
    hipLaunchKernelGGL(k_cols_to_rows, dim3(p.nring, (p.nm + 63) / 64, (nb + 63) / 64), dim3(256), 0,
                       p.stream, p.d_ph32, p.d_phf, p.nring, p.nm, p.nm32, nb, p.C2, p.d_cscale);
    MFWF_HIP(hipGetLastError());
    return MFWF_OK;
}

// active columns of a launch: the real columns of nb maps (per map w floats) rounded up to
// whole 32-column MFMA tiles; never beyond the padded width (w Bp, a multiple of 32)
static int active_cols(int nb, int w) { return 32 * ((w * nb + 31) / 32); }

// Column tile of a launch of the analysis (which = 0) or synthesis (1) over nc active columns for
// a choice 1: 64 columns, 2: 128, 3: 32: 32 columns where tiles of 64 would leave the chip's 512
// places for workgroups filled less than about twice (nside 128, 40 maps, 1028 such workgroups:
// synthesis 51 us with them, 34 with 32 columns; at nside 256, 20 maps, 2052 of them, 82 against
// 89), the narrowest that holds all columns, or else the choice; a forced choice as it is.  The
// analysis that generates lambda takes 128 columns for more than 32: each tile generates anew, and
// eight waves hide that better than four (nside 2048, lmax 4096, sht_fwd, ms with 64 / 128 columns:
// 24 maps 67.2 / 59.7, 32 maps 72.2 / 64.9; lmax 2048, 24 maps 26.6 / 24.4).
static int gemm_tile(const Plan &p, int which, int choice, int nc) {
    const int ct = choice == 2 ? 128 : (choice == 3 ? 32 : 64);
    if (p.gemm_forced[which]) return ct;
    const int ntile = 8 * (which ? p.syn_per_xcd : p.ana_per_xcd);
    if (ntile * ((nc + 63) / 64) < 1200) return 32;
    if (nc <= 32) return 32;
    if (p.lam_gen && which == 0) return 128;
    return nc <= 64 ? std::min(ct, 64) : ct;
}

int gemm_effective(const Plan &p, int which, int choice) {
    const int ct = gemm_tile(p, which, choice, active_cols(p.max_batch, p.spin == 2 ? 4 : 2));
    return ct == 128 ? 2 : (ct == 32 ? 3 : 1);
}

static LamGen lam_gen(const Plan &p) {
    return LamGen{p.d_lck, p.d_segoff, p.d_z, p.d_A, p.d_c};
}

// table == nullptr: lambda rows generated in the kernels (the plan's segment states)
static int analysis_launch(const Plan &p, int nc, int C2, const float *table, const float *cols,
                           float *a_out, float *s_out, double scale_s, double lto,
                           const double *tau_b, double lto_per_tau, int flip) {
    const int ct = gemm_tile(p, 0, p.gemm_ct[0], nc), ncg = (nc + ct - 1) / ct;
    const dim3 grid(8 * p.ana_per_xcd * ncg), block(ct == 64 ? 256 : 512);
    const LamGen g = lam_gen(p);
    if (table == nullptr && !p.d_lck) return fail(MFWF_EINVAL, "no lambda segment states in this plan");
#define MFWF_ANA(CT, GEN)                                                                          \
    hipLaunchKernelGGL((k_gemm_analysis<CT, GEN>), grid, block, 0, p.stream, table, g, p.d_loff,     \
                       p.d_Lp, p.d_minls32, p.d_ana_items, p.d_ana_tab, p.ana_per_xcd, cols,         \
                       p.d_mofs, p.d_cl, a_out, s_out, scale_s, lto, p.lmax, p.npair, p.Rp,          \
                       p.nring, p.nm, C2, nc, ncg, tau_b, lto_per_tau, flip, p.d_zrow)
    if (table == nullptr) {
        if (ct == 128) MFWF_ANA(128, true);
        else if (ct == 64) MFWF_ANA(64, true);
        else MFWF_ANA(32, true);
    } else {
        if (ct == 128) MFWF_ANA(128, false);
        else if (ct == 64) MFWF_ANA(64, false);
        else MFWF_ANA(32, false);
    }
#undef MFWF_ANA
    MFWF_HIP(hipGetLastError());
    return MFWF_OK;
}

// Streaming loads of the table, which leave the 256 MB last-level cache to coefficients and rings,
// where one column group reads the table (with two, the second finds the first one's rows in L2:
// nside 256, 64 maps, us a call of sht_inv 795 cached, 803 streaming) and it is somewhat larger than
// that cache: a smaller one stays there from one contraction to the next, and of a much larger one
// nothing is lost.  An iteration, us cached / streaming, with 1, 4, 24 maps: 130 MB (nside 256) 97 / 105,
// 118 / 124, 345 / 349; 260 MB (nside 512) 202 / 206, 283 / 285; 321 MB (nside 256) 190 / 184, 216 / 204, 501 / 490;
// 542 MB 292 / 278, 320 / 305, 657 / 653; 642 MB (nside 512) 375 / 366, 457 / 451; 1143 MB 581 / 579, 672 / 676;
// 2308 MB 1048 / 1065, 1159 / 1175.
static bool synthesis_once(const Plan &p, int ncg) {
    return ncg == 1 && p.table_bytes > (288L << 20) && p.table_bytes <= (768L << 20);
}

static int synthesis_launch(const Plan &p, int nc, int C2, const float *table, const float *s_in,
                            float *out, int flip, int comb) {
    const int ct = gemm_tile(p, 1, p.gemm_ct[1], nc), ncg = (nc + ct - 1) / ct;
    const dim3 grid(8 * p.syn_per_xcd * ncg), block(ct == 64 ? 256 : 512);
    const LamGen g = lam_gen(p);
    if (table == nullptr && !p.d_lck) return fail(MFWF_EINVAL, "no lambda segment states in this plan");
#define MFWF_SYN(CT, GEN, ONCE)                                                                     \
    hipLaunchKernelGGL((k_gemm_synthesis<CT, GEN, ONCE>), grid, block, 0, p.stream, table, g, p.d_loff,\
                       p.d_Lp, p.d_minls32, p.d_syn_items, p.d_syn_tab, p.syn_per_xcd, s_in,          \
                       p.d_mofs, out, p.lmax, p.npair, p.Rp, p.nring, p.nm, C2, nc, ncg, flip, comb)
    if (table == nullptr) {
        if (ct == 128) MFWF_SYN(128, true, false);
        else if (ct == 64) MFWF_SYN(64, true, false);
        else MFWF_SYN(32, true, false);
    } else if (synthesis_once(p, ncg)) {
        if (ct == 128) MFWF_SYN(128, false, true);
        else if (ct == 64) MFWF_SYN(64, false, true);
        else MFWF_SYN(32, false, true);
    } else {
        if (ct == 128) MFWF_SYN(128, false, false);
        else if (ct == 64) MFWF_SYN(64, false, false);
        else MFWF_SYN(32, false, false);
    }
#undef MFWF_SYN
    MFWF_HIP(hipGetLastError());
    return MFWF_OK;
}

int launch_gemm_analysis(const Plan &p, int nb, float *a_out, float *s_out, double scale_s,
                         double lto, double lto_per_tau) {
    return analysis_launch(p, active_cols(nb, 2), p.C2, p.lam_gen ? nullptr : p.d_lam, p.d_ph32,
                           a_out, s_out, scale_s,
                           lto, s_out ? p.d_tau : nullptr, lto_per_tau, 0);
}

int launch_gemm_synthesis(const Plan &p, int nb) {
    return synthesis_launch(p, active_cols(nb, 2), p.C2, p.lam_gen ? nullptr : p.d_lam, p.d_s32,
                            p.d_ph32, 0, 0);
}

// Raw analysis sums a_out[alm][w Bp] = table x cols[m][ring][w Bp] for nb maps of w columns
int launch_gemm_analysis_raw(const Plan &p, int nb, int w, const float *table, const float *cols,
                             float *a_out, int flip) {
    return analysis_launch(p, active_cols(nb, w), w * p.Bp, table, cols, a_out, nullptr, 0.0, 0.0,
                           nullptr, 0.0, flip);
}

// Synthesis out[m][ring][w Bp] = table x s_in[alm][w Bp] for nb maps of w columns; comb
// (w = 4): out holds P' and receives (Q, U) formed from it and this product R'
int launch_gemm_synthesis_on(const Plan &p, int nb, int w, const float *table, const float *s_in,
                             float *out, int flip, int comb) {
    if (comb && w != 4) return fail(MFWF_EINVAL, "combined synthesis needs four columns per map");
    return synthesis_launch(p, active_cols(nb, w), w * p.Bp, table, s_in, out, flip, comb);
}

int launch_alm_to_cols(const Plan &p, const double2 *alm, float *x32, int nb, int mode) {
    hipLaunchKernelGGL(k_alm_to_cols, dim3((p.nalm + 63) / 64, (p.C2 + 63) / 64), dim3(256), 0,
                       p.stream, alm, x32, p.d_cl, p.d_lofi, p.nalm, nb, p.C2, mode, p.d_cscale);
    MFWF_HIP(hipGetLastError());
    return MFWF_OK;
}

int launch_cols_to_alm(const Plan &p, const float *x32, double2 *alm, int nb, double scale) {
    hipLaunchKernelGGL(k_cols_to_alm, dim3((p.nalm + 63) / 64, (p.C2 + 63) / 64), dim3(256), 0,
                       p.stream, x32, alm, p.nalm, nb, p.C2, scale, p.d_cscale);
    MFWF_HIP(hipGetLastError());
    return MFWF_OK;
}

}  // namespace mfwf
