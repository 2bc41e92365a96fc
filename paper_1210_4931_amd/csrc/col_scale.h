// The scale of a map's FP32 columns.  The contractions split FP32 values into bf16 pieces; the last
// piece of a value below 2^-110 lies below bf16's smallest number, so small maps would lose
// bits that FP32 keeps down to 2^-126 (1.3e-7 relative error, but 2.6e-4 at 1e-37).  The
// columns of a map therefore carry the map times a power of two, which changes no rounding:
// 2^40 if no value of the map reaches 2^-70, else 1.  The regrouping and conversion kernels and the
// ring step apply it and take it off; everything else is linear in it.
#pragma once

#include "mfwf_internal.h"

namespace mfwf {

static constexpr double kSmallMap = 0x1p-70;
static constexpr ColScale kUnitScale{1.0, 1.0, 1.f, 1.f}, kSmallScale{0x1p40, 0x1p-40, 0x1p40f, 0x1p-40f};

// The search for a value that reaches 2^-70 (a NaN does) among n, by col_scale_parts(n)
// workgroups of T threads, part = 0, 1, ..: each looks at one value per thread first, spread over
// its share, which ends it on any map that is not small or nearly empty (two memory latencies), then
// through its share in order, until one is found there or by another part; the last part to
// finish writes the scale and clears the state for the next search.  One workgroup took 0.65 ms for
// a zero map of nside 512 (25 MB), sixteen 0.02 ms.  More parts than
// the size asks for hold places that the transforms beside them wait for (nside 128, 7 maps: a call
// of sht_fwd 95 us with one or three, 99 with sixteen).
static inline int col_scale_parts(long n) { return (int)(n < (2L << 16) ? 1 : (n < (16L << 16) ? n >> 16 : 16)); }

template <int T, typename F>
__device__ __forceinline__ void find_col_scale(long n, int part, int parts, int *lds, ColScaleSearch *st,
                                               ColScale *out, ColScale *out2, F value) {
    const long len = (n + parts - 1) / parts, lo = min(part * len, n - 1), hi = min(lo + len, n);
    auto any = [&](bool mine) {  // over the workgroup; another part's find counts too
        if (threadIdx.x == 0) *lds = __hip_atomic_load(&st->found, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (mine) *lds = 1;
        __syncthreads();
        const bool r = *lds != 0;
        __syncthreads();
        return r;
    };
    auto reaches = [&](long i) { return !(fabs(value(i)) < kSmallMap); };
    bool big = any(reaches(min(lo + threadIdx.x * max((hi - lo) / T, 1L), hi - 1)));
    for (long k = lo; k < hi && !big; k += 16L * T) {
        bool mine = false;
#pragma unroll
        for (int u = 0; u < 16; u++) mine |= reaches(min(k + (long)T * u + threadIdx.x, hi - 1));
        big = any(mine);
    }
    if (threadIdx.x != 0) return;
    if (big) __hip_atomic_store(&st->found, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // every part's find is visible to the one that counts last
    if (__hip_atomic_fetch_add(&st->done, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) != parts - 1) return;
    const ColScale s = __hip_atomic_load(&st->found, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ? kUnitScale : kSmallScale;
    *out = s;
    if (out2) *out2 = s;
    st->found = st->done = 0;
}

}  // namespace mfwf
