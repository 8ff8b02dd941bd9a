// Device-side helpers shared by the HIP translation units of libah.
#pragma once

#include "ah_internal.h"

namespace ah {

// Fold nblocks diagnostics records (kMeasStride doubles each) into
// out[0 .. M_COUNT) with kFoldThreads threads in a fixed order.  Sums except
// M_GMAX, which is max-reduced.  `red` is kFoldRed doubles of LDS.
//
// One block folds the records of a lattice (a few hundred to a few thousand
// of 128 bytes), so its time is latency.  Thread t takes slot t % 16 of the
// records t / 16, t / 16 + 64, ..., so that all slots go through one chain of
// whole-line loads (eight in flight), shuffles and one pass through LDS,
// rather than through a chain and a barrier tree per slot, one slot after
// another.  With the record written straight to the host this took
// ah_measure of a 32^3 FP32 lattice on MI355X from 48.8 us (a slot at a time
// and a copy behind it) to 35.6, of a 256^3 FP64 lattice from 859 us to 843
// (26.5 and 650 us with the present march).
constexpr int kFoldThreads = 1024;
constexpr int kFoldRed = kFoldThreads / 64 * kMeasStride;
__device__ inline void fold_records(const double* __restrict__ partials, int nblocks, double* __restrict__ out,
                                    double* red)
{
    static_assert(kMeasStride == 16, "a record is 16 slots: four records per wave");
    constexpr int kRows = kFoldThreads / kMeasStride, kUnroll = 8;
    const int k = threadIdx.x % kMeasStride, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const auto add = [&](double a, double b) { return k == M_GMAX ? fmax(a, b) : a + b; };
    double r = 0.0;
    for (int b = threadIdx.x / kMeasStride; b < nblocks; b += kRows * kUnroll) {
        double v[kUnroll];
        for (int j = 0; j < kUnroll; ++j) {
            const int i = b + j * kRows;
            v[j] = i < nblocks ? partials[(int64_t)i * kMeasStride + k] : 0.0;
        }
        for (int j = 0; j < kUnroll; ++j) r = add(r, v[j]);
    }
    r = add(r, __shfl_xor(r, 16, 64));
    r = add(r, __shfl_xor(r, 32, 64));
    if (lane < kMeasStride) red[wv * kMeasStride + lane] = r;
    __syncthreads();
    if (threadIdx.x < 64) {
        // four of the waves' sums per lane, then the four lanes of a slot
        const double* q = red + (lane / kMeasStride) * 4 * kMeasStride + k;
        r = add(add(q[0], q[kMeasStride]), add(q[2 * kMeasStride], q[3 * kMeasStride]));
        r = add(r, __shfl_xor(r, 16, 64));
        r = add(r, __shfl_xor(r, 32, 64));
        if (lane < M_COUNT) out[lane] = r;
    }
}

}  // namespace ah
