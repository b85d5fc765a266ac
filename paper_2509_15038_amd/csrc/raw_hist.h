// Histograms of scores for the split selection (split_select.hip), made by the workgroups that score
// or by a kernel that reads scores from memory; for gfx950.
#pragma once

#include "curdkv_internal.h"

namespace curdkv {

// 4096 bins of a score, normalised or not:
// exponent and top four mantissa bits of a non-negative float, 16 bins per binade whatever its size.
// A workgroup counts fewer than 65536 tokens, 16 bits each, two to a word.
constexpr int kRawShift = 19;
constexpr int kRawHistWords = 2048;

// v: a score (never negative).  counts = false adds nothing, without a branch.
__device__ __forceinline__ void raw_hist_count(uint32_t* hist, float v, bool counts = true) {
    const uint32_t bits = __float_as_uint(v);
    const uint32_t one = (bits >> kRawShift) & 1u ? 0x10000u : 1u;
    atomicAdd(&hist[(bits >> (kRawShift + 1)) & (kRawHistWords - 1)], counts ? one : 0u);
}

// Takes back what raw_hist_count added for the same v and `counts`.
__device__ __forceinline__ void raw_hist_uncount(uint32_t* hist, float v, bool counts = true) {
    const uint32_t bits = __float_as_uint(v);
    const uint32_t one = (bits >> kRawShift) & 1u ? 0x10000u : 1u;
    atomicSub(&hist[(bits >> (kRawShift + 1)) & (kRawHistWords - 1)], counts ? one : 0u);
}

// Writes the workgroup's histogram (complete, in LDS) and its sums per exponent to place `at`.
template <int THREADS>
__device__ __forceinline__ void raw_hist_store(const uint32_t* hist, uint32_t* __restrict__ out,
                                               uint32_t* __restrict__ coarse, int at) {
    out += (size_t)at * kRawHistWords;
    coarse += (size_t)at * 256;
    for (int i = threadIdx.x; i < kRawHistWords; i += THREADS) out[i] = hist[i];
    for (int e = threadIdx.x; e < 256; e += THREADS) {
        uint32_t sum = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t w = hist[8 * e + i];
            sum += (w & 0xFFFFu) + (w >> 16);
        }
        coarse[e] = sum;
    }
}

}  // namespace curdkv
