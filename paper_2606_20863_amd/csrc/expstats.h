// The call statistics from the exponent pass's row blocks.
#pragma once

#include "mdgemm_internal.h"

#include <climits>

namespace mdg {
namespace {

// Block blk's {span, largest, smallest shared exponent} at lo[4 blk], for
// one operand of n blocks, reduced by 256 threads into the operand's span
// maximum and extreme exponents.
__device__ __forceinline__ void exp_block_stats(const int32_t* lo, int64_t n, int32_t* span_max, int32_t* ext)
{
    __shared__ int red[3][4];
    int span = 0, emax = INT_MIN, emin = INT_MAX;
    for (int64_t b = threadIdx.x; b < n; b += 256) {
        span = max(span, lo[4 * b]);
        emax = max(emax, lo[4 * b + 1]);
        emin = min(emin, lo[4 * b + 2]);
    }
    for (int o = 1; o < 64; o <<= 1) {
        span = max(span, __shfl_xor(span, o));
        emax = max(emax, __shfl_xor(emax, o));
        emin = min(emin, __shfl_xor(emin, o));
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = span;
        red[1][threadIdx.x >> 6] = emax;
        red[2][threadIdx.x >> 6] = emin;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        *span_max = max(max(red[0][0], red[0][1]), max(red[0][2], red[0][3]));
        ext[0] = max(max(red[1][0], red[1][1]), max(red[1][2], red[1][3]));
        ext[1] = min(min(red[2][0], red[2][1]), min(red[2][2], red[2][3]));
    }
}

}  // namespace
}  // namespace mdg
