// Exact greedy round-to-nearest of a multi-word integer into m doubles: the
// renormalisation step of the m-double product (the paper's postponed
// renormalisation, done once per output entry).
//
// The value is X 2^scale with X an integer held as 4 beta-bit columns
// (carried, the top one signed) and then in 32-bit two's complement limbs
// L[0..NL).
// Word t is RN(X_t 2^scale), X_0 = X, X_(t+1) = X_t - word t, round to
// nearest with ties to even and the unit clamped at 2^-1074 (subnormal
// words).  Every limb index is a compile-time constant, so the limbs stay in
// registers: data-dependent positions become selects and shift networks.
//
// Plain C++ apart from the __device__ __forceinline__ annotations, so that a
// host build of this header can be checked against an exact reference.
#pragma once

#include <cmath>
#include <cstdint>

namespace mdg {

__device__ __forceinline__ int imax(int a, int b) { return a > b ? a : b; }

// Register layout for S diagonals of B-bit digits (B = 7 or 8): four
// diagonals per column, kCols columns of weight 2^(kCW j) (the top one takes
// only carries and is signed) and the kLimbs 32-bit limbs of the magnitude
// (kCols-1 columns of kCW bits, a top one below 2^64).
template <int S, int B = 7>
struct Tri {
    static constexpr int kCW = 4 * B;
    static constexpr int kCols = (S + 3) / 4 + 1;
    static constexpr int kLimbs = (kCW * (kCols - 1) + 64 + 31) / 32;
};

// Carry every column but the top one into [0, 2^CW).
template <int CW, int NC>
__device__ __forceinline__ void carry_cols(int64_t (&x)[NC])
{
#pragma unroll
    for (int j = 0; j + 1 < NC; ++j) {
        x[j + 1] += x[j] >> CW;
        x[j] &= ((int64_t)1 << CW) - 1;
    }
}

// Limb k of the integer whose limb 0 is zero and limbs 1..NL are L[0..NL-1]
// (bits of X shifted up by 32, so that bit unit-1 >= -1 of X has a place).
template <int NL>
__device__ __forceinline__ uint32_t shifted_limb(const uint32_t (&L)[NL], int k)
{
    return (k >= 1 && k <= NL) ? L[k - 1] : 0u;
}

// One greedy round-to-nearest step on (-1)^neg X 2^scale, X >= 0 held in
// 32-bit limbs L: returns the word RN(X 2^scale) (with sign) and leaves the
// remainder in L and its sign in sgn.  Any unit (clamped at 2^-1074 and at
// bit 0 of X); no branches, so that the steps of several outputs interleave.
template <int NL>
__device__ __forceinline__ double rn_step(uint32_t (&L)[NL], double& sgn, int umin, int scale)
{
    int top = -1;
#pragma unroll
    for (int k = 0; k < NL; ++k)
        top = L[k] ? 32 * k + 31 - __builtin_clz(L[k]) : top;
    const int unit = imax(imax(top - 52, umin), 0);
    // 64 bits of X from bit unit-1: the round bit, then the 53-bit
    // significand; sticky: any bit below unit-1
    const int P = unit + 31, q = P >> 5, r = P & 31;
    uint32_t l0 = 0, l1 = 0, l2 = 0, st = 0;
#pragma unroll
    for (int k = 0; k <= NL; ++k) {
        const uint32_t v = shifted_limb(L, k);
        st |= k < q ? v : (k == q ? v & ((1u << r) - 1u) : 0u);
        l0 = k == q ? v : l0;
        l1 = k == q ? shifted_limb(L, k + 1) : l1;
        l2 = k == q ? shifted_limb(L, k + 2) : l2;
    }
    const uint64_t lo = (uint64_t)l0 | ((uint64_t)l1 << 32);
    const uint64_t win = r ? ((lo >> r) | ((uint64_t)l2 << (64 - r))) : lo;
    uint64_t n = win >> 1;
    const bool up = (win & 1) && (st || (n & 1));
    n += up;
    const double w = top >= 0 ? sgn * ldexp((double)n, unit + scale) : 0.0;
    // remainder: the bits below unit; rounded up, 2^unit minus them with the
    // sign flipped
    uint64_t cy = 1;
#pragma unroll
    for (int k = 0; k < NL; ++k) {
        const int b = unit - 32 * k;
        const uint32_t keep = b >= 32 ? ~0u : (b <= 0 ? 0u : (1u << b) - 1u);
        const uint64_t v = (uint64_t)(~L[k]) + cy;
        cy = v >> 32;
        L[k] = (up ? (uint32_t)v : L[k]) & keep;
    }
    sgn = up ? -sgn : sgn;
    return w;
}

// Signed form: X = sg 2^(32 NL) + U, U the unsigned integer in the limbs and
// sg 0 or -1 (the limbs are X's two's complement, sg its sign).  A greedy
// step then needs no magnitude: n = floor(X / unit) rounds up by the round,
// sticky and odd bits whatever the sign, and the remainder, the bits below
// the unit minus the unit if it rounded up, is those bits with sg = -1: no
// negation, no carry chain.  (Rounding |X| instead, with the remainder
// negated when it flips sign, took about 2.5 times the instructions per
// word: quad-double 1024^3 330 us a call against 319, hexa-double 1024^3 2158
// against 2046.)
// The unit of a negative X comes from its leading sign bits; X = -2^t, whose
// magnitude has one bit more than they say, is exact at either unit.

// Limbs k - 1 and k as one number, shifted left by r in [0, 31]: limb k.
__device__ __forceinline__ uint32_t limb_left(uint32_t lo, uint32_t hi, int r)
{
    return (uint32_t)((((uint64_t)hi << 32 | lo) << r) >> 32);
}

// Shift the limbs left by r in [0, 31] bits whose upper neighbours are sign
// bits; X 2^scale is kept.
template <int NL>
__device__ __forceinline__ void shift_bits(uint32_t (&L)[NL], int r, int& scale)
{
#pragma unroll
    for (int k = NL - 1; k >= 0; --k)
        L[k] = limb_left(k ? L[k - 1] : 0u, L[k], r);
    scale -= r;
}

// Shift the limbs left until bit 32 NL - 1 differs from the sign; X 2^scale
// is kept.  False if X is zero.
template <int NL>
__device__ __forceinline__ bool align_signed(uint32_t (&L)[NL], int32_t sg, int& scale)
{
    int top = -1;
#pragma unroll
    for (int k = 0; k < NL; ++k)
        top = (L[k] ^ (uint32_t)sg) ? 32 * k + 31 - __builtin_clz(L[k] ^ (uint32_t)sg) : top;
    // no bit differs: zero, or -1, whose bits all leave (X = -2^(32 NL))
    const int d = top < 0 ? (sg ? 32 * NL : 0) : 32 * NL - 1 - top;
    const int q = d >> 5, r = d & 31;
    // whole limbs: a shift by q as a network of shifts by 1, 2, 4, 8 limbs
#pragma unroll
    for (int b = 1; b <= NL; b <<= 1) {
        const bool on = (q & b) != 0;
#pragma unroll
        for (int k = NL - 1; k >= 0; --k)
            L[k] = on ? (k >= b ? L[k - b] : 0u) : L[k];
    }
    scale -= 32 * q;
    shift_bits(L, r, scale);
    return top >= 0 || sg;
}

// |X| in the limbs and its sign; X = -2^(32 NL) first moves down a bit.
template <int NL>
__device__ __forceinline__ double to_magnitude(uint32_t (&L)[NL], int32_t sg, int& scale)
{
    uint32_t any = 0;
    uint64_t cy = 1;
#pragma unroll
    for (int k = 0; k < NL; ++k) {
        any |= L[k];
        const uint64_t v = (uint64_t)(~L[k]) + cy;
        cy = v >> 32;
        L[k] = sg ? (uint32_t)v : L[k];
    }
    if (sg && !any) {
        L[NL - 1] = 0x80000000u;
        scale += 1;
    }
    return sg ? -1.0 : 1.0;
}

// X from its magnitude in the limbs; returns sg.
template <int NL>
__device__ __forceinline__ int32_t from_magnitude(uint32_t (&L)[NL], double sgn)
{
    uint32_t any = 0;
    uint64_t cy = 1;
#pragma unroll
    for (int k = 0; k < NL; ++k) {
        any |= L[k];
        const uint64_t v = (uint64_t)(~L[k]) + cy;
        cy = v >> 32;
        L[k] = sgn < 0.0 ? (uint32_t)v : L[k];
    }
    return sgn < 0.0 && any ? -1 : 0;
}

// One greedy round-to-nearest step on X 2^scale: returns the word and leaves
// the remainder.  A remainder left by a step has sign bits down to bit
// 32 NL - 53, so it moves up by 53 bits at fixed places and then by the top
// limb's remaining sign bits; only the first word, or a remainder with 32
// more sign bits, takes the limb network.  The general step serves words
// whose unit would fall below 2^-1074.
template <int NL>
__device__ __forceinline__ double rn_signed(uint32_t (&L)[NL], int32_t& sg, int& scale)
{
    static_assert(NL >= 3, "at least three limbs");
    const uint32_t fill = (uint32_t)sg;
    if (L[NL - 1] == fill && ((L[NL - 2] ^ fill) >> 11) == 0) {
#pragma unroll
        for (int k = NL - 1; k >= 0; --k)
            L[k] = k >= 2 ? (L[k - 1] << 21) | (L[k - 2] >> 11) : (k == 1 ? L[0] << 21 : 0u);
        scale -= 53;
    }
    if (L[NL - 1] != fill)
        shift_bits(L, __builtin_clz(L[NL - 1] ^ fill), scale);
    else if (!align_signed(L, sg, scale))
        return 0.0;
    if (32 * NL - 53 + scale < -1074) {
        double sgn = to_magnitude(L, sg, scale);
        const double w = rn_step(L, sgn, -1074 - scale, scale);
        sg = from_magnitude(L, sgn);
        return w;
    }
    // significand, round and sticky bits at fixed places
    const uint64_t n = ((uint64_t)L[NL - 1] << 21) | (L[NL - 2] >> 11);
    uint32_t st = L[NL - 2] & 0x3ffu;
#pragma unroll
    for (int k = 0; k < NL - 2; ++k)
        st |= L[k];
    const uint32_t up = (L[NL - 2] >> 10) & (uint32_t)(st != 0 || (n & 1));
    const uint32_t rnd = up & 1u;
    // |n + rnd - 2^53 (negative X)| <= 2^53: exact
    const int64_t v = (int64_t)(n + rnd) + (int64_t)((uint64_t)(int64_t)sg << 53);
    const double w = ldexp((double)v, 32 * NL - 53 + scale);
    sg = -(int32_t)rnd;
    L[NL - 1] = (uint32_t)sg;
    L[NL - 2] = (L[NL - 2] & 0x7ffu) | ((uint32_t)sg << 11);
    return w;
}

// The same on a sign and magnitude (-1)^neg X 2^scale, X >= 0 in the limbs:
// with to_limbs the form in which the host tests put integers to the steps;
// the kernels hold two's complement (rn_signed, to_limbs_signed).
template <int NL>
__device__ __forceinline__ double rn_next(uint32_t (&L)[NL], double& sgn, int& scale)
{
    int32_t sg = from_magnitude(L, sgn);
    const double w = rn_signed(L, sg, scale);
    sgn = to_magnitude(L, sg, scale);
    return w;
}

// Magnitude limbs of the carried CW-bit columns; returns the sign.
template <int CW, int NC, int NL>
__device__ __forceinline__ bool to_limbs(int64_t (&x)[NC], uint32_t (&L)[NL])
{
    const bool neg = x[NC - 1] < 0;
#pragma unroll
    for (int j = 0; j < NC; ++j)
        x[j] = neg ? -x[j] : x[j];
    carry_cols<CW>(x);
#pragma unroll
    for (int k = 0; k < NL; ++k)
        L[k] = 0;
#pragma unroll
    for (int j = 0; j < NC; ++j) {
        const uint64_t v = (uint64_t)x[j];
        const int b = CW * j, k = b >> 5, r = b & 31;
        L[k] |= (uint32_t)(v << r);
        if (k + 1 < NL)
            L[k + 1] |= (uint32_t)(r ? v >> (32 - r) : v >> 32);
        if (k + 2 < NL && r)
            L[k + 2] |= (uint32_t)(v >> (64 - r));
    }
    return neg;
}

// Two's complement limbs of the carried CW-bit columns (the top one signed);
// returns the sign word.
template <int CW, int NC, int NL>
__device__ __forceinline__ int32_t to_limbs_signed(const int64_t (&x)[NC], uint32_t (&L)[NL])
{
    static_assert(CW * (NC - 1) + 64 > 32 * (NL - 1) && CW * (NC - 1) + 64 <= 32 * NL, "the top column ends in the top limb");
#pragma unroll
    for (int k = 0; k < NL; ++k)
        L[k] = 0;
#pragma unroll
    for (int j = 0; j < NC; ++j) {
        const uint64_t v = (uint64_t)x[j];
        const int b = CW * j, k = b >> 5, r = b & 31;
        L[k] |= (uint32_t)(v << r);
        if (k + 1 < NL)
            L[k + 1] |= (uint32_t)(r ? v >> (32 - r) : v >> 32);
        if (k + 2 < NL && r)
            L[k + 2] |= (uint32_t)(v >> (64 - r));
    }
    const int32_t sg = x[NC - 1] < 0 ? -1 : 0;
    constexpr int pos = CW * (NC - 1) + 64 - 32 * (NL - 1);   // top limb's bits from here up: the sign
    if (pos < 32)
        L[NL - 1] |= (uint32_t)sg << (pos & 31);
    return sg;
}

}  // namespace mdg
