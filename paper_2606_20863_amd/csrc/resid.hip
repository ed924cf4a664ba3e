// The residue contraction (resid.h): tables, evaluation, the batched INT8
// products and the interpolation with the exact fold and rounding.
#include "resid.h"
#include "ldslimbs.h"
#include "renorm.h"
#include "split.h"

#include <algorithm>
#include <cmath>

namespace mdg {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));

// the largest primes below 256; eight multiply to 2^62.8
constexpr int kPrimes[kResMaxPrimes] = {251, 241, 239, 233, 229, 227, 223, 211};

__device__ const int d_primes[kResMaxPrimes] = {251, 241, 239, 233, 229, 227, 223, 211};

int64_t round_up64(int64_t x, int64_t q) { return (x + q - 1) / q * q; }
// 64-depth chunks of the residue planes: an even number, at least 4
int64_t res_steps(int64_t K) { return std::max<int64_t>(4, (K + 2 * kKcI8 - 1) / (2 * kKcI8) * 2); }
size_t up256(size_t x) { return (x + 255) / 256 * 256; }

// Tables of one call in scratch: evaluation weights of both operands
// ([planes padded to 16][64 kt] bytes), moduli per plane ({1 / p, p} as
// floats), interpolation weights ([prime][L padded to 16][N padded to 32]
// bytes).
struct ResTables {
    int8_t *VA, *VB, *W;
    float2* pc;
    int Lp, Np, KD, pl16;
    int packed;
};

struct ResShape {   // plan values the kernels use
    int L, N, P, SB, nb, S, beta, nbd;
};

// v mod p in [0, p), 0 <= v < 2^23
__device__ __forceinline__ int umod(int v, int p, float inv)
{
    int r = v - p * (int)((float)v * inv);
    r += r < 0 ? p : 0;
    return r >= p ? r - p : r;
}

__device__ __forceinline__ int centred(int r, int p) { return r > p / 2 ? r - p : r; }

constexpr int kResGroups = 256;   // workgroups of the products: one per compute unit

// Two workgroups of 512 threads per prime, one for the evaluation weights and
// one for the interpolation's, and one for the last diagonal's rows.  Point j: 0, +1, -1, +2, -2, ..  The interpolation weights come from
// Q(x) = x G(x^2), G(z) = prod_i (z - i^2): Q / (x - x_j) is G(x^2) for the
// point 0 and (x^2 + x_j x) H_i(x^2), H_i = G / (z - i^2), for +-i, with
// Q'(x_j) = G(0) or 2 i^2 H_i(i^2).  The Chinese remainder's factor
// (M / p)^-1 is folded in.  It takes a few microseconds against products of
// hundreds, and nothing has to be kept between calls.
__global__ __launch_bounds__(512) void k_res_tables(ResShape s, ResTables t)
{
    const int tid = threadIdx.x, i = blockIdx.x >> 1;
    if (i == s.P) {
        // last diagonal: one digit per plane, modulus 256 (the digit itself).
        // A plane q takes digit 2 q, B plane q the digit that completes S - 1.
        const int q0 = s.N * s.P;
        for (int e = tid; e < (t.pl16 - q0) * t.KD; e += 512) {
            const int q = e / t.KD, u = e % t.KD;
            t.VA[(int64_t)(q0 + q) * t.KD + u] = q < s.nbd && u == 2 * q;
            t.VB[(int64_t)(q0 + q) * t.KD + u] = q < s.nbd && u == s.S - 1 - 2 * q;
        }
        for (int q = tid; q < t.pl16 - q0; q += 512)
            t.pc[q0 + q] = float2{1.0f / 256.0f, 256.0f};
        return;
    }
    __shared__ int G[96], H[96][97], den[96];
    __shared__ int crt;
    const int p = d_primes[i], L = s.L;
    const float inv = 1.0f / (float)p;
    // evaluation weights: thread (part, j) takes a quarter of the digits
    if ((blockIdx.x & 1) == 0) {
        const int j = tid & 127, part = tid >> 7;
        const int per = (t.KD + 3) / 4;
        for (int jj = j; jj < s.N; jj += 128) {
            const int xi = (jj + 1) / 2;
            const int x = (jj & 1) || xi == 0 ? xi : p - xi;
            const int row = i * s.N + jj;
            t.pc[row] = float2{inv, (float)p};
            if (s.nb) {   // FP64 digits: byte k of digit d weighs x^d 256^k
                int d = (part * per) / s.nb, pw = 1;
                for (int b = 1, e = x; b <= d; b <<= 1) {
                    pw = (d & b) ? umod(pw * e, p, inv) : pw;
                    e = umod(e * e, p, inv);
                }
                int u = d * s.nb;
                for (; d < L && u < (part + 1) * per; ++d) {
                    int v = pw;
                    for (int k = 0; k < s.nb; ++k, ++u) {
                        if (u >= part * per && u < (part + 1) * per)
                            t.VA[(int64_t)row * t.KD + u] = t.VB[(int64_t)row * t.KD + u] = (int8_t)centred(v, p);
                        v = umod(v * 256, p, inv);
                    }
                    pw = umod(pw * x, p, inv);
                }
                for (u = max(u, part * per); u < min((part + 1) * per, t.KD); ++u)
                    t.VA[(int64_t)row * t.KD + u] = t.VB[(int64_t)row * t.KD + u] = 0;
            } else {
                // INT8 pairs: digit u of A is in block u / 2, of B in block
                // (u + 1 - S % 2) / 2; the upper digit of a pair weighs 2^beta
                const int base = umod(1 << s.beta, p, inv);
                for (int side = 0; side < 2; ++side) {
                    const int sh = side && s.S % 2 == 0 ? 1 : 0;
                    int8_t* V = side ? t.VB : t.VA;
                    int u = part * per, c = (u + sh) / 2, pw = 1;
                    for (int b = 1, e = x; b <= c; b <<= 1) {
                        pw = (c & b) ? umod(pw * e, p, inv) : pw;
                        e = umod(e * e, p, inv);
                    }
                    for (; u < min((part + 1) * per, t.KD); ++u) {
                        const bool low = (u + sh) & 1;
                        const int v = low ? pw : umod(pw * base, p, inv);
                        V[(int64_t)row * t.KD + u] = c < L && u < s.S ? (int8_t)centred(v, p) : 0;
                        if (low) {
                            pw = umod(pw * x, p, inv);
                            ++c;
                        }
                    }
                }
            }
        }
    }
    if ((blockIdx.x & 1) == 0)
        return;
    // G, one factor (z - i^2) after the other
    if (tid < 96)
        G[tid] = tid == 0;
    if (tid == 511) {
        int m = 1;
        for (int q = 0; q < s.P; ++q)
            m = q == i ? m : umod(m * d_primes[q], p, inv);
        int e = p - 2, r = 1;   // m^(p-2)
        for (; e; e >>= 1) {
            r = (e & 1) ? umod(r * m, p, inv) : r;
            m = umod(m * m, p, inv);
        }
        crt = r;
    }
    __syncthreads();
    for (int f = 1; f < L; ++f) {
        const int z = umod(f * f, p, inv);
        int v = 0;
        if (tid <= f)
            v = umod((tid ? G[tid - 1] : 0) + (p - z) * G[tid], p, inv);
        __syncthreads();
        if (tid <= f)
            G[tid] = v;
        __syncthreads();
    }
    if (tid < L) {
        int d;
        if (tid == 0) {
            d = G[0];
        } else {
            const int z = umod(tid * tid, p, inv);
            int h = 1, val = 1;   // H_i from the top, and H_i(i^2) by Horner
            H[tid][L - 2] = 1;
            for (int k = L - 2; k >= 1; --k) {
                h = umod(G[k] + z * h, p, inv);
                H[tid][k - 1] = h;
                val = umod(val * z + h, p, inv);
            }
            d = umod(umod(2 * z, p, inv) * val, p, inv);
        }
        int e = p - 2, r = 1;
        for (; e; e >>= 1) {
            r = (e & 1) ? umod(r * d, p, inv) : r;
            d = umod(d * d, p, inv);
        }
        den[tid] = umod(r * crt, p, inv);
    }
    __syncthreads();
    // packed (res_packed): two primes to a 16 x 32 tile, the even one's rows
    // 0 .. 7 and columns 0 .. 15, the odd one's the others
    const bool packed = t.packed;
    const int half = packed ? i & 1 : 0;
    int8_t* W = t.W + (packed ? (int64_t)(i / 2) * 512 : (int64_t)i * t.Lp * t.Np);
    // an odd number of primes: the last one fills the missing one's half
    const int rows = packed ? (half == 0 && i + 1 == s.P ? 16 : 8) : t.Lp;
    for (int e = tid; e < rows * t.Np; e += 512) {
        const int tau = e / t.Np, j = e % t.Np - 16 * half;
        int v = 0;
        if (tau < L && j >= 0 && j < s.N) {
            const int xi = (j + 1) / 2;
            if (xi == 0) {
                v = (tau & 1) ? 0 : G[tau / 2];
            } else if (tau & 1) {
                v = tau / 2 <= L - 2 ? umod(((j & 1) ? xi : p - xi) * H[xi][tau / 2], p, inv) : 0;
            } else {
                v = tau ? H[xi][tau / 2 - 1] : 0;
            }
            v = centred(umod(v * den[xi], p, inv), p);
        }
        W[8 * half * t.Np + e] = (int8_t)v;
    }
}

// v - p rint(v / p) in the low byte, |v| < 2^22: the fused multiply-add
// rounds v / p to the integer in the low mantissa bits of 1.5 2^23 + q, and
// the 24-bit product takes those bits as 2^22 + q (p 2^22 is 0 mod 256)
__device__ __forceinline__ int residue_f32(int v, float inv, int negp)
{
    const float u = __builtin_fmaf((float)v, inv, 12582912.0f);
    return v + __mul24(__builtin_bit_cast(int, u), negp);
}

// the same for |v| < 2^30, in two steps: the first one's quotient may be off
// by the rounding of v to 24 bits and of 1 / p, which leaves a remainder
// below 2^10
__device__ __forceinline__ int residue_wide(int v, float inv, int negp)
{
    return residue_f32(residue_f32(v, inv, negp) + (1 << 22) * -negp, inv, negp);
}

// low bytes of four words
__device__ __forceinline__ uint32_t pack4(int a, int b, int c, int d)
{
    const uint32_t lo = __builtin_amdgcn_perm((uint32_t)b, (uint32_t)a, 0x0c0c0400u);
    const uint32_t hi = __builtin_amdgcn_perm((uint32_t)d, (uint32_t)c, 0x04000c0cu);
    return lo | hi;
}

// 4 x 4 bytes transposed
__device__ __forceinline__ void transpose4(uint32_t& a, uint32_t& b, uint32_t& c, uint32_t& d)
{
    const uint32_t t0 = __builtin_amdgcn_perm(b, a, 0x05010400u), t1 = __builtin_amdgcn_perm(b, a, 0x07030602u);
    const uint32_t t2 = __builtin_amdgcn_perm(d, c, 0x05010400u), t3 = __builtin_amdgcn_perm(d, c, 0x07030602u);
    a = __builtin_amdgcn_perm(t2, t0, 0x05040100u);
    b = __builtin_amdgcn_perm(t2, t0, 0x07060302u);
    c = __builtin_amdgcn_perm(t3, t1, 0x05040100u);
    d = __builtin_amdgcn_perm(t3, t1, 0x07060302u);
}

struct ResEvalArgs {
    const char* dig;      // digit planes, INT8 fragment order, from the panel's first row block
    char* out;            // residue planes of the panel
    const int8_t* V;
    const float2* pc;
    int64_t plane;        // bytes of one residue plane
    int nkc, nkr;         // 64-depth chunks of the digit planes and of the residue planes
    int SB, planes, KD;
};

// Digits of one row as evaluation operands: T[kt][e] holds digits 4 PL kt +
// PL q .. + PL - 1 of depth e, transposed from 16 depths of one digit at a
// time; digit(s) gives those (16 bytes), zeros from the last digit on.
template <int KT, class F>
__device__ __forceinline__ void res_operands(F&& digit, int q, uint32_t (&T)[KT ? KT : 1][16][KT ? 4 : 2])
{
    constexpr int KN = KT ? KT : 1, PL = KT ? 16 : 8;   // operands, digits per lane and operand
#pragma unroll
    for (int kt = 0; kt < KN; ++kt) {
        v4i D[PL];
#pragma unroll
        for (int i = 0; i < PL; ++i)
            D[i] = digit(4 * PL * kt + PL * q + i);
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int g = 0; g < PL / 4; ++g) {
                uint32_t w0 = D[4 * g][c], w1 = D[4 * g + 1][c], w2 = D[4 * g + 2][c], w3 = D[4 * g + 3][c];
                transpose4(w0, w1, w2, w3);
                T[kt][4 * c][g] = w0;
                T[kt][4 * c + 1][g] = w1;
                T[kt][4 * c + 2][g] = w2;
                T[kt][4 * c + 3][g] = w3;
            }
    }
}

// Residues of one 16 x 64 digit fragment (all planes).  The evaluation is a
// matrix product, weights [planes x digits] by digits [digits x entries]:
// wave w takes the 16 rows at depths 16 w .. 16 w + 15 of the fragment (lane
// n of a 16-byte group n holds row n), lane (q, n) the digits 16 q .. 16 q +
// 15 of its row, byte-transposed to one 16-digit operand per depth.  A lane
// then holds four planes of its row and depth, reduces them modulo p and
// stores 16 depths at once.  Residue planes keep the digits' fragment order
// (16 rows x 64 depths per 1 KB), their depth padded with zeros to an even
// number of chunks (the products take two at a time).
// KT: 64-digit operands (v_mfma_i32_16x16x64_i8); 0: up to 32 digits, eight
// per lane (v_mfma_i32_16x16x32_i8), half the loads, transposes and registers:
// four waves per SIMD instead of three (4096^2 entries, 27 digits to 164
// planes: 735 -> 628 us, 5.1 TB/s).
template <int KT>
__device__ __forceinline__ void res_planes(const uint32_t (&T)[KT ? KT : 1][16][KT ? 4 : 2], const int8_t* weights,
                                           const float2* pc, int KD, int planes, char* dst, int64_t plane, int n, int q)
{
    constexpr int KN = KT ? KT : 1, PL = KT ? 16 : 8;
    for (int t = 0; t < planes; t += 16) {
        const int8_t* V = weights + (int64_t)(t + n) * KD + PL * q;
        int64_t vh = 0;
        v4i vf[KN];
        if constexpr (KT == 0) {
            vh = *(const int64_t*)V;
        } else {
#pragma unroll
            for (int kt = 0; kt < KN; ++kt)
                vf[kt] = *(const v4i*)(V + 64 * kt);
        }
        float inv[4];
        int negp[4];
#pragma unroll
        for (int o = 0; o < 4; ++o) {
            const float2 c = pc[t + 4 * q + o];
            inv[o] = c.x;
            negp[o] = -(int)c.y;
        }
        v4i w[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            v4i acc[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                acc[e] = v4i{0, 0, 0, 0};
                if constexpr (KT == 0) {
                    const uint32_t* d = T[0][4 * g + e];
                    acc[e] = __builtin_amdgcn_mfma_i32_16x16x32_i8(vh, (int64_t)(((uint64_t)d[1] << 32) | d[0]), acc[e], 0,
                                                                   0, 0);
                } else {
#pragma unroll
                    for (int kt = 0; kt < KN; ++kt) {
                        const uint32_t* d = T[kt][4 * g + e];
                        acc[e] = __builtin_amdgcn_mfma_i32_16x16x64_i8(
                            vf[kt], v4i{(int)d[0], (int)d[1], (int)d[PL / 4 - 2], (int)d[PL / 4 - 1]}, acc[e], 0, 0, 0);
                    }
                }
            }
#pragma unroll
            for (int o = 0; o < 4; ++o)
                w[o][g] = (int)pack4(residue_f32(acc[0][o], inv[o], negp[o]), residue_f32(acc[1][o], inv[o], negp[o]),
                                     residue_f32(acc[2][o], inv[o], negp[o]), residue_f32(acc[3][o], inv[o], negp[o]));
        }
        // past the caches: a product's planes are far larger than they are
        // (hexa-doubles 1024^2, 671 planes: 253 -> 198 us an operand; octo-
        // doubles, 358: 96 -> 80; quad-doubles 4096^2: 1460 -> 1420 for both)
#pragma unroll
        for (int o = 0; o < 4; ++o)
            if (t + 4 * q + o < planes)
                __builtin_nontemporal_store(w[o], (v4i*)(dst + (int64_t)(t + 4 * q + o) * plane));
    }
}

template <int KT>
__global__ __launch_bounds__(256) void k_res_eval(ResEvalArgs a)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = lane & 15, q = lane >> 4;
    const int64_t rb = blockIdx.y;
    const int kc = blockIdx.x;
    const char* src = a.dig + (rb * a.nkc + kc) * ((int64_t)a.SB * 1024) + (wave * 16 + n) * 16;
    uint32_t T[KT ? KT : 1][16][KT ? 4 : 2];
    res_operands<KT>(
        [&](int s) { return s < a.SB && kc < a.nkc ? *(const v4i*)(src + (int64_t)s * 1024) : v4i{0, 0, 0, 0}; }, q, T);
    res_planes<KT>(T, a.V, a.pc, a.KD, a.planes, a.out + (rb * a.nkr + kc) * 1024 + (wave * 16 + n) * 16, a.plane, n, q);
}

constexpr int kCutF64 = 0, kCutSm = 1, kCutBal = 2;   // the digit forms

// One or both operands (z) of a product: words in, residue planes out.
struct ResCutArgs {
    SplitSide s[2];       // op from the panel's first row, E, nrb; out: residue planes
    const int8_t* V[2];
    int64_t plane[2];     // bytes of one residue plane
    const float2* pc;
    int64_t rb0;          // row block of blockIdx.y = 0
    int S, beta, nb, SB, planes, KD;
};

// The split and the evaluation of up to 32 digits of 1, 2 or 4 words in one
// kernel: a workgroup cuts the digits of one fragment (16 rows x 64 depths,
// four entries a thread, as the split kernels do: word placement for the
// INT8 forms, byte planes of the FP64 digits) into LDS in fragment order and
// evaluates them from there, so the digits are neither written to memory nor
// read back.  Bound by its stores (and the cut's integer instructions under
// them): 32 KB of LDS and 124 registers, four waves per SIMD.  Both operands,
// the split and two evaluations before against this kernel: 4096^2 quad-
// doubles, 164 planes, 1688 -> 1482 us (4.5 TB/s); 1000 x 1200 x 1100 in
// FP64 digits 163 -> 130; 2048^2 double-doubles in FP64 digits 237 -> 181.
// More digits or words stay with the split and k_res_eval: their LDS would
// leave one or two workgroups per compute unit.  FORM: kCut*.
template <int MW, int FORM>
__global__ __launch_bounds__(256) void k_res_cut(ResCutArgs a)
{
    constexpr int SC = 32;
    constexpr bool BAL = FORM == kCutBal;
    // the digits; before them, in the same place, the entries' limbs
    __shared__ __attribute__((aligned(16))) uint32_t dig[SC * 256];
    const int z = blockIdx.z, t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const SplitSide sd = z ? a.s[1] : a.s[0];
    const int64_t rb = a.rb0 + blockIdx.y;
    if (rb >= sd.nrb)
        return;   // the whole workgroup
    const Operand op = sd.op;
    const int kc = blockIdx.x;
    const int64_t r = rb * 16 + (t >> 2 & 15);
    const int64_t kbase = (int64_t)kc * kKcI8 + 16 * wave + 4 * (t & 3);
    const bool row_ok = r < op.R;
    const int Er = row_ok ? sd.E[r] : 0;
    double x[4][MW];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const bool ok = row_ok && kbase + q < op.K;
#pragma unroll
        for (int w = 0; w < MW; ++w)
            x[q][w] = ok ? op.p[w * op.ps + r * op.sr + (kbase + q) * op.sk] : 0.0;
    }
    if constexpr (FORM == kCutF64) {
        uint64_t mant[4][MW];
        int sh0[4][MW];
        bool neg[4][MW];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int w = 0; w < MW; ++w) {
                int ex;
                neg[q][w] = decode(x[q][w], mant[q][w], ex);
                sh0[q][w] = ex - Er;
            }
        const int D = 63 / a.beta, W = D * a.beta, nl = (a.S + D - 1) / D;
        const uint64_t wmask = (1ull << W) - 1, dmask = (1ull << a.beta) - 1;
        for (int j = 0; j < nl; ++j) {
            uint64_t P[4], N[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                limb_pair<MW>(mant[q], sh0[q], neg[q], W * (j + 1), wmask, P[q], N[q]);
            for (int i = 0; i < D && D * j + i < a.S; ++i) {
                const int rs = W - a.beta * (i + 1);
                uint32_t u[4];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    u[q] = (uint32_t)((int)((P[q] >> rs) & dmask) - (int)((N[q] >> rs) & dmask)) + 0x80808080u;
                for (int k = 0; k < a.nb; ++k) {
                    uint32_t packed = 0;
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        packed |= (((u[q] >> (8 * k)) & 0xffu) ^ 0x80u) << (8 * q);
                    dig[((D * j + i) * a.nb + k) * 256 + t] = packed;
                }
            }
        }
    } else {
        constexpr int bits = BAL ? 8 : 7, NS = store_limbs<SC, BAL>();
        static_assert(NS * 4 * 64 * 8 <= SC * 1024, "the limbs fit below the digits");
        const int kn = Er + 1075 - bits * a.S, pad = bits * (SC - a.S);
        LdsLimbs Ls{reinterpret_cast<uint64_t*>(dig) + wave * NS * 64 + lane};
#pragma unroll
        for (int i = 0; i < NS; ++i)
            Ls.col[i * 64] = 0;
        uint32_t xs[SC];
#pragma unroll
        for (int s = 0; s < SC; ++s)
            xs[s] = 0;
        unroll<4>([&](auto QQ) {
            constexpr int q = decltype(QQ)::value;
            if constexpr (BAL)
                digits_bal<q, MW, SC>(x[q], kn, pad, xs, Ls);
            else
                digits_sm<q, MW, SC>(x[q], kn, pad, xs, Ls);
        });
        __syncthreads();
#pragma unroll
        for (int s = 0; s < SC; ++s)
            if (s < a.S)
                dig[s * 256 + t] = BAL ? xs[s] ^ 0x80808080u : xs[s];
    }
    __syncthreads();
    const int n = lane & 15, q = lane >> 4;
    const uint32_t* src = dig + (wave * 16 + n) * 4;
    uint32_t T[1][16][2];
    res_operands<0>([&](int s) { return s < a.SB ? *(const v4i*)(src + s * 256) : v4i{0, 0, 0, 0}; }, q, T);
    res_planes<0>(T, z ? a.V[1] : a.V[0], a.pc, a.KD, a.planes,
                  (char*)sd.out + (rb * gridDim.x + kc) * 1024 + (wave * 16 + n) * 16, z ? a.plane[1] : a.plane[0], n, q);
}

template <int MW>
hipError_t launch_res_cut(const ResCutArgs& a, int form, dim3 grid, hipStream_t st)
{
    switch (form) {
    case kCutF64: hipLaunchKernelGGL((k_res_cut<MW, kCutF64>), grid, dim3(256), 0, st, a); break;
    case kCutSm: hipLaunchKernelGGL((k_res_cut<MW, kCutSm>), grid, dim3(256), 0, st, a); break;
    default: hipLaunchKernelGGL((k_res_cut<MW, kCutBal>), grid, dim3(256), 0, st, a); break;
    }
    return hipGetLastError();
}

struct ResGemmArgs {
    const char *A, *B;     // residue planes of the panel
    char* R;               // residues of the products: [point][16 x 16 block][64 dwords]
    int32_t* Rb;           // the last diagonal's sums: [unit][16 x 16 block][64 lanes][4]
    int64_t psA, psB, psR; // bytes of a plane
    int nbA, nbB;          // 16-row blocks
    int gx, gy, nkc;       // nkc: 64-depth steps, even
    int N, npp, nbd, bq, nchunk;
    int p[kResMaxPrimes];
};

// s_waitcnt with lgkmcnt and expcnt at their maxima and vmcnt = N
template <int N>
__device__ __forceinline__ void res_wait_vm()
{
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (0x7 << 4) | (0xf << 8));
}

__device__ __forceinline__ void res_barrier() { asm volatile("s_barrier" ::: "memory"); }

// Tile id -> (unit, tile).  The units of the last diagonal (up to bq products
// each) come first, so that the long ones do not end the launch.  Ids go
// round-robin over the 8 XCDs (workgroups are dispatched that way, and the
// number of workgroups is a multiple of 8).  From 64 tiles a plane, every XCD
// takes an eighth of each unit's tiles, a compact block whose panels it
// shares in its L2; below that whole units go to XCDs in turn, so that a
// plane is read by one L2.
__device__ __forceinline__ void res_tile(const ResGemmArgs& a, int id, int& unit, int& ty, int& tx)
{
    const int T = a.gx * a.gy, units = a.npp + a.nchunk;
    int l;
    if (T % 8 == 0 && T >= 64) {
        unit = id / T;
        l = id % T;
        l = (l % 8) * (T / 8) + l / 8;
    } else if (id < units / 8 * 8 * T) {
        unit = (id / 8) / T * 8 + id % 8;
        l = (id / 8) % T;
    } else {
        unit = id / T;
        l = id % T;
    }
    const int per = 4 * a.gx, g = l / per, r = l % per, rows = min(4, a.gy - g * 4);
    ty = g * 4 + r % rows;
    tx = r / rows;
}

// acc += a b with the accumulator kept in accumulation registers, in place
// (the compiler, given the builtin in this loop, keeps some accumulators in
// vector registers and moves them back and forth, one move per matrix
// instruction).  Its sources come from LDS reads, whose waits the compiler
// places; consecutive instructions take different accumulators.  What it
// does not see are the wait states between these and other instructions on
// the accumulators: res_settle() stands before the first and after the last.
__device__ __forceinline__ void res_mfma(v4i& acc, const v4i& a, const v4i& b)
{
    asm volatile("v_mfma_i32_16x16x64_i8 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}

__device__ __forceinline__ void res_pin(v4i (&acc)[8][8])
{
#pragma unroll
    for (int x = 0; x < 8; ++x)
#pragma unroll
        for (int y = 0; y < 8; ++y)
            asm volatile("" : "+a"(acc[x][y]));
}

__device__ __forceinline__ void res_settle(v4i (&acc)[8][8])
{
    res_pin(acc);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    res_pin(acc);
}

// An accumulator into vector registers, here and not earlier (left to the
// compiler, the copies of many gather before the reduction and spill)
__device__ __forceinline__ v4i res_read(const v4i& acc)
{
    v4i v;
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v[0]) : "a"(acc[0]));
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v[1]) : "a"(acc[1]));
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v[2]) : "a"(acc[2]));
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v[3]) : "a"(acc[3]));
    return v;
}

// What a wave loads of a tile: row blocks 4 w .. 4 w + 3 of its sixteen on
// both sides (clamped to the last one: those outputs are not stored).
struct ResLoads {
    const char *pA, *pB;
    int oA[4], oB[4], steps;
    __device__ __forceinline__ ResLoads(const ResGemmArgs& a, int unit, int ty, int tx, int wave)
    {
        const bool bnd = unit < a.nchunk;
        const int pl0 = bnd ? a.npp + unit * a.bq : unit - a.nchunk;
        steps = (bnd ? min(a.bq, a.nbd - unit * a.bq) : 1) * a.nkc;
        const int bytes = a.nkc * 1024;   // one row block's depth
        const int fA = min(ty * 16 + wave * 4, a.nbA - 1), fB = min(tx * 16 + wave * 4, a.nbB - 1);
        pA = a.A + pl0 * a.psA + (int64_t)fA * bytes;
        pB = a.B + pl0 * a.psB + (int64_t)fB * bytes;
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            oA[f] = min(f, a.nbA - 1 - fA) * bytes;
            oB[f] = min(f, a.nbB - 1 - fB) * bytes;
        }
    }
};

// 256 x 256 tiles of the units, one workgroup per compute unit taking every
// gridDim-th: a product of residue planes reduced modulo its prime to one
// byte per output, or the sum of up to bq products of the last diagonal.
// Four waves of 128 x 128 outputs (8 x 8 accumulators of
// v_mfma_i32_16x16x64_i8, 256 registers); per 64 depths the workgroup's 16 +
// 16 fragments go straight into one of four LDS slots (each wave issues
// eight loads, three steps ahead, across tiles: the loads of a tile's first
// steps are under way while the tile before it is reduced and stored), and
// each wave reads its 8 + 8 fragments one step ahead of their use.  At the
// top of step k the wave's own loads of step k + 1 are done (the 8 of step k
// + 2 may be open), and the barrier makes everyone's visible; the slot
// written then, (k + 3) mod 4, was last read for step k - 1, whose matrix
// instructions every wave has issued before that barrier.  A tile's first
// two steps follow the stores of the tile before it (64, after their loads),
// so an open count of 63 there already means that the loads are done.
//
// What bounds it: a step's 64 matrix instructions are 1024 cycles; with the
// loads left out it runs at 92% of the matrix cores' peak on zeros, with
// them at 72% (a load instruction issued among matrix instructions holds the
// wave less than eight in a row: 3.55 against 3.30 POP/s on zeros), and on
// residues the clock falls with the power drawn (4096^3, 164 planes: 64% of
// the cycles at 1.75 GHz, 9.3 to 9.8 ms, 2.3 to 2.4 POP/s).
// v_mfma_i32_32x32x32_i8 on the same tile was 10% slower on residues.  No
// change from every tile reading one panel, a fifth LDS slot, B straight to
// registers, the row blocks of a depth step side by side in memory, or
// stores past the caches.
// WIDE: sums that one rounding of the quotient in single precision could
// leave outside a byte (see launch_resid).
template <bool WIDE>
__global__ __launch_bounds__(256, 1) void k_res_gemm(ResGemmArgs a)
{
    __shared__ __attribute__((aligned(16))) char lds[4 * 32768];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int total = a.gx * a.gy * (a.npp + a.nchunk);
    const int nkc = a.nkc;
    int id = blockIdx.x, unit, ty, tx;
    res_tile(a, id, unit, ty, tx);
    ResLoads cur(a, unit, ty, tx, wave), nxt = cur;   // nxt: the tile after the one being loaded
    const int voff = lane * 16;
    int ik = 0, left = cur.steps;   // depth step of the next issue, issues left of its tile
    int ws = 0, rs = 0;             // LDS slot written next, slot of the current step
    auto issue_one = [&](int f) {
        if (f < 4) {
            const __amdgpu_buffer_rsrc_t d =
                __builtin_amdgcn_make_buffer_rsrc((void*)cur.pA, 0, cur.oA[3] + nkc * 1024, 0x00020000);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                d, (__attribute__((address_space(3))) void*)(lds + ws * 32768 + wave * 4096 + f * 1024), 16, voff,
                ik * 1024 + cur.oA[f], 0, 0);
        } else {
            const __amdgpu_buffer_rsrc_t d =
                __builtin_amdgcn_make_buffer_rsrc((void*)cur.pB, 0, cur.oB[3] + nkc * 1024, 0x00020000);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                d, (__attribute__((address_space(3))) void*)(lds + ws * 32768 + 16384 + wave * 4096 + (f - 4) * 1024), 16,
                voff, ik * 1024 + cur.oB[f - 4], 0, 0);
        }
    };
    // to the next depth step: of the same product, of the next product of the
    // unit, or of the next tile (selects, not branches: a step stays one
    // basic block)
    auto advance = [&] {
        --left;
        ++ik;
        const bool wrap = ik == nkc, sw = left == 0;
        ik = wrap ? 0 : ik;
        cur.pA = sw ? nxt.pA : cur.pA + (wrap ? a.psA : 0);
        cur.pB = sw ? nxt.pB : cur.pB + (wrap ? a.psB : 0);
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            cur.oA[f] = sw ? nxt.oA[f] : cur.oA[f];
            cur.oB[f] = sw ? nxt.oB[f] : cur.oB[f];
        }
        left = sw ? nxt.steps : left;
        ws = (ws + 1) & 3;
    };
    const char* la = lds + (wave >> 1) * 8192 + lane * 16;
    const char* lb = lds + 16384 + (wave & 1) * 8192 + lane * 16;
    v4i acc[8][8], fa[2][8], fb[2][8];
#pragma unroll
    for (int s = 0; s < 3; ++s) {   // a tile has at least four steps
#pragma unroll
        for (int f = 0; f < 8; ++f)
            issue_one(f);
        advance();
    }
    res_wait_vm<0>();
    res_barrier();
#pragma unroll
    for (int f = 0; f < 8; ++f) {
        fa[0][f] = *(const v4i*)(la + f * 1024);
        fb[0][f] = *(const v4i*)(lb + f * 1024);
    }
    auto step = [&](auto PP, auto WW) {
        constexpr int P = decltype(PP)::value;   // register buffer of this step
        res_wait_vm<decltype(WW)::value>();
        res_barrier();
        __builtin_amdgcn_sched_barrier(0);
        const int so = ((rs + 1) & 3) * 32768;
#pragma unroll
        for (int x = 0; x < 8; ++x)
#pragma unroll
            for (int y = 0; y < 8; ++y) {
                res_mfma(acc[x][y], fa[P][x], fb[P][y]);
                // between matrix instructions: a fragment read of the next
                // step on either side of one load
                if (y == 1 || y == 3 || y == 6) {
                    __builtin_amdgcn_sched_barrier(0);
                    if (y == 1)
                        fa[P ^ 1][x] = *(const v4i*)(la + so + x * 1024);
                    if (y == 3)
                        issue_one(x);
                    if (y == 6)
                        fb[P ^ 1][x] = *(const v4i*)(lb + so + x * 1024);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        __builtin_amdgcn_sched_barrier(0);
        advance();
        rs = (rs + 1) & 3;
    };
    using std::integral_constant;
    for (;;) {
        // this tile's outputs, and the loads of the one after it (a
        // workgroup's last tile is followed by unused loads of its own)
        const bool bnd = unit < a.nchunk;
        const int u0 = unit, pl0 = bnd ? 0 : unit - a.nchunk;
        const int steps = (bnd ? min(a.bq, a.nbd - unit * a.bq) : 1) * nkc;
        const int rA = ty * 16 + (wave >> 1) * 8, rB = tx * 16 + (wave & 1) * 8;
        const bool more = id + (int)gridDim.x < total;
        id += more ? (int)gridDim.x : 0;
        res_tile(a, id, unit, ty, tx);
        nxt = ResLoads(a, unit, ty, tx, wave);
#pragma unroll
        for (int x = 0; x < 8; ++x)
#pragma unroll
            for (int y = 0; y < 8; ++y)
                acc[x][y] = v4i{0, 0, 0, 0};
        res_settle(acc);
        step(integral_constant<int, 0>{}, integral_constant<int, 63>{});
        step(integral_constant<int, 1>{}, integral_constant<int, 63>{});
        for (int k = 2; k < steps; k += 2) {   // an even number: nkc is even
            step(integral_constant<int, 0>{}, integral_constant<int, 8>{});
            step(integral_constant<int, 1>{}, integral_constant<int, 8>{});
        }
        res_settle(acc);

        // accumulator element o of lane l: row 4 (l / 16) + o, column l % 16.
        // Blocks past the padded rows or columns store to an offset outside
        // the descriptor, which drops them.
        const int nx = a.nbA - rA, ny = a.nbB - rB;   // blocks to store
        const int64_t blk = (int64_t)rA * a.nbB + rB;
        constexpr uint32_t kNone = 0x7fffff00u;
        if (bnd) {
            const __amdgpu_buffer_rsrc_t d = __builtin_amdgcn_make_buffer_rsrc(
                a.Rb + ((int64_t)u0 * a.nbA * a.nbB + blk) * 256, 0, kNone, 0x00020000);
#pragma unroll
            for (int x = 0; x < 8; ++x) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int y = 0; y < 8; ++y)
                    __builtin_amdgcn_raw_buffer_store_b128(res_read(acc[x][y]), d, lane * 16,
                                                           x < nx && y < ny ? (x * a.nbB + y) * 1024 : kNone, 0);
            }
        } else {
            const int p = a.p[pl0 / a.N];
            const float inv = 1.0f / (float)p;
            const __amdgpu_buffer_rsrc_t d = __builtin_amdgcn_make_buffer_rsrc(
                a.R + (int64_t)pl0 * a.psR + blk * 256, 0, kNone, 0x00020000);
#pragma unroll
            for (int x = 0; x < 8; ++x) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int y = 0; y < 8; ++y) {
                    const v4i v = res_read(acc[x][y]);
                    int r[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        r[e] = WIDE ? residue_wide(v[e], inv, -p) : residue_f32(v[e], inv, -p);
                    __builtin_amdgcn_raw_buffer_store_b32(pack4(r[0], r[1], r[2], r[3]), d, lane * 4,
                                                          x < nx && y < ny ? (x * a.nbB + y) * 256 : kNone, 0);
                }
            }
        }
        if (!more)
            break;
    }
    res_wait_vm<0>();   // every load issued has landed before the workgroup ends
}

// low bits of the Chinese remainder's factors (M / p < 2^56)
constexpr int kResSplit = 27;

// a + b over the wave's two halves: lanes 0 .. 31 get a(l) + a(l + 32), lanes
// 32 .. 63 b(l - 32) + b(l)
__device__ __forceinline__ double add_halves(double a, double b)
{
    const uint64_t ua = __builtin_bit_cast(uint64_t, a), ub = __builtin_bit_cast(uint64_t, b);
    const auto l = __builtin_amdgcn_permlane32_swap((uint32_t)ua, (uint32_t)ub, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap((uint32_t)(ua >> 32), (uint32_t)(ub >> 32), false, false);
    return __builtin_bit_cast(double, ((uint64_t)h[0] << 32) | l[0]) +
           __builtin_bit_cast(double, ((uint64_t)h[1] << 32) | l[1]);
}

struct ResFinalArgs {
    const char* R;
    const int32_t* Rb;
    const int8_t* W;
    int64_t psR;
    int nbA, nbB;
    int L, N, P, Lp, Np, w, nchunk;
    double Wh[kResMaxPrimes], Wl[kResMaxPrimes];   // M / p = Wh 2^kResSplit + Wl
    double Mh, Ml, invM;
    int64_t r0, c0;        // first row and column of the panel
    GemmArgs g;
};

// Interpolation, Chinese remainder, fold and rounding.  A workgroup takes a
// 16 x 16 block of outputs, a wave 4 rows of it (64 outputs).  The
// interpolation is a matrix product, weights [coefficients x points] by
// residues [points x outputs] on 32 points at a time (lane (q, n): points
// 8 q .. 8 q + 7 of column n, four rows, byte-transposed to one operand per
// row; the next 32 points are in flight meanwhile), 16 NT coefficients at
// once.  The remainder needs no reduction modulo p before it: with |v| <
// 2^21 the sums of v (M / p) in two doubles stay exact (v Wh < 2^49, v Wl <
// 2^48, at most 8 of each), and taking M off rint(sum / M) times leaves the
// coefficient.  The coefficients come from the last one down (the least
// significant), pass 16 at a time through LDS to the lane that folds their
// output, and enter a signed 96-bit window whose low 32 bits leave as limbs;
// then the limbs are rounded (as k_gemm_final's).
// PK (L <= 8): two primes at a time, one on the weights' rows 0 .. 7 and
// points 0 .. 15 (lanes q = 0, 1), the other on the rest (q = 2, 3); the two
// halves' sums meet at the end, each half of the wave keeping every other
// row (double-doubles 2048^3, 8 primes of 9 points: a step of three products
// 3216 -> 3050 us).
// Waves per SIMD: four, three where the LDS (32 KB and one per limb) holds
// no more, two with two tiles' registers.
template <int NL, int NT, bool FIX, bool PK>
__global__ __launch_bounds__(256, NT == 2 ? 2 : NL <= 8 ? 4 : 3) void k_res_final(ResFinalArgs a)
{
    __shared__ int64_t coef[4][16][64];
    __shared__ uint32_t limb[4][NL][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, q = lane >> 4;
    const int64_t blk = blockIdx.x;
    const int64_t dw = blk * 64 + wave * 16 + n;   // dword of this column's four rows

    const int e = q;                                // row of this lane's output
    // the window on the folded integer, from bit 32 k up: wl + 2^32 wh
    int64_t wh = 0;
    {
        const int32_t* rb = a.Rb + dw * 4 + e;
        const int64_t stride = (int64_t)a.nbA * a.nbB * 256;
        for (int c = 0; c < a.nchunk; c += 4) {   // four loads in flight
            int32_t v[4];
#pragma unroll
            for (int x = 0; x < 4; ++x)
                v[x] = rb[min(c + x, a.nchunk - 1) * stride];
#pragma unroll
            for (int x = 0; x < 4; ++x)
                wh += c + x < a.nchunk ? v[x] : 0;
        }
    }
    uint32_t wl = (uint32_t)wh;
    wh >>= 32;
    int bit = 0, k = 0;                             // position of the next coefficient, limbs done
    const int nj = PK ? 1 : a.Np / 32, its = PK ? (a.P + 1) / 2 : a.P * nj;
    const int half = PK ? q >> 1 : 0;   // the prime of this lane's points and coefficients
    // (32-bit offsets: below 32 planes.)  Points past a prime's last one weigh
    // zero: they read the next prime's
    // plane, or past the last prime zeros (out of the descriptor's range)
    uint32_t voff[8], nx[8];
#pragma unroll
    for (int j = 0; j < 8; ++j)
        voff[j] = (uint32_t)(((PK ? half * a.N + 8 * (q & 1) : 8 * q) + j) * a.psR + wave * 64 + n * 4);
    auto load = [&](int i, int j0) {
        const int64_t pt = (int64_t)(PK ? 2 * i : i) * a.N + j0;
        const int64_t left = ((int64_t)a.P * a.N - pt) * a.psR - blk * 256;
        const __amdgpu_buffer_rsrc_t d = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<char*>(a.R) + pt * a.psR + blk * 256, 0, (int)min(left, (int64_t)0xffffff00), 0x00020000);
#pragma unroll
        for (int j = 0; j < 8; ++j)
            nx[j] = __builtin_amdgcn_raw_buffer_load_b32(d, voff[j], 0, 0);
    };
    load(0, 0);
    for (int t0 = (a.L - 1) / (16 * NT) * (16 * NT); t0 >= 0; t0 -= 16 * NT) {
        double hi[NT][16], lo[NT][16];
#pragma unroll
        for (int x = 0; x < NT; ++x)
#pragma unroll
            for (int y = 0; y < 16; ++y)
                hi[x][y] = lo[x][y] = 0.0;
        v4i acc[NT][4];
        for (int it = 0, i = 0, jb = 0; it < its; ++it) {
            uint32_t d[8];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                d[j] = nx[j];
            int64_t wf[NT];
#pragma unroll
            for (int x = 0; x < NT; ++x)   // rows past Lp: the last tile again (not kept)
                wf[x] = *(const int64_t*)(a.W + (uint32_t)((i * a.Lp + min(t0 + 16 * x, a.Lp - 16) + n) * a.Np + jb * 32 +
                                                           8 * q));   // PK: Lp = 16, Np = 32
            const int i0 = i;
            const bool first = jb == 0, last = jb + 1 == nj;
            jb = last ? 0 : jb + 1;
            i = last ? (i + 1 == (PK ? its : a.P) ? 0 : i + 1) : i;
            load(i, jb * 32);
            transpose4(d[0], d[1], d[2], d[3]);
            transpose4(d[4], d[5], d[6], d[7]);
#pragma unroll
            for (int x = 0; x < NT; ++x)
#pragma unroll
                for (int y = 0; y < 4; ++y) {
                    const int64_t df = (int64_t)(((uint64_t)d[4 + y] << 32) | d[y]);
                    if (first)
                        acc[x][y] = __builtin_amdgcn_mfma_i32_16x16x32_i8(wf[x], df, v4i{0, 0, 0, 0}, 0, 0, 0);
                    else
                        acc[x][y] = __builtin_amdgcn_mfma_i32_16x16x32_i8(wf[x], df, acc[x][y], 0, 0, 0);
                }
            if (last) {
                const double Wh = PK ? (half ? a.Wh[2 * i0 + 1] : a.Wh[2 * i0]) : a.Wh[i0];
                const double Wl = PK ? (half ? a.Wl[2 * i0 + 1] : a.Wl[2 * i0]) : a.Wl[i0];
#pragma unroll
                for (int x = 0; x < NT; ++x)
#pragma unroll
                    for (int y = 0; y < 4; ++y)
#pragma unroll
                        for (int o = 0; o < 4; ++o) {
                            const double v = (double)acc[x][y][o];
                            hi[x][4 * y + o] = __builtin_fma(v, Wh, hi[x][4 * y + o]);
                            lo[x][4 * y + o] = __builtin_fma(v, Wl, lo[x][4 * y + o]);
                        }
            }
        }
        if constexpr (PK) {
            // rows 2 y and 2 y + 1: lanes 0 .. 31 end with both halves' sum
            // of row 2 y, lanes 32 .. 63 of row 2 y + 1
#pragma unroll
            for (int y = 0; y < 2; ++y)
#pragma unroll
                for (int o = 0; o < 4; ++o) {
                    hi[0][4 * y + o] = add_halves(hi[0][8 * y + o], hi[0][8 * y + 4 + o]);
                    lo[0][4 * y + o] = add_halves(lo[0][8 * y + o], lo[0][8 * y + 4 + o]);
                }
        }
#pragma unroll
        for (int x = NT - 1; x >= 0; --x) {
#pragma unroll
            for (int y = 0; y < (PK ? 2 : 4); ++y)
#pragma unroll
                for (int o = 0; o < 4; ++o) {
                    constexpr double kMagic = 6755399441055744.0;   // 1.5 2^52
                    constexpr double kSplit = (double)(1 << kResSplit);
                    const double h = hi[x][4 * y + o], z = lo[x][4 * y + o];
                    const double kq = __builtin_rint(__builtin_fma(h, kSplit, z) * a.invM);
                    const double hr = __builtin_fma(-kq, a.Mh, h) + kMagic, zr = __builtin_fma(-kq, a.Ml, z) + kMagic;
                    const int64_t bits = __builtin_bit_cast(int64_t, kMagic);
                    coef[wave][PK ? 4 * (q & 1) + o : 4 * q + o][(PK ? 2 * y + half : y) * 16 + n] =
                        (int64_t)((uint64_t)(__builtin_bit_cast(int64_t, hr) - bits) << kResSplit) +
                        (__builtin_bit_cast(int64_t, zr) - bits);
                }
            // the wave's own LDS writes, then its reads (other lanes')
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            for (int t = min(16, a.L - t0 - 16 * x) - 1; t >= 0; --t) {
                // a block is at most 24 bits wide: at most one limb leaves per step
                if (bit >= 32) {
                    limb[wave][k++][lane] = wl;
                    wl = (uint32_t)wh;
                    wh >>= 32;
                    bit -= 32;
                }
                const int64_t v = coef[wave][t][lane];   // below 2^62: wh holds its upper part
                const uint64_t lo = (uint64_t)wl + ((uint32_t)v << bit);
                wl = (uint32_t)lo;
                wh += (v >> (32 - bit)) + (int64_t)(lo >> 32);
                bit += a.w;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    }
    for (; k < NL; ++k) {
        limb[wave][k][lane] = wl;
        wl = (uint32_t)wh;
        wh >>= 32;
    }
    uint32_t L[NL];
#pragma unroll
    for (int x = 0; x < NL; ++x)
        L[x] = limb[wave][x][lane];

    const GemmArgs& ga = a.g;
    const int64_t bi = blk / a.nbB, bj = blk % a.nbB;
    const int64_t i = a.r0 + bi * 16 + 4 * wave + e, j = a.c0 + bj * 16 + n;
    const bool ok = i < ga.M && j < ga.N;
    const int scale0 = ok ? ga.E[i] + ga.F[j] - ga.beta * (ga.S + 1) : 0;
    if constexpr (FIX) {
        if (!ok)
            return;
        const int64_t count = ga.M * ga.N, at = i * ga.N + j;
        for (int x = 0; x < ga.fixNL; ++x)
            ga.fixX[(int64_t)x * count + at] = x < NL ? (int32_t)limb[wave][x][lane] : (wh < 0 ? -1 : 0);
        ga.fixScale[at] = scale0;
        return;
    }
    int32_t sg = wh < 0 ? -1 : 0;
    int scale = scale0;
    double* out = ga.C + (ok ? i * ga.ldc + j : 0);
    for (int x = 0; x < ga.m; ++x) {
        const double wv = rn_signed(L, sg, scale);
        if (ok)
            out[x * ga.psc] = wv;
    }
}

template <int NL>
hipError_t launch_res_final(const ResFinalArgs& a, bool packed, hipStream_t st)
{
    const dim3 blocks((unsigned)((int64_t)a.nbA * a.nbB));
    if constexpr (NL <= 8)
        if (packed) {
            if (a.g.fixX)
                hipLaunchKernelGGL((k_res_final<NL, 1, true, true>), blocks, dim3(256), 0, st, a);
            else
                hipLaunchKernelGGL((k_res_final<NL, 1, false, true>), blocks, dim3(256), 0, st, a);
            return hipGetLastError();
        }
    if (packed)   // L <= 8 coefficients of at most 24 bits fold into 8 limbs
        return hipErrorInvalidValue;
    // two tiles of 16 coefficients at once (four, for L > 32, leave one wave
    // per SIMD: 549 -> 761 us at hexa-double 1024^3)
    if (a.L > 16) {
        if (a.g.fixX)
            hipLaunchKernelGGL((k_res_final<NL, 2, true, false>), blocks, dim3(256), 0, st, a);
        else
            hipLaunchKernelGGL((k_res_final<NL, 2, false, false>), blocks, dim3(256), 0, st, a);
        return hipGetLastError();
    }
    if constexpr (NL <= 16) {   // up to 16 coefficients of at most 24 bits fold into 14 limbs
        if (a.g.fixX)
            hipLaunchKernelGGL((k_res_final<NL, 1, true, false>), blocks, dim3(256), 0, st, a);
        else
            hipLaunchKernelGGL((k_res_final<NL, 1, false, false>), blocks, dim3(256), 0, st, a);
        return hipGetLastError();
    }
    return hipErrorInvalidValue;
}

// limbs that hold |X| < K 2^(beta (S + 1) + 1) and its sign, rounded up to
// an instantiated count
hipError_t dispatch_res_final(const ResFinalArgs& a, int nl, bool packed, hipStream_t st)
{
    if (nl <= 4) return launch_res_final<4>(a, packed, st);
    if (nl <= 6) return launch_res_final<6>(a, packed, st);
    if (nl <= 8) return launch_res_final<8>(a, packed, st);
    if (nl <= 10) return launch_res_final<10>(a, packed, st);
    if (nl <= 12) return launch_res_final<12>(a, packed, st);
    if (nl <= 16) return launch_res_final<16>(a, packed, st);
    if (nl <= 20) return launch_res_final<20>(a, packed, st);
    if (nl <= 24) return launch_res_final<24>(a, packed, st);
    if (nl <= 28) return launch_res_final<28>(a, packed, st);
    if (nl <= 32) return launch_res_final<32>(a, packed, st);
    return hipErrorInvalidValue;
}

// Few coefficients (L <= 8, so N <= 15 points): two primes share a tile of
// the interpolation.
bool res_packed(const ResPlan& r) { return r.L <= 8; }

// scratch layout of one panel
struct ResLayout {
    int64_t psA, psB, psR, nbA, nbB;
    size_t A, B, R, Rb, total;
    ResTables t;
};

void res_layout(const ResPlan& r, int64_t mr, int64_t nc, int nchunk, int64_t K, char* base, ResLayout& l)
{
    const int64_t Kp = res_steps(K) * kKcI8;
    l.nbA = (mr + 15) / 16;
    l.nbB = (nc + 15) / 16;
    l.psA = l.nbA * 16 * Kp;
    l.psB = l.nbB * 16 * Kp;
    // the interpolation reads every point's plane at the same place: an odd
    // number of 256-byte steps between planes spreads those reads over the
    // memory channels (4096^2 outputs, 150 planes of 2^24 bytes: 1035 -> 945 us)
    l.psR = l.nbA * l.nbB * 256 + 1280;
    l.t.KD = 64 * r.kt();
    l.t.pl16 = (r.planes() + 15) / 16 * 16;
    l.t.Lp = (r.L + 15) / 16 * 16;
    l.t.Np = (r.N + 31) / 32 * 32;
    l.t.packed = res_packed(r);
    size_t at = 0;
    auto take = [&](size_t n) {
        const size_t o = at;
        at += up256(n);
        return o;
    };
    const size_t va = take((size_t)l.t.pl16 * l.t.KD), vb = take((size_t)l.t.pl16 * l.t.KD);
    const size_t w = take((size_t)r.P * l.t.Lp * l.t.Np), pc = take((size_t)l.t.pl16 * sizeof(float2));
    l.A = take((size_t)l.psA * r.planes());
    l.B = take((size_t)l.psB * r.planes());
    l.R = take((size_t)l.psR * r.npp());
    l.Rb = take((size_t)l.psR * 4 * nchunk);
    l.total = at;
    l.t.VA = (int8_t*)(base + va);
    l.t.VB = (int8_t*)(base + vb);
    l.t.W = (int8_t*)(base + w);
    l.t.pc = (float2*)(base + pc);
}

}  // namespace

int res_limbs(const ResPlan& r, int64_t K)
{
    int lg = 0;
    while ((INT64_C(1) << lg) < K)
        ++lg;
    return (r.beta * (r.S + 1) + 1 + lg + 1 + 31) / 32;
}

int res_f64_bytes(int beta) { return beta <= 14 ? 2 : (beta <= 22 ? 3 : 4); }

bool res_plan(bool balanced, bool fp64, int S, int beta, int64_t K, ResPlan& r)
{
    // INT32 sums of residue products (125^2 each) and of one product of the
    // last diagonal (128^2) stay exact; 32-bit offsets within a row panel
    if (K < 1 || K > 65536 || S < 3 || (!fp64 && (beta != 7 && beta != 8)) || (fp64 && (beta < 1 || beta > 24)))
        return false;
    r = ResPlan();
    r.S = S;
    r.beta = beta;
    const int64_t Kp = round_up64(K, kKcI8);   // padded depths hold zeros
    double blk;   // largest block magnitude
    if (fp64) {
        r.L = S;
        r.w = beta;
        r.nb = res_f64_bytes(beta);
        r.SB = r.nb * S;
        blk = (double)((1 << beta) - 1);
    } else {
        r.L = S % 2 ? (S - 1) / 2 : S / 2;
        r.w = 2 * beta;
        r.SB = S;
        r.nbd = S % 2 ? r.L + 1 : r.L;
        blk = balanced ? 128.0 * 257.0 : 127.0 * 129.0;
        const int64_t fit = ((INT64_C(1) << 31) - 1) / (Kp * 128 * 128);   // products per exact INT32 sum
        r.bfit = (int)std::max<int64_t>(1, std::min<int64_t>(fit, 8));
    }
    r.N = 2 * r.L - 1;
    // points 0, +-1 .. +-(L-1) distinct modulo every prime; the table kernel
    // holds L <= 96 and the evaluation three operands of 64 digits
    if (r.L < 2 || r.L > 64 || r.SB > 192 || res_limbs(r, Kp) > 32)
        return false;
    // the product of the primes exceeds twice the largest coefficient, with
    // a margin for the quotient's rounding
    const double need = 2.0 * r.L * (double)Kp * blk * blk * (1.0 + 1e-6);
    double M = 1.0;
    while (r.P < kResMaxPrimes && M <= need)
        M *= kPrimes[r.P++];
    return M > need;
}

// Expected microseconds of the residue contraction and of the slice products
// for one product, and the line between them.  Fitted to both paths' times
// on one MI355X over m = 1 .. 16, the three forms, cubes from 64 to 3072 and
// up to nine oblong sizes from 64 x 64 x 4096 to 1024 x 1024 x 128 (the
// residues within 11%, 16% once).
//
// Residues: 256 x 256 tiles of all planes in rounds of one per compute unit,
// 0.85 us per 64 depths and 5 to 7 us of reduction each; cutting and
// evaluating up to 32 digits 5.3e6 bytes of words and residues per us,
// evaluating more 4.5e6 residues per us; the interpolation and the rounding;
// fixed costs that grow with the planes (the evaluation's loop over them is
// serial).  Slice products: the INT8 kernels' 64 x 32 tiles in rounds,
// S (S+1) matrix instructions per 64 depths; the FP64 kernel at 62 TFLOP/s,
// or a tile's serial depth where tiles are few.
//
// So (slices against residues, us) FP64 digits change over below 384^3
// doubles and double-doubles (57 against 47 and 93 against 65) and below
// 128^3 quad-doubles (115 against 90); INT8 octo-doubles at about 256^3 (52
// balanced digits: 143 against 133; 192^3: 115 against 127), hexa-doubles
// below 96^3 (368 against 240), quad-doubles between 1536^3 (27 balanced
// digits: 952 against 921) and 2048^3 (1989 against 1825), double-doubles
// never.
bool res_pays(const ResPlan& r, int64_t M, int64_t N, int64_t K, bool duo, double tri_us)
{
    const double dM = (double)M, dN = (double)N, dK = (double)K, dS = r.S;
    const double steps = (double)res_steps(K), planes = r.planes();
    const double T = std::ceil(dM / 256) * std::ceil(dN / 256);
    const double words = r.beta * r.S / 53.0;
    const double rounds = std::ceil(T * planes / kResGroups);
    const double residues =
        r.SB <= 32 ? 25 + 0.07 * planes + rounds * (steps * 0.85 + 6.7) +
                         (dM + dN) * steps * 64 * (planes + 8 * words) / 5.3e6 +
                         dM * dN * 1e-6 * (21 + 0.45 * words * res_limbs(r, K))
                   : 13 + 0.265 * planes + rounds * (steps * 0.864 + 4.7) +
                         (dM + dN) * steps * 64 * planes / 4.5e6 +
                         dM * dN * 1e-6 * (19 + 0.9 * words * res_limbs(r, K));
    double slices;
    if (r.nb) {
        slices = std::min(40.0, 18 + 2.4 * dS) + std::max(dM * dN * dK * dS * (dS + 1) / 62e6, 0.0045 * dK * dS * (dS + 1));
    } else if (tri_us > 0) {
        slices = 8 + 1.03 * tri_us;
    } else {
        const bool two = duo && r.S <= kDuoMax;
        const double per = two ? 0.0095 : 0.0134;
        slices = (two ? 25 : 30) + std::ceil(std::ceil(dM / 64) * std::ceil(dN / 32) / 256) *
                          (std::ceil(dK / 64) * dS * (dS + 1) * per + 15);
    }
    return residues * 1.03 < slices;
}

bool res_panels(const ResPlan& r, int64_t M, int64_t N, int64_t K, ResPanels& p)
{
    constexpr size_t kLimit = (size_t)9 << 30;
    p.mr = M;
    p.nc = N;
    ResLayout l;
    for (;;) {
        // the last diagonal's products in as many units as fill the chip once
        // (a unit of several is as long as several others, and the workgroups
        // take tiles in a fixed order)
        const int64_t T = ((p.mr + 255) / 256) * ((p.nc + 255) / 256);
        p.bq = p.nchunk = 0;
        if (r.nbd) {
            const int64_t want = std::min<int64_t>(r.nbd, (kResGroups + T - 1) / T);
            p.bq = (int)std::min<int64_t>(r.bfit, (r.nbd + want - 1) / want);
            p.nchunk = (r.nbd + p.bq - 1) / p.bq;
        }
        res_layout(r, p.mr, p.nc, p.nchunk, K, nullptr, l);
        // the interpolation reaches 32 planes with 32-bit offsets
        if (l.total <= kLimit && l.nbA * l.nbB * 256 <= (INT64_C(1) << 27) &&
            T * (r.npp() + p.nchunk) <= 0x7fffffff) {
            p.bytes = l.total;
            p.res_at = l.R;
            p.single = p.mr == M && p.nc == N;
            return true;
        }
        int64_t& side = p.mr >= p.nc ? p.mr : p.nc;
        if (side <= 4 * kResTile)
            return false;
        side = round_up64((side + 1) / 2, kResTile);
    }
}

bool res_cuts(const ResPlan& r, int m) { return m <= 4 && r.SB <= 32; }

hipError_t launch_resid(const ResPlan& r, const ResPanels& pn, const GemmArgs& g, const SplitSide& sideA,
                        const SplitSide& sideB, char* scratch, hipStream_t st)
{
    const int64_t K = g.nkc * kKcI8, nkr = res_steps(K);
    ResLayout l;
    res_layout(r, pn.mr, pn.nc, pn.nchunk, K, scratch, l);
    const ResShape s{r.L, r.N, r.P, r.SB, r.nb, r.S, r.beta, r.nbd};
    hipLaunchKernelGGL(k_res_tables, dim3(2 * r.P + 1), dim3(512), 0, st, s, l.t);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;

    ResFinalArgs fa;
    fa.L = r.L;
    fa.N = r.N;
    fa.P = r.P;
    fa.Lp = l.t.Lp;
    fa.Np = l.t.Np;
    fa.w = r.w;
    fa.nchunk = pn.nchunk;
    fa.W = l.t.W;
    fa.g = g;
    unsigned __int128 Mq = 1;
    for (int i = 0; i < r.P; ++i)
        Mq *= (unsigned)kPrimes[i];
    const uint64_t Mm = (uint64_t)Mq;   // below 2^63
    for (int i = 0; i < kResMaxPrimes; ++i) {
        const uint64_t c = i < r.P ? Mm / (uint64_t)kPrimes[i] : 0;
        fa.Wh[i] = (double)(c >> kResSplit);
        fa.Wl[i] = (double)(c & ((1u << kResSplit) - 1));
    }
    fa.Mh = (double)(Mm >> kResSplit);
    fa.Ml = (double)(Mm & ((1u << kResSplit) - 1));
    fa.invM = 1.0 / (double)Mm;

    const int nl = res_limbs(r, K);

    // A sum v of products of centred residues has |v| <= K ((p-1)/2)^2.  The
    // one-step reduction's quotient is v / p up to half a unit of v's 24-bit
    // rounding and the relative error of 1 / p (below 2^-24: 0.50 of it for p =
    // 251, 0.88 for 241, 0.84 for 223), so it leaves |r| <= p / 2 + 1 + that
    // error times v.  At K = 2048 that is 127.45 for p = 251, the binding one
    // (125.5 + 1 + 0.95), and at most 123.1 for the others: over all sums r
    // reaches 127, and past 2048 depths p = 251 leaves the byte.
    const bool wide = nkr * kKcI8 > 2048;

    auto eval = [&](const char* dig, int64_t rows, const int8_t* V, char* out, int64_t plane) {
        ResEvalArgs ea{dig, out, V, l.t.pc, plane, (int)g.nkc, (int)nkr, r.SB, r.planes(), l.t.KD};
        const int64_t nrb = (rows + 15) / 16;
        for (int64_t y0 = 0; y0 < nrb; y0 += 65535) {
            const dim3 grid((unsigned)nkr, (unsigned)std::min<int64_t>(nrb - y0, 65535));
            ResEvalArgs ey = ea;
            ey.dig += y0 * g.nkc * (int64_t)r.SB * 1024;
            ey.out += y0 * nkr * 1024;
            switch (r.SB <= 32 ? 0 : r.kt()) {
            case 0: hipLaunchKernelGGL((k_res_eval<0>), grid, dim3(256), 0, st, ey); break;
            case 1: hipLaunchKernelGGL((k_res_eval<1>), grid, dim3(256), 0, st, ey); break;
            case 2: hipLaunchKernelGGL((k_res_eval<2>), grid, dim3(256), 0, st, ey); break;
            default: hipLaunchKernelGGL((k_res_eval<3>), grid, dim3(256), 0, st, ey); break;
            }
            const hipError_t ee = hipGetLastError();
            if (ee != hipSuccess)
                return ee;
        }
        return hipSuccess;
    };
    // residues of A's rows r0 .. and / or of B's columns c0 .. from the words
    auto cut = [&](int64_t r0, int64_t mr, int64_t c0, int64_t nc, char* outA, char* outB) {
        ResCutArgs ca;
        auto side = [&](int k, const SplitSide& x, int64_t at, int64_t rows, char* out, const int8_t* V, int64_t plane) {
            ca.s[k] = x;
            ca.s[k].op.p += at * x.op.sr;
            ca.s[k].op.R -= at;
            ca.s[k].E += at;
            ca.s[k].nrb = (rows + 15) / 16;
            ca.s[k].out = out;
            ca.V[k] = V;
            ca.plane[k] = plane;
        };
        int n = 0;
        if (outA)
            side(n++, sideA, r0, mr, outA, l.t.VA, l.psA);
        if (outB)
            side(n++, sideB, c0, nc, outB, l.t.VB, l.psB);
        if (n == 1)
            ca.s[1] = ca.s[0], ca.V[1] = ca.V[0], ca.plane[1] = ca.plane[0];   // not read
        ca.pc = l.t.pc;
        ca.S = r.S;
        ca.beta = r.beta;
        ca.nb = r.nb;
        ca.SB = r.SB;
        ca.planes = r.planes();
        ca.KD = l.t.KD;
        const int form = r.nb ? kCutF64 : r.beta == 7 ? kCutSm : kCutBal;
        const int64_t nrb = std::max(ca.s[0].nrb, ca.s[1].nrb);
        for (ca.rb0 = 0; ca.rb0 < nrb; ca.rb0 += 65535) {
            const dim3 grid((unsigned)nkr, (unsigned)std::min<int64_t>(nrb - ca.rb0, 65535), n);
            const hipError_t ce = g.m == 1   ? launch_res_cut<1>(ca, form, grid, st)
                                  : g.m == 2 ? launch_res_cut<2>(ca, form, grid, st)
                                             : launch_res_cut<4>(ca, form, grid, st);
            if (ce != hipSuccess)
                return ce;
        }
        return hipSuccess;
    };
    const bool cuts = res_cuts(r, g.m);
    const int64_t row_bytes = g.nkc * (int64_t)r.SB * 64;   // digit bytes of one row (64 depths x SB per chunk)
    char* pA = scratch + l.A;
    char* pB = scratch + l.B;
    for (int64_t r0 = 0; r0 < g.M; r0 += pn.mr) {
        const int64_t mr = std::min(pn.mr, g.M - r0);
        if (!cuts && (e = eval((const char*)g.A + r0 * row_bytes, mr, l.t.VA, pA, l.psA)) != hipSuccess)
            return e;
        for (int64_t c0 = 0; c0 < g.N; c0 += pn.nc) {
            const int64_t nc = std::min(pn.nc, g.N - c0);
            const bool newB = r0 == 0 || pn.nc < g.N;
            if (cuts) {
                if ((c0 == 0 || newB) &&
                    (e = cut(r0, mr, c0, nc, c0 == 0 ? pA : nullptr, newB ? pB : nullptr)) != hipSuccess)
                    return e;
            } else if (newB && (e = eval((const char*)g.B + c0 * row_bytes, nc, l.t.VB, pB, l.psB)) != hipSuccess) {
                return e;
            }
            ResGemmArgs ga;
            ga.A = pA;
            ga.B = pB;
            ga.R = scratch + l.R;
            ga.Rb = (int32_t*)(scratch + l.Rb);
            ga.psA = l.psA;
            ga.psB = l.psB;
            ga.psR = l.psR;
            ga.nbA = (int)((mr + 15) / 16);
            ga.nbB = (int)((nc + 15) / 16);
            ga.gx = (int)((nc + kResTile - 1) / kResTile);
            ga.gy = (int)((mr + kResTile - 1) / kResTile);
            ga.nkc = (int)nkr;
            ga.N = r.N;
            ga.npp = r.npp();
            ga.nbd = r.nbd;
            ga.bq = pn.bq;
            ga.nchunk = pn.nchunk;
            for (int i = 0; i < kResMaxPrimes; ++i)
                ga.p[i] = kPrimes[i];
            hipLaunchKernelGGL((wide ? k_res_gemm<true> : k_res_gemm<false>),
                               dim3((unsigned)std::min<int64_t>((int64_t)ga.gx * ga.gy * (r.npp() + pn.nchunk), kResGroups)),
                               dim3(256), 0, st, ga);
            if ((e = hipGetLastError()) != hipSuccess)
                return e;
            fa.R = ga.R;
            fa.Rb = ga.Rb;
            fa.psR = l.psR;
            fa.nbA = ga.nbA;
            fa.nbB = ga.nbB;
            fa.r0 = r0;
            fa.c0 = c0;
            if ((e = dispatch_res_final(fa, nl, res_packed(r), st)) != hipSuccess)
                return e;
        }
    }
    return hipSuccess;
}

}  // namespace mdg
