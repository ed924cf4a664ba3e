// The residue contraction: the same exact diagonal sums as the triangle of
// slice products, from fewer matrix products.
//
// The digits of an entry are read as the coefficients of a polynomial,
//   A(y) = sum_{b < L} a_b y^b,   B(y) = sum_{c < L} b_c y^c,
// with blocks a_b of one FP64 digit or of two adjacent INT8 digits, so the
// sums the method needs are the low half of a matrix polynomial product:
//   P_t = sum_{b + c = t} sum_k a_ik,b b_kj,c,   t < L,
//   X = sum_t P_t 2^(w (L - 1 - t)) + Q,
// w the width of a block in bits.  A polynomial product of degree 2 L - 2
// is fixed by its values at N = 2 L - 1 points, and a value is one matrix
// product instead of t + 1 per coefficient.  To stay in INT8 the values are
// taken modulo primes p < 256 (points 0, +-1, .., +-(L-1), distinct modulo
// every prime used): per prime N products of INT8 residue matrices with
// INT32 accumulation, then per output the interpolation modulo p and the
// Chinese remainder, which give every |P_t| < (product of the primes) / 2
// exactly.  All of it is integer arithmetic: X is the triangle's X bit for
// bit.
//
// INT8 digits in pairs: with S odd, a_b = (d_2b, d_2b+1) on both sides; the
// pairs s + u <= S - 1 are the blocks with b + c < L = (S-1)/2 and, on the
// last diagonal s + u = S - 1, the L + 1 products of even digits, which run
// as they are (Q).  With S even B's blocks start one digit earlier (b_0 =
// (0, e_0), b_c = (e_2c-1, e_2c)), L = S / 2 and Q has L products.
//
// Work per output: N P + |Q| INT8 products of depth K against S (S+1) / 2
// (S = 27: 164 against 378; 56: 358 against 1596; 105: 683 against 5565;
// 10 FP64 digits of 21 bits: 152 INT8 products against 55 FP64 ones), plus
// the residues (per entry) and the interpolation (per output).
#pragma once

#include "mdgemm_internal.h"

namespace mdg {

constexpr int kResMaxPrimes = 8;
constexpr int kResTile = 256;        // outputs per workgroup side

struct ResPlan {
    int L = 0, N = 0, P = 0;         // coefficients, points, primes
    int SB = 0;                      // digit planes (bytes per entry) read by the evaluation
    int nb = 0;                      // FP64 form: byte planes per digit (0: INT8 digits)
    int S = 0, beta = 0, w = 0;      // slices, digit bits, block bits
    int nbd = 0;                     // products of the last diagonal (INT8)
    int bfit = 1;                    // those whose INT32 sum stays exact
    int npp() const { return N * P; }
    int planes() const { return N * P + nbd; }
    int kt() const { return (SB + 63) / 64; }
};

// Parameters for a product of depth K; false where the method does not
// apply (see the conditions in resid.hip).
bool res_plan(bool balanced, bool fp64, int S, int beta, int64_t K, ResPlan& r);

// 32-bit limbs of the folded integer (with its sign) at depth K.
int res_limbs(const ResPlan& r, int64_t K);

// Whether it is expected to be faster than the form's slice products (duo:
// the call may take the two-band INT8 kernel; tri_us: what the whole-triangle
// INT8 kernels are expected to take, where they apply, else 0).
bool res_pays(const ResPlan& r, int64_t M, int64_t N, int64_t K, bool duo, double tri_us);

// Scratch of one panel (Mr x Nc outputs, depth K) and the panel sizes that
// keep it below the limit; false if none does.
struct ResPanels {
    int64_t mr = 0, nc = 0;          // multiples of kResTile, or the whole extent
    int bq = 0, nchunk = 0;          // products of the last diagonal per unit, their units
    size_t bytes = 0;                // of one panel's planes, residues and tables
    size_t res_at = 0;               // from here on the products' residues: free until the products run
    bool single = false;             // one panel is the whole product
};
bool res_panels(const ResPlan& r, int64_t M, int64_t N, int64_t K, ResPanels& p);

// Fixed-point and rounded outputs as GemmArgs' (C, ldc, psc, E, F, M, N, m,
// fixX, fixScale, fixNL, ncol, beta, S).  Where res_cuts the digits are cut
// from the operands' words (A, B: op and E) by the evaluation itself; else
// a.A and a.B are digit planes in INT8 fragment order (launch_split_i8, or
// launch_split_f64b for the FP64 form).
bool res_cuts(const ResPlan& r, int m);
hipError_t launch_resid(const ResPlan& r, const ResPanels& p, const GemmArgs& a, const SplitSide& A, const SplitSide& B,
                        char* scratch, hipStream_t st);

// FP64 digits of beta bits as byte planes: digit s is sum_k c_k 256^k with
// c_k in [-128, 127], byte k in plane s nb + k, INT8 fragment order
hipError_t launch_split_f64b(const SplitSide& a, const SplitSide& b, int m, int S, int beta, int nb, int64_t nkc,
                             hipStream_t st);
int res_f64_bytes(int beta);

}  // namespace mdg
