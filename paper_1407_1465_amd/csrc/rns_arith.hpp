// RNS Montgomery products on the integer matrix cores (gfx950).
//
// An integer x is held as its residues modulo two bases of k primes just
// below 2^31 each, with products A and B.  A Montgomery product with A in the
// place of the power of two,
//     x, y  ->  r = (x y + q n) / A,   q = -x y n^-1 mod A (plus a multiple
//     of A),
// takes k independent word products per base and two base extensions: q from
// its residues in A to B, and r from B back to A.  An extension
//     sum_i xi_i * (A / a_i) mod b_j
// is a product with a constant matrix, the same for every modulus n, so a
// wave runs it for its 16 integers at once on the matrix cores: residues as
// four signed base-256 digits, the matrix's entries likewise, exact 32-bit
// accumulators.  What is left for the vector unit grows with k, not with
// k^2 (25 instructions per residue pair and product; the positional product
// of radix_bn.hpp grows with the square of the width).
//
// Values are bounded, never reduced: residues are signed 32-bit words below
// 0.9 * 2^31 (those in A below 0.73 m; those of an entering x, whose limbs are
// converted in sums of 7, below 0.94 * 2^31 in A).  q carries a multiple of A
// (its extension is not corrected): its residues are below 0.86 m where both
// factors have just entered, less otherwise, so |r| <= |x y| / A + 0.86 k n <
// 0.875 k n (rns_tables.py checks A and B against it).  The extension back is
// exact: alpha = round(sum_j xi_j / b_j) comes from the sum of the residues'
// top digits (off by at most k / 256 < 0.3 + |r| / B), and -alpha B is one
// more term of the matrix product.
//
// A residue is stored as x mod a_i in A, and as x * w_j mod b_j,
// w_j = (B / b_j)^-1, in B (the form the extension back takes as it is).
// Word products reduce by Montgomery's method with 2^32 and signed words:
// for |t| < 2^63 and u = -t / m mod 2^32 as a signed word, (t + u m) / 2^32
// is below |t| / 2^32 + m / 2.
//
// In B the new residue is red(s kappa + q v) with s = red(x y) and v from n;
// the extended q is a 47-bit sum lo + 2^16 hi of accumulators, and enters as
// lo v + hi v16 with v16 = 2^16 v mod b_j: no reduction of its own.
//
// Layout: lane l holds the residues 4 u + g, u < U, g = l / 16, of integer
// l % 16.  That is at once the second-operand and the accumulator layout of
// v_mfma_i32_16x16x64_i8 with the rows and columns of the constant matrices
// in the right order: four residues are one lane's 16 operand bytes of a k
// step, and a lane's four accumulators of a row tile (the four planes) are
// one residue.  No lane moves.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rsagpu {

// Constants of the configuration with U residues per lane and base
// (generated, see rns_tables.py).
template <int U>
struct RnsTables;

typedef int v4i __attribute__((ext_vector_type(4)));

// Montgomery reduction of a signed 64-bit value by 2^32 (see above).
__device__ __forceinline__ int rns_red(int64_t t, int m, int minv)
{
    const int u = (int)((uint32_t)t * (uint32_t)minv);
    t += (int64_t)u * m;
    return (int)(t >> 32);
}

// Added to a word, and exclusive-ored with the sum, this gives the word's
// signed base-256 digits as bytes.
constexpr int kDigitBias = 0x00808080;
__device__ __forceinline__ int rns_digits(int biased) { return biased ^ kDigitBias; }

// A residue's four planes acc0 + 2^8 acc1 + 2^16 acc2 + 2^24 acc3 as lo +
// 2^16 hi, and as one value.
__device__ __forceinline__ int rns_lo(v4i acc) { return acc[0] + (acc[1] << 8); }
__device__ __forceinline__ int rns_hi(v4i acc) { return acc[2] + (acc[3] << 8); }
__device__ __forceinline__ int64_t rns_planes(v4i acc)
{
    int k = 65536;
    asm("" : "+s"(k));                          // one multiply-add, not a 64-bit shift and add
    return (int64_t)rns_hi(acc) * k + rns_lo(acc);
}

// Work split of a tile of 16 integers over W waves: wave v owns the units
// v, v + W, ... below U of each base, at most UW, and the extensions' row
// tiles of its units.
template <int U_, int W_>
struct Rns {
    static constexpr int U = U_, W = W_;
    static constexpr int UW = (U + W - 1) / W;
    static constexpr int K = 4 * U;                     // residues per base
    static constexpr int KS = (U + 3) / 4;              // k steps of an extension
    using Tab = RnsTables<U>;

    static __device__ __forceinline__ v4i matrix_word(const uint32_t *mat, int tile, int s, int lane)
    {
        return reinterpret_cast<const v4i *>(mat)[(tile * KS + s) * 64 + lane];
    }
    // One row tile times the operand.
    static __device__ __forceinline__ v4i tile(const v4i (&mat)[KS], const v4i (&x)[KS])
    {
        v4i acc = {};
#pragma unroll
        for (int s = 0; s < KS; ++s) acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(mat[s], x[s], acc, 0, 0, 0);
        return acc;
    }
};

}  // namespace rsagpu
