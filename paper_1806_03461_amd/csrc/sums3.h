// An external product's two output components from three sums instead of four.
//
// A blind-rotation step needs P_c = sum_r digit_r * key_{r,c} mod (X^1024 + 1, 2^32) for c = 0, 1, the four digit
// polynomials with coefficients in [-512, 512) and the key's 32 bits wide.  A double-precision product leaves the
// integers exact only while the key's factor stays well below 32 bits, so 2 x 32 bits of key have to be spread over
// several inverse transforms.  Cutting every component into two limbs of 16 bits takes four; these three, of
// 21 or 22 bits each, are enough (b = kSumBits = 11):
//     low    Q = sum_r digit_r * centred((key_{r,0} + 2^b key_{r,1}) mod 2^(2b))      an integer, |Q| <= 2^42
//     top 0  A = sum_r digit_r * key_{r,0} / 2^b                                      = P_0 / 2^b as an integer product
//     top 1  B = sum_r digit_r * key_{r,1} / 2^b                                      = P_1 / 2^b
// Q is rounded to the integer it is.  Q = P_0 (mod 2^b), and 2^b A is P_0 to within far less than 2^(b-1): P_0 is the one
// number near 2^b A that agrees with Q.  Then (Q - P_0) / 2^b = P_1 (mod 2^b), and P_1 follows from B in the same way.
//
// Exactness.  With the bound 10 u log2(512) |digit|_2 |factor|_2 over four rows, which is 2^-10.5 for factors of 16
// bits, the error of Q (22 bits) is below 2^-4.5 and that of A and B (21 bits) below 2^-5.5; each has to stay below
// 1/2.  Seen on the host: Q 3.5e-5, A and B 1.8e-5 with random operands; 3.5e-3 and 1.8e-3 with every operand at one end of its
// range.
#pragma once
#include "fft512.h"

namespace fft512 {

constexpr int kSums = 3;            // sums in the order low, top 0, top 1
constexpr int kSumBits = 11;
constexpr uint32_t kSumMask = (1u << kSumBits) - 1u;

// factor o of the key coefficients (component 0, component 1) of a row
FFT_HD double sum_factor(uint32_t key0, uint32_t key1, int o) {
    if (o == 0) return (double)((int32_t)((key0 + (key1 << kSumBits)) << (32 - 2 * kSumBits)) >> (32 - 2 * kSumBits));
    return (double)(int32_t)(o == 1 ? key0 : key1) * (1.0 / (1 << kSumBits));
}

// The factors' spectra of one step, in the order in which a wave that holds whole polynomials reads them: a sum at a time, at
// one frequency of every lane, its four rows behind each other.  Complex word of row r of sum o at register k2 of a lane.
FFT_HD constexpr int sum_key_word(int k2, int o, int r, int lane) { return ((k2 * kSums + o) * 4 + r) * 64 + lane; }
constexpr int kSumKeyWords = sum_key_word(8, 0, 0, 0);

// Added to a number in a double's middle, these leave it in fixed point in the low word: an integer, or (with 2^-10 as
// the unit of the last place and 2^(b-1) units of half a P added, which turns rounding down into rounding to nearest) P / 2.
// |A|, |B| < 2^41: 4,096 terms of at most 512 * 2^31 / 2^b, of which not all 4,096 can be the largest with the same sign
// on the side where 1.5 * 2^42 - A would leave its binade.
constexpr double kIntegerShift = 6755399441055744.0;                       // 1.5 * 2^52
constexpr double kHalfShift = 6597069766656.0 + 0.5;                       // 1.5 * 2^42 + 2^(b-2) * 2^-10

// -P_0 from q = low word of kIntegerShift + Q and h = low word of kHalfShift - A; q becomes (Q - P_0) / 2^b = P_1 mod 2^b,
// with which the same step gives -P_1 from B.
FFT_HD uint32_t minus_product(uint32_t &q, uint32_t h) {
    const uint32_t w = ((h << 1) + q) & ~kSumMask;        // 2 h + q = (Q - P) + 2^(b-1) + error
    const uint32_t r = w - q;
    q = w >> kSumBits;
    return r;
}

}  // namespace fft512
