// Host side of the base conversions: the constant row of a source basis B =
// {b_i} and a target prime c, in the form the kernels' sums take it (shared by
// the context and a host-side check).
#pragma once
#include "modarith.h"

namespace ckks {

constexpr int kMaxDigitPrimes = 16;  // primes per digit / in the special basis

// Words of a constant row.  Targets below 2^50 with at most kFoldMaxTerms
// source rows hold {fold_const(h_i), fold_const([2^32 h_i]_c)} at 2 i, h_i =
// [B/b_i]_c; other targets hold h_i at i (split_const(h_i) below 2^50).  The
// last two words are the columns' start values of a FoldSum, else {0, corr}
// with corr added to the reduced sum.
constexpr uint32_t kConvRow = 2 * kMaxDigitPrimes + 2;
constexpr uint32_t kConvStart = 2 * kMaxDigitPrimes;

// shifted: the inputs are centred y_i plus b_i, below 3/2 b_i (ModDown), so the
// plain sum is ns [B]_c too large; the start value or corr takes that off.
inline void conv_row(uint64_t *row, const uint64_t *src, uint32_t ns, uint64_t c, bool shifted)
{
    typedef unsigned __int128 wide;
    auto mul = [c](uint64_t a, uint64_t b) { return (uint64_t)((wide)a * b % c); };
    const bool fold = c < kFpMaxPrime && ns <= kFoldMaxTerms;
    uint64_t B = 1;
    wide smax = 0;
    for (uint32_t i = 0; i < ns; ++i) {
        uint64_t h = 1;
        for (uint32_t k = 0; k < ns; ++k)
            if (k != i) h = mul(h, src[k] % c);
        B = mul(B, src[i] % c);
        if (fold) {
            const uint64_t h32 = mul(h, (1ull << 32) % c);
            row[2 * i] = fold_const(h);
            row[2 * i + 1] = fold_const(h32);
            const uint64_t ymax = shifted ? src[i] + src[i] / 2 : src[i];
            smax += (wide)0xFFFFFFFFu * h + (wide)(ymax >> 32) * h32;
        } else {
            row[i] = c < kFpMaxPrime ? split_const(h) : h;
        }
    }
    const uint64_t back = mul(ns % c, B), corr = shifted && back ? c - back : 0;
    const uint64_t half = fold ? (uint64_t)(smax >> (kFoldShift + 1)) : 0;
    row[kConvStart] = 0 - half;
    row[kConvStart + 1] = (mul(half % c, (1ull << kFoldShift) % c) + corr) % c;
}

}  // namespace ckks
