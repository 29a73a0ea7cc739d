// Host side of the base conversions: the constant row of a source basis B =
// {b_i} and a target prime c, in the form the kernels' sums take it (shared by
// the context and a host-side check).
#pragma once
#include "modarith.h"

namespace ckks {

constexpr int kMaxDigitPrimes = 16;  // primes per digit / in the special basis

// Words of a constant row.  With at most kFoldMaxTerms source rows, and for
// targets of 2^50 and above where the columns hold the sum, it is in the form of
// FoldSum (FoldSumWide): {fold_const(h_i), fold_const([2^30 h_i]_c)} at 2 i, h_i =
// [B/b_i]_c.  Others hold h_i at i (split_const(h_i) below 2^50).  The last two
// words: the start values of a FoldSum's columns; {1, corr} for FoldSumWide, whose
// column b starts at corr; {0, corr} else, corr added to the reduced sum.
constexpr uint32_t kConvRow = 2 * kMaxDigitPrimes + 2;
constexpr uint32_t kConvStart = 2 * kMaxDigitPrimes;

// shifted: the inputs are centred y_i plus b_i, below 3/2 b_i (ModDown), so the
// plain sum is ns [B]_c too large; the start value or corr takes that off.
inline void conv_row(uint64_t *row, const uint64_t *src, uint32_t ns, uint64_t c, bool shifted)
{
    typedef unsigned __int128 wide;
    auto mul = [c](uint64_t a, uint64_t b) { return (uint64_t)((wide)a * b % c); };
    const bool fp = c < kFpMaxPrime;
    const int sh = fp ? kFoldShift : kFoldShiftWide;
    uint64_t B = 1, h[kMaxDigitPrimes], hc[kMaxDigitPrimes];
    wide smax = 0, amax = 0, bmax = c;
    for (uint32_t i = 0; i < ns; ++i) {
        h[i] = 1;
        for (uint32_t k = 0; k < ns; ++k)
            if (k != i) h[i] = mul(h[i], src[k] % c);
        B = mul(B, src[i] % c);
        hc[i] = mul(h[i], (1ull << kFoldCut) % c);
        const uint64_t ymax = shifted ? src[i] + src[i] / 2 : src[i];
        const uint64_t y0 = (1ull << kFoldCut) - 1, y1 = ymax >> kFoldCut, mask = (1ull << sh) - 1;
        smax += (wide)y0 * h[i] + (wide)y1 * hc[i];
        amax += (wide)y0 * (h[i] >> sh) + (wide)y1 * (hc[i] >> sh);
        bmax += (wide)y0 * (h[i] & mask) + (wide)y1 * (hc[i] & mask);
    }
    const bool fold = ns <= kFoldMaxTerms && (fp || ((amax >> 64) == 0 && (bmax >> 64) == 0));
    for (uint32_t i = 0; i < ns; ++i) {
        if (!fold) {
            row[i] = fp ? split_const(h[i]) : h[i];
        } else {
            row[2 * i] = fp ? fold_const<kFoldShift>(h[i]) : fold_const<kFoldShiftWide>(h[i]);
            row[2 * i + 1] = fp ? fold_const<kFoldShift>(hc[i]) : fold_const<kFoldShiftWide>(hc[i]);
        }
    }
    const uint64_t back = mul(ns % c, B), corr = shifted && back ? c - back : 0;
    const uint64_t half = fold && fp ? (uint64_t)(smax >> (kFoldShift + 1)) : 0;
    row[kConvStart] = fold && !fp ? 1 : 0 - half;
    row[kConvStart + 1] = (mul(half % c, (1ull << kFoldShift) % c) + corr) % c;
}

}  // namespace ckks
