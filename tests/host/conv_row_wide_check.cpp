// CPU check of the base conversions' rows that are summed in exact 128 bits
// (conv_row.h's {h_i ..., 0, corr} of targets of 2^50 and above): MacCols' columns
// and carries (modarith.h, inline assembly on the GPU, formed here step by step)
// hold the sum at the largest primes, and the sum reduced plus corr is the
// conversion.  Arguments: primes, the first of them the target.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../../paper_2507_04775_amd/csrc/conv_row.h"

using namespace ckks;
typedef unsigned __int128 wide;

static uint64_t state = 61;
static uint64_t rng()
{
    state ^= state << 13;
    state ^= state >> 7;
    state ^= state << 17;
    return state;
}

int main(int argc, char **argv)
{
    std::vector<uint64_t> all;
    for (int i = 1; i < argc; ++i) all.push_back(std::strtoull(argv[i], nullptr, 10));
    if (all.size() != 17) return 2;
    const uint64_t c = all[0];
    Prime P = {};
    P.q = c, P.two_q = 2 * c;
    P.r64 = (uint64_t)(((wide)1 << 64) % c);
    P.r64_s = (uint64_t)(((wide)P.r64 << 64) / c);
    P.one_s = (uint64_t)(((wide)1 << 64) / c);
    int checked = 0;
    for (uint32_t ns = 1; ns <= kMaxDigitPrimes; ++ns)
        for (int shifted = 0; shifted < 2; ++shifted) {
            const std::vector<uint64_t> src(all.begin() + 1, all.begin() + 1 + ns);
            std::vector<uint64_t> row(kConvRow, 0), h(ns);
            conv_row(row.data(), src.data(), ns, c, shifted != 0);
            if (row[kConvStart]) continue;  // summed in two columns
            uint64_t B = 1;
            for (uint32_t i = 0; i < ns; ++i) {
                B = (uint64_t)((wide)B * (src[i] % c) % c);
                h[i] = 1;
                for (uint32_t k = 0; k < ns; ++k)
                    if (k != i) h[i] = (uint64_t)((wide)h[i] * (src[k] % c) % c);
            }
            for (int rep = 0; rep < 500; ++rep) {
                MacCols m;
                wide exact = 0, hi = 0;
                uint64_t want = shifted ? c - (uint64_t)((wide)ns * B % c) : 0;
                for (uint32_t i = 0; i < ns; ++i) {
                    const uint64_t top = shifted ? src[i] + (src[i] - 1) / 2 : src[i] - 1, low = shifted ? (src[i] + 1) / 2 : 0;
                    const uint64_t y = join_word(cut_word(rep == 0 ? top : rep == 1 ? low : low + rng() % (top - low + 1)));
                    // rep 0 also takes the largest constant there is, for the columns' sake
                    const uint64_t k = rep == 0 ? c - 1 : row[i];
                    const uint32_t y0 = (uint32_t)y, y1 = (uint32_t)(y >> 32), k0 = (uint32_t)k, k1 = (uint32_t)(k >> 32);
                    m.lo += (uint64_t)y0 * k0, m.clo += m.lo < (uint64_t)y0 * k0;
                    m.mid += (uint64_t)y0 * k1, m.cmid += m.mid < (uint64_t)y0 * k1;
                    m.mid += (uint64_t)y1 * k0, m.cmid += m.mid < (uint64_t)y1 * k0;
                    m.hi += (uint64_t)y1 * k1, hi += (wide)y1 * k1;
                    exact += (wide)y * k;
                    want = (uint64_t)(((wide)(y % c) * h[i] + want) % c);
                }
                const u128 t = mac_total(m);
                if (hi >> 63 || t.lo != (uint64_t)exact || t.hi != (uint64_t)(exact >> 64)) {
                    std::printf("ns %u shifted %d: the columns do not hold the sum\n", ns, shifted);
                    return 1;
                }
                if (rep && addmod(reduce128(t, P), row[kConvStart + 1], c) != want) {
                    std::printf("ns %u shifted %d: wrong residue\n", ns, shifted);
                    return 1;
                }
                ++checked;
            }
        }
    if (!checked) return 1;
    std::printf("%d ok\n", checked);
    return 0;
}
