// CPU check of the base conversions' constant rows (conv_row.h) with the
// kernels' own sums (modarith.h): FoldSum for targets below 2^50 and at most
// kFoldMaxTerms source rows, FoldSumWide above 2^50 where the row says so,
// MacSplit's exact columns for more source rows, against the exact sum of y_i
// [B/b_i]_c reduced by 128-bit arithmetic.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../../paper_2507_04775_amd/csrc/conv_row.h"

using namespace ckks;
typedef unsigned __int128 u128x;

static uint64_t state = 250704775;
static uint64_t rng()
{
    state ^= state << 13;
    state ^= state >> 7;
    state ^= state << 17;
    return state;
}

static uint64_t powm(uint64_t b, uint64_t e, uint64_t m)
{
    u128x r = 1, x = b % m;
    for (; e; e >>= 1, x = x * x % m)
        if (e & 1) r = r * x % m;
    return (uint64_t)r;
}

static bool prime(uint64_t n)
{
    uint64_t d = n - 1;
    int s = 0;
    while (d % 2 == 0) d /= 2, ++s;
    for (uint64_t b : {2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37}) {
        if (n % b == 0) return n == b;
        uint64_t x = powm(b, d, n);
        bool ok = x == 1 || x == n - 1;
        for (int i = 1; i < s && !ok; ++i) ok = (x = (uint64_t)((u128x)x * x % n)) == n - 1;
        if (!ok) return false;
    }
    return true;
}

static std::vector<uint64_t> primes_of(int bits, size_t count)
{
    std::vector<uint64_t> out;
    for (uint64_t q = (1ull << bits) - 131071; out.size() < count; q -= 131072)
        if (prime(q)) out.push_back(q);
    return out;
}

int main()
{
    int fails = 0;
    for (int sbits : {30, 50, 60, 61}) {
        const std::vector<uint64_t> all = primes_of(sbits, 16);
        for (int tbits : {20, 30, 40, 50, 51, 60, 61}) {
            // a target outside the source basis
            const uint64_t c = primes_of(tbits, tbits == sbits ? 17 : 1).back();
            const FpMod m = {(double)c, 1.0 / (double)c};
            Prime P = {};
            P.q = c, P.two_q = 2 * c;
            P.r64 = (uint64_t)(((u128x)1 << 64) % c);
            P.r64_s = (uint64_t)(((u128x)P.r64 << 64) / c);
            P.one_s = (uint64_t)(((u128x)1 << 64) / c);
            for (uint32_t ns : {1u, 2u, 4u, 11u, 12u, 13u, 16u})
                for (int shifted = 0; shifted < 2; ++shifted) {
                    std::vector<uint64_t> src(all.begin(), all.begin() + ns), row(kConvRow, 0), h(ns);
                    conv_row(row.data(), src.data(), ns, c, shifted != 0);
                    uint64_t B = 1;
                    for (uint32_t i = 0; i < ns; ++i) {
                        B = (uint64_t)((u128x)B * (src[i] % c) % c);
                        h[i] = 1;
                        for (uint32_t k = 0; k < ns; ++k)
                            if (k != i) h[i] = (uint64_t)((u128x)h[i] * (src[k] % c) % c);
                    }
                    for (int rep = 0; rep < 400; ++rep) {
                        u128x want = shifted ? (u128x)(c - (uint64_t)((u128x)ns * B % c)) : 0;
                        std::vector<uint64_t> y(ns);
                        for (uint32_t i = 0; i < ns; ++i) {
                            const uint64_t b = src[i], top = shifted ? b + b / 2 : b - 1, lo = shifted ? (b + 1) / 2 : 0;
                            const uint64_t edge[] = {lo, top, (1ull << 32) - 1 < top ? (1ull << 32) - 1 : top, top - 1};
                            y[i] = rep < 4 ? edge[rep] : rep % 5 == 0 ? edge[rng() % 4] : lo + rng() % (top - lo + 1);
                            want = (want + (u128x)(y[i] % c) * h[i]) % c;
                        }
                        want %= c;
                        uint64_t got;
                        if (c >= kFpMaxPrime) {
                            if (!row[kConvStart]) {  // mac_cols: inline assembly, checked on the GPU
                                if (rep == 0 && ns <= kFoldMaxTerms && sbits <= 50 && !shifted) {
                                    std::printf("ns %u of %d bits into %d bits is not folded\n", ns, sbits, tbits);
                                    ++fails;
                                }
                                continue;
                            }
                            FoldSumWide s = {{0, row[kConvStart + 1]}};
                            for (uint32_t i = 0; i < ns; ++i) s.add(cut_word(y[i]), row[2 * i], row[2 * i + 1]);
                            got = s.residue(c, m.qinv);
                            if (!((double)got > 0.48 * (double)c && (double)got < 1.52 * (double)c)) {
                                std::printf("ns %u c %llu: residue out of range\n", ns, (unsigned long long)c);
                                ++fails;
                            }
                            got %= c;
                        } else if (ns <= kFoldMaxTerms) {
                            FoldSum s = {{row[kConvStart], row[kConvStart + 1]}};
                            for (uint32_t i = 0; i < ns; ++i) s.add(cut_word(y[i]), row[2 * i], row[2 * i + 1]);
                            const double r = s.residue(m), bound = (0.5 + 0x1p-14) * (double)c + 0x1p32;
                            if (!(r <= bound && r >= -bound)) {
                                std::printf("ns %u c %llu: |residue| %g above %g\n", ns, (unsigned long long)c, r, bound);
                                ++fails;
                            }
                            got = fp_canonical(r, m);
                        } else {
                            MacSplit s;
                            for (uint32_t i = 0; i < ns; ++i) s.add(join_word(cut_word(y[i])), row[i]);
                            got = addmod(reduce128(s.total(), P), row[kConvStart + 1], c);
                        }
                        if (got != (uint64_t)want) {
                            std::printf("ns %u shifted %d source %d-bit target %llu: got %llu want %llu\n", ns, shifted,
                                        sbits, (unsigned long long)c, (unsigned long long)got, (unsigned long long)want);
                            if (++fails > 20) return 1;
                        }
                    }
                }
        }
    }
    if (fails) return 1;
    std::printf("ok\n");
    return 0;
}
