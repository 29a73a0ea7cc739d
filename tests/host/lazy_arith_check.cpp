// CPU check of the integer NTT path's lazy arithmetic (modarith.h): shoup_add's
// product range and residue for any 64-bit input, csub_sign, and the ranges of
// a whole transform's butterflies, for primes up to 2^61.
#include <cstdio>
#include <vector>

#include "../../paper_2507_04775_amd/csrc/modarith.h"

using namespace ckks;
typedef unsigned __int128 u128x;

static uint64_t state = 42;
static uint64_t rng()
{
    state ^= state << 13;
    state ^= state >> 7;
    state ^= state << 17;
    return state;
}

int main()
{
    int fails = 0;
    auto check = [&](bool ok, const char *what, uint64_t q) {
        if (!ok && ++fails < 20) std::printf("%s, q = %llu\n", what, (unsigned long long)q);
    };
    // odd moduli are enough: nothing here needs a prime
    const std::vector<uint64_t> qs = {(1ull << 61) - 1, (1ull << 61) - (1ull << 20) + 1, (1ull << 60) - 93, (1ull << 60) + 33,
                                      (1ull << 50) + 1, (1ull << 50) + 4097, 3 * (1ull << 57) + 5, 786433};
    for (uint64_t q : qs) {
        const uint64_t nq = 0 - q, q4 = 4 * q;
        auto comp = [&](uint64_t w) { return (uint64_t)(((u128x)w << 64) / q); };
        const uint64_t we[] = {0, 1, 2, q / 2, q - 2, q - 1, 0xFFFFFFFFull % q, (1ull << 32) % q};
        const uint64_t ye[] = {0, 1, 0xFFFFFFFFull, 1ull << 32, ~0ull, ~0ull - 0xFFFFFFFFull, 8 * q - 1, q4 - 1, q};
        for (int rep = 0; rep < 20000; ++rep) {
            const uint64_t w = rep < 200 ? we[rep % 8] : rng() % q;
            const uint64_t y = rep < 200 ? ye[rep / 8 % 9] : rep % 3 ? rng() : rng() % (8 * q);
            const uint64_t acc = rng() % q4, r = shoup_add(acc, y, w, comp(w), nq) - acc;
            check(r < q4, "shoup_add range", q);
            check(r % q == (uint64_t)((u128x)y * w % q), "shoup_add residue", q);
            for (uint64_t m : {q4, 2 * q, q}) {
                const uint64_t x = rng() % (2 * m);
                check(csub_sign(x, 0 - m) == (x >= m ? x - m : x), "csub_sign", q);
            }
        }
        // butterflies over many stages, each pair's partner at its extremes now and then
        uint64_t x = q - 1, y = q - 1, u = q4 - 1, v = 0;
        for (int st = 0; st < 4000; ++st) {
            const uint64_t w = st % 5 ? rng() % q : q - 1, ws = comp(w);
            const uint64_t a = csub_sign(x, 4 * nq), want = (uint64_t)(((u128x)y * w + x) % q);
            const uint64_t wneg = (uint64_t)((x % q + q - (uint64_t)((u128x)y * w % q)) % q);
            x = shoup_add(a, y, w, ws, nq);
            y = shl_add<1>(a, q4) - x;
            check(x < 8 * (u128x)q && y < 8 * (u128x)q && x % q == want && y % q == wneg, "forward butterfly", q);
            const uint64_t d = u + q4 - v, ds = (uint64_t)((u128x)(u % q + q - v % q) % q * w % q), s = (uint64_t)(((u128x)u + v) % q);
            u = csub_sign(u + v, 4 * nq);
            v = shoup_add(0, d, w, ws, nq);
            check(u < q4 && v < q4 && u % q == s && v % q == ds, "inverse butterfly", q);
            if (st % 7 == 0) u = q4 - 1, v = st % 2 ? 0 : q4 - 1;
            if (st % 11 == 0) x = 8 * q - 1, y = 8 * q - 1;
        }
    }
    if (fails) return 1;
    std::printf("ok\n");
    return 0;
}
