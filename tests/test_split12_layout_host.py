"""Host check of slot12 (csrc/ntt.hip), the LDS slot of the N = 2^12 transforms:
a bijection on a limb and on a wave's tile, and 32 distinct 8-byte banks per
half-wave in every layout that exchanges through it.  The formulas are restated
from the kernel source, which the test reads to make sure of them."""
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def slot12(e):
    h = (e >> 5) & 7
    return e ^ h ^ ((h >> 1) << 3)


# element of lane (or thread) t's i-th value
WHOLE = {"a": lambda t, i: t + 512 * i, "b": lambda t, i: 512 * (t >> 6) + (t & 63) + 64 * i,
         "c": lambda t, i: 64 * (t >> 3) + (t & 7) + 8 * i, "d": lambda t, i: 8 * t + i}
TILE = {"column A": lambda t, i: 8 * ((t >> 3) + 8 * i) + (t & 7), "column B": lambda t, i: 8 * (8 * (t >> 3) + i) + (t & 7),
        "row A": lambda t, i: 64 * (t >> 3) + (t & 7) + 8 * i, "row B": lambda t, i: 64 * (t >> 3) + 8 * (t & 7) + i}


@pytest.mark.parametrize("layouts,threads", [(WHOLE, 512), (TILE, 64)])
def test_slot12_is_a_conflict_free_bijection(layouts, threads):
    n = 8 * threads
    assert sorted(slot12(e) for e in range(n)) == list(range(n))
    for name, f in layouts.items():
        assert sorted(f(t, i) for t in range(threads) for i in range(8)) == list(range(n)), name
        for t0 in range(0, threads, 32):
            for i in range(8):
                assert len({slot12(f(t, i)) % 32 for t in range(t0, t0 + 32)}) == 32, (name, t0, i)


def test_formulas_match_the_kernel_source():
    src = re.sub(r"\s+", " ", open(os.path.join(ROOT, "paper_2507_04775_amd", "csrc", "ntt.hip")).read())
    assert "const uint32_t h = (e >> 5) & 7; return e ^ h ^ ((h >> 1) << 3); }" in src
    for name, body in (("p12a", "t + 512 * i"), ("p12b", "512 * (t >> 6) + (t & 63) + 64 * i"),
                       ("p12c", "64 * (t >> 3) + (t & 7) + 8 * i"), ("p12d", "8 * t + i")):
        assert "%s(uint32_t t, int i) { return %s; }" % (name, body) in src
    assert "exchange12(ar, v, L, [&](int i) { return e(s + 8 * i); }, [&](int i) { return e(8 * s + i); });" in src
    assert src.count("[&](uint32_t p) { return 8 * p + col; }") == 2 and src.count("return 64 * row + p; }") == 3
