"""Host logic of the autotuner: every launch size is timed through an operation
that has a launch of that size, and results measured on other launches are not
taken from the cache.  No GPU."""
import os
import re

import pytest

from paper_2507_04775_amd import ckks, tune

CSRC = os.path.join(os.path.dirname(os.path.abspath(tune.__file__)), "csrc")


class _Ctx:
    logn = 16

    def __init__(self, nq, K, dnum):
        self.nq, self.np, self.alpha = nq, K, -(-nq // dnum)

    def beta(self, level):
        return -(-(level + 1) // self.alpha)


ROWS, WHOLE = ckks.TILE_ROWS, ckks.TILE_TRANSFORM


@pytest.mark.parametrize("nq,K,dnum,level,modup,op,down", [
    (31, 4, 3, 30, 74, ("hoisted", ROWS), ROWS),    # HMult finishes ModUp's rows inside its inner product
    (31, 4, 3, 12, 21, ("hoisted", ROWS), ROWS),
    (24, 4, 2, 23, 32, ("hoisted", ROWS), ROWS),    # digits of 12: the last size with a column launch
    (26, 4, 2, 25, 34, ("hmult", WHOLE), ROWS),     # digits of 13: separate passes
    (26, 4, 2, 11, 4, ("hoisted", ROWS), ROWS),     # a level whose only digit has 12 primes
    (10, 2, 5, 9, 50, ("hoisted", WHOLE), ROWS),    # five digits: finished rows go through separate passes
    (16, 13, 4, 15, 100, ("hoisted", ROWS), WHOLE),  # ModDown from 13 primes has no column launch
])
def test_launches_are_timed_where_and_as_they_are_made(nq, K, dnum, level, modup, op, down):
    got = tune.op_launches(_Ctx(nq, K, dnum), level)
    assert got == {modup: op, 2 * (level + 1): ("hmult", down), 2 * level: ("rescale", ROWS)}
    assert tune.op_launch_sizes(_Ctx(nq, K, dnum), level) == {"ntt_fwd": sorted(got)}


def test_limits_are_the_librarys():
    mod = open(os.path.join(CSRC, "modarith.h")).read()
    assert int(re.search(r"kFoldMaxTerms = (\d+);", mod).group(1)) == tune.COLUMN_SOURCES
    assert "if (!cols16_fits(ns) || (finish && s.beta > %d)) {" % tune.FINISHED_DIGITS in open(os.path.join(CSRC, "api.cpp")).read()
    assert "bool cols16_fits(uint32_t ns) { return ns <= kFoldMaxTerms; }" in open(os.path.join(CSRC, "ntt.hip")).read()


def test_cache_of_other_launches_is_not_used(monkeypatch):
    key = tune._key(16, 74, 4, "ntt_fwd", "gfx950")
    assert key != "logN=16|limbs=74|K=4|op=ntt_fwd|arch=gfx950"
    monkeypatch.setattr(tune, "LAUNCHES", tune.LAUNCHES + 1)
    assert tune._key(16, 74, 4, "ntt_fwd", "gfx950") != key


def test_kinds_of_launch_have_codes_of_their_own():
    """A width for whole transforms leaves the row passes next to a column launch
    on their own rule; ckks_ntt_tile_set sets both."""
    try:
        ckks.ntt_tile_set_kind(WHOLE, False, 60, 4)
        assert ckks.ntt_tile_get(False, 60) == ckks.ntt_tile_get_kind(WHOLE, False, 60) == 4
        assert ckks.ntt_tile_get_kind(ROWS, False, 60) == 8
        ckks.ntt_tile_set_kind(ROWS, False, 60, 16)
        assert ckks.ntt_tile_get_kind(WHOLE, False, 60) == 4 and ckks.ntt_tile_get_kind(ROWS, False, 60) == 16
        ckks.ntt_tile_set(False, 60, 8)
        assert ckks.ntt_tile_get_kind(WHOLE, False, 60) == ckks.ntt_tile_get_kind(ROWS, False, 60) == 8
    finally:
        ckks.ntt_tile_set(False, 60, 0)
    assert [ckks.ntt_tile_get_kind(k, False, n) for k in (WHOLE, ROWS) for n in (7, 8)] == [8, 16, 4, 8]
    assert [ckks.ntt_tile_get_kind(k, True, n) for k in (WHOLE, ROWS) for n in (8, 9)] == [2, 16, 2, 8]
    for kind, inverse, n, tile in [(2, 0, 8, 8), (ROWS, 0, 8, 2), (WHOLE, 0, 129, 8), (ROWS, 0, 0, 8), (ROWS, 0, 8, 5)]:
        with pytest.raises(ckks.CkksError):
            ckks.ntt_tile_set_kind(kind, bool(inverse), n, tile)
