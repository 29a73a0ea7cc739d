"""Host logic of the autotuner: every launch size is timed through an operation
that has a launch of that size, and results measured on other launches are not
taken from the cache.  No GPU."""
import os
import re

import pytest

from paper_2507_04775_amd import tune

CSRC = os.path.join(os.path.dirname(os.path.abspath(tune.__file__)), "csrc")


class _Ctx:
    logn = 16

    def __init__(self, nq, K, dnum):
        self.nq, self.np, self.alpha = nq, K, -(-nq // dnum)

    def beta(self, level):
        return -(-(level + 1) // self.alpha)


@pytest.mark.parametrize("nq,K,dnum,level,modup,op", [
    (31, 4, 3, 30, 74, "hoisted"),   # HMult finishes ModUp's rows inside its inner product
    (31, 4, 3, 12, 21, "hoisted"),
    (24, 4, 2, 23, 32, "hoisted"),   # digits of 12: the last size with a column launch
    (26, 4, 2, 25, 34, "hmult"),     # digits of 13: separate passes
    (26, 4, 2, 11, 4, "hoisted"),    # a level whose only digit has 12 primes
])
def test_modup_is_timed_where_it_is_launched(nq, K, dnum, level, modup, op):
    got = tune.op_launches(_Ctx(nq, K, dnum), level)
    assert got == {modup: op, 2 * (level + 1): "hmult", 2 * level: "rescale"}
    assert tune.op_launch_sizes(_Ctx(nq, K, dnum), level) == {"ntt_fwd": sorted(got)}


def test_column_launch_limit_is_the_librarys():
    mod = open(os.path.join(CSRC, "modarith.h")).read()
    assert int(re.search(r"kFoldMaxTerms = (\d+);", mod).group(1)) == tune.COLUMN_SOURCES
    assert "bool cols16_fits(uint32_t ns) { return ns <= kFoldMaxTerms; }" in open(os.path.join(CSRC, "ntt.hip")).read()


def test_cache_of_other_launches_is_not_used(monkeypatch):
    key = tune._key(16, 74, 4, "ntt_fwd", "gfx950")
    assert key != "logN=16|limbs=74|K=4|op=ntt_fwd|arch=gfx950"
    monkeypatch.setattr(tune, "LAUNCHES", tune.LAUNCHES + 1)
    assert tune._key(16, 74, 4, "ntt_fwd", "gfx950") != key
