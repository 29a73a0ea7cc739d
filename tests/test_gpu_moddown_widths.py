"""ModDown from 13 special primes at N = 2^16 (no column launch) on both sides of
its tile widths' line at 24 limbs, bit for bit against the oracle."""
import pytest

import oracle
from gpu_common import assert_equal, gpu_available
from paper_2507_04775_amd import inputs

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("level", [0, 7, 23, 24])
def test_moddown_of_13_special_primes(level):
    import torch
    from paper_2507_04775_amd import ckks
    big = inputs.ntt_primes(60, 14, 16)
    q, p = [big[0]] + inputs.ntt_primes(50, 24, 16), big[1:]
    P, ctx = oracle.Params(16, q, p, 2), ckks.Context(16, q, p, 2)
    x = inputs.uniform_residues(inputs.rng(level), P.row_moduli(level), 1 << 16)
    out = ctx.empty_poly(level)
    ctx.ckks_moddown(ckks.to_device(x), level, out)
    torch.cuda.synchronize()
    assert_equal(ckks.to_host(out), oracle.moddown(P, x, level), "moddown level %d" % level)
    ctx.close()
