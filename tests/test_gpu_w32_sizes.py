"""The 32-bit word path over digits and special bases of 1 to 16 primes and 1 to
15 digits, the limits of its 64-bit sums, with maximal and uniform residues:
HMult, rotation and Rescale at the top level, bit for bit against the oracle."""
import numpy as np
import pytest

import oracle
from gpu_common import assert_equal, gpu_available
from paper_2507_04775_amd import inputs

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("nq,K,dnum", [(1, 1, 1), (2, 1, 2), (5, 3, 2), (16, 16, 1), (13, 16, 1), (15, 2, 15), (17, 9, 2)])
def test_hmult_rotate_rescale_at_the_limits(nq, K, dnum):
    import torch
    from paper_2507_04775_amd import ckks
    pr = inputs.ntt_primes(30, nq + K, 16)
    ps = inputs.ParamSet("w32", 16, pr[:nq], pr[nq:], dnum, 26)
    P, ctx = oracle.Params(16, ps.q, ps.p, dnum), ckks.Context32(16, ps.q, ps.p, dnum)
    level, g = nq - 1, pow(5, 321, 2 * ps.N)
    key = inputs.random_key(nq + K, ps)
    top_key = np.broadcast_to(np.array([m - 1 for m in pr], dtype=np.uint64)[None, None, :, None], key.shape).copy()
    top = np.array([[m - 1] * ps.N for m in ps.q], dtype=np.uint64)
    dev = ckks.to_device32

    def host(ts):
        torch.cuda.synchronize()
        return [ckks.to_host32(t) for t in ts]

    for k, a, b in ((key, inputs.random_ct(1, ps, level), inputs.random_ct(2, ps, level)), (top_key, (top, top), (top, top))):
        kd, da, db = dev(k.reshape(-1, ps.N)).reshape(k.shape), [dev(x) for x in a], [dev(x) for x in b]
        out = [ctx.empty(nq), ctx.empty(nq)]
        ctx.hmult_relin(*da, *db, level, kd, *out)
        for got, want in zip(host(out), oracle.hmult_relin(P, a, b, k, level)):
            assert_equal(got, want, "hmult")
        ctx.apply_galois(*da, level, g, kd, *out)
        for got, want in zip(host(out), oracle.apply_galois(P, a, g, k, level)):
            assert_equal(got, want, "rotation")
        if level:
            low = [ctx.empty(level), ctx.empty(level)]
            ctx.rescale(*da, level, *low)
            for got, want in zip(host(low), oracle.rescale(P, a, level)):
                assert_equal(got, want, "rescale")
    ctx.close()
