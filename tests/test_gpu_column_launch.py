"""N = 2^16 key switching where its route changes: ModUp's tiles read by the
inner product (up to 12 primes a digit, any number of digits), finished rows
from tiles (up to 4 digits) or from separate passes (more), the separate passes
throughout (13 primes a digit, 13 special primes); and Rescale from level 1 up.
Bit for bit against the oracle."""
import numpy as np
import pytest

import oracle
from gpu_common import assert_equal, gpu_available
from paper_2507_04775_amd import inputs

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]
LOGN = 16


# alpha = nq / dnum; the top levels: 4 and 5 digits, one-prime digits, 12 and 13 primes a digit
@pytest.mark.parametrize("nq,K,dnum,level", [(8, 2, 4, 7), (10, 2, 5, 9), (5, 1, 5, 4), (5, 1, 5, 0), (14, 12, 2, 13),
                                             (24, 12, 2, 23), (14, 13, 1, 13), (14, 13, 1, 11)])
def test_key_switching_ops(nq, K, dnum, level):
    import torch
    from paper_2507_04775_amd import ckks
    big = inputs.ntt_primes(60, 1 + K, LOGN)
    ps = inputs.ParamSet("cols", LOGN, [big[0]] + inputs.ntt_primes(50, nq - 1, LOGN), big[1:], dnum, 40)
    P, ctx = oracle.Params(LOGN, ps.q, ps.p, dnum), ckks.Context(LOGN, ps.q, ps.p, dnum)
    a, b = (inputs.random_ct(s, ps, level) for s in (1, 2))
    ta, tb = (ckks.Ciphertext(ckks.to_device(x), ckks.to_device(y), level, 1.0) for x, y in (a, b))

    def check(out, want, what):
        torch.cuda.synchronize()
        assert_equal(ckks.to_host(out.c0), want[0], what + " c0")
        assert_equal(ckks.to_host(out.c1), want[1], what + " c1")

    rlk, out = inputs.random_key(3, ps), ctx.empty_ct(level)
    kh = ctx.key(ckks.to_device(rlk), 0)
    ctx.ckks_hmult_relin(ta, tb, kh, out)
    check(out, oracle.hmult_relin(P, a, b, rlk, level), "hmult")
    rots = [1, 5]
    gs = [oracle.galois_for_rotation(LOGN, k) for k in rots]
    keys = [inputs.random_key(4 + i, ps) for i in range(2)]
    khs = [ctx.key(ckks.to_device(k), g) for k, g in zip(keys, gs)]
    outs = [ctx.empty_ct(level) for _ in rots]
    ctx.ckks_hrotate(ta, rots[1], khs[1], out)
    check(out, oracle.apply_galois(P, a, gs[1], keys[1], level), "rotation")
    ctx.ckks_hrotate_hoisted(ta, rots, khs, outs)
    w0, w1 = oracle.hoisted_rotate(P, a, gs, keys, level)
    for i, k in enumerate(rots):
        check(outs[i], (w0[i], w1[i]), "hoisted rotation %d" % k)
    ctx.close()


@pytest.mark.parametrize("level", [1, 2, 8, 9, 17])
def test_rescale(level):
    import torch
    from paper_2507_04775_amd import ckks
    big = inputs.ntt_primes(60, 3, LOGN)
    ps = inputs.ParamSet("cols", LOGN, [big[0]] + inputs.ntt_primes(50, 17, LOGN), big[1:], 9, 40)
    P, ctx = oracle.Params(LOGN, ps.q, ps.p, 9), ckks.Context(LOGN, ps.q, ps.p, 9)
    c = inputs.random_ct(level, ps, level)
    c[0][level, ::3] = ps.q[level] - 1  # the lift's ends
    c[1][level, ::5] = 0
    out = ctx.empty_ct(level - 1)
    ctx.ckks_rescale(ckks.Ciphertext(ckks.to_device(c[0]), ckks.to_device(c[1]), level, 1.0), out)
    want = oracle.rescale(P, c, level)
    torch.cuda.synchronize()
    assert_equal(ckks.to_host(out.c0), want[0], "rescale c0")
    assert_equal(ckks.to_host(out.c1), want[1], "rescale c1")
    ctx.close()
