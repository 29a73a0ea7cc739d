"""Primes just below 2^61, the largest a context accepts, where the integer path's
lazy values come closest to 2^64 and ModDown's inputs reach 1.5 2^61: HMult,
rotation, hoisted rotation, key switch, ModDown and Rescale with maximal and
uniform residues and keys, bit for bit against the oracle.  wide "ends": q_0 and
the special primes (the rest of 49 bits); "all": every prime."""
import numpy as np
import pytest

import oracle
from gpu_common import assert_equal, gpu_available
from paper_2507_04775_amd import inputs

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("logn,nq,K,dnum,wide", [
    (12, 4, 1, 2, "all"), (12, 8, 4, 2, "all"), (12, 12, 12, 1, "all"), (12, 14, 13, 1, "ends"), (12, 16, 16, 1, "all"),
    (16, 4, 4, 2, "ends"), (16, 5, 4, 5, "all"), (16, 12, 12, 1, "all"), (16, 13, 13, 1, "all"), (16, 4, 16, 1, "ends")])
def test_largest_primes(logn, nq, K, dnum, wide):
    import torch
    from paper_2507_04775_amd import ckks
    if wide == "all":
        pr = inputs.ntt_primes(61, nq + K, logn)
        q, p = pr[:nq], pr[nq:]
    else:
        pr = inputs.ntt_primes(61, 1 + K, logn)
        q, p = [pr[0]] + inputs.ntt_primes(49, nq - 1, logn), pr[1:]
    ps = inputs.ParamSet("wide", logn, q, p, dnum, 40)
    P, ctx = oracle.Params(logn, q, p, dnum), ckks.Context(logn, q, p, dnum)
    level, N = nq - 1, ps.N
    g = [oracle.galois_for_rotation(logn, k) for k in (1, 5)]
    dev = ckks.to_device

    def same(got, want, what):
        torch.cuda.synchronize()
        for i, (x, w) in enumerate(zip(got, want)):
            assert_equal(ckks.to_host(x), w, "%s half %d" % (what, i))

    def ct(x):
        return ckks.Ciphertext(dev(x[0]), dev(x[1]), level, 1.0)

    def top(mods):
        return np.array([[m - 1] * N for m in mods], dtype=np.uint64)

    keys = [inputs.random_key(s, ps) for s in range(3)]
    top_key = np.broadcast_to(top(q + p)[None, None], keys[0].shape).copy()
    full = top(q)
    for what, a, b, ks in (("uniform", inputs.random_ct(1, ps, level), inputs.random_ct(2, ps, level), keys),
                           ("maximal", (full, full), (full, full), [top_key] * 3)):
        ta, tb, out = ct(a), ct(b), ctx.empty_ct(level)
        kh = [ctx.key(dev(k), e) for k, e in zip(ks, [0] + g)]
        ctx.ckks_hmult_relin(ta, tb, kh[0], out)
        same((out.c0, out.c1), oracle.hmult_relin(P, a, b, ks[0], level), what + " hmult")
        ctx.ckks_keyswitch(ta.c1, level, kh[0], out.c0, out.c1)
        same((out.c0, out.c1), oracle.keyswitch(P, a[1], ks[0], level), what + " keyswitch")
        ctx.ckks_hrotate(ta, 5, kh[2], out)
        same((out.c0, out.c1), oracle.apply_galois(P, a, g[1], ks[2], level), what + " rotation")
        outs = [ctx.empty_ct(level) for _ in g]
        ctx.ckks_hrotate_hoisted(ta, [1, 5], kh[1:], outs)
        w0, w1 = oracle.hoisted_rotate(P, a, g, ks[1:], level)
        for i in range(2):
            same((outs[i].c0, outs[i].c1), (w0[i], w1[i]), what + " hoisted %d" % i)
        ext = torch.empty((ctx.beta(level), nq + K, N), dtype=torch.uint64, device="cuda")
        ctx.ckks_modup(ta.c1, level, ext)
        same(ext, oracle.modup(P, a[1], level), what + " modup")
        rows = P.row_moduli(level)
        x = top(rows) if what == "maximal" else inputs.uniform_residues(inputs.rng(9), rows, N)
        down = ctx.empty_poly(level)
        ctx.ckks_moddown(dev(x), level, down)
        same((down,), (oracle.moddown(P, x, level),), what + " moddown")
        low = ctx.empty_ct(level - 1)
        ctx.ckks_rescale(ta, low)
        same((low.c0, low.c1), oracle.rescale(P, a, level), what + " rescale")
    ctx.close()
