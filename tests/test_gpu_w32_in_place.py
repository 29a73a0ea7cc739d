"""Rotations and conjugation of the 32-bit word path whose outputs overlap their
input: exactly in place, swapped, one half only, and shifted by a limb, bit for
bit against the oracle.  The addend phi_g(c0) is gathered across the whole limb,
so it has to be out of the outputs' way before they are written."""
import pytest

import oracle
from gpu_common import assert_equal, gpu_available
from paper_2507_04775_amd import inputs

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

# where (out0, out1) lie: "a", "b" are c0's and c1's buffers, "a1" c0's shifted by one limb, "x", "y" others
LAYOUTS = [("a", "b"), ("b", "a"), ("x", "a"), ("a", "x"), ("a1", "x"), ("x", "a1"), ("x", "b"), ("x", "y")]


@pytest.mark.parametrize("level", [7, 0])
@pytest.mark.parametrize("g", [1, pow(5, 321, 2 << 16), (2 << 16) - 1])
def test_galois_outputs_may_overlap_the_input(g, level):
    import torch
    from paper_2507_04775_amd import ckks
    ps = inputs.params32("w32-small")
    P, ctx = oracle.Params(ps.logn, ps.q, ps.p, ps.dnum), ckks.Context32(ps.logn, ps.q, ps.p, ps.dnum)
    key, c, n = inputs.random_key(5 + g % 1000, ps), inputs.random_ct(level, ps, level), level + 1
    kd = ckks.to_device32(key.reshape(-1, ps.N)).reshape(key.shape)
    want = oracle.apply_galois(P, c, g, key, level)
    for layout in LAYOUTS:
        buf = {k: ctx.empty(n + 1) for k in "abxy"}
        place = {k: v[:n] for k, v in buf.items()}
        place["a1"] = buf["a"][1:]
        for k, half in zip("ab", c):
            place[k].copy_(ckks.to_device32(half))
        out = [place[k] for k in layout]
        ctx.apply_galois(place["a"], place["b"], level, g, kd, *out)
        torch.cuda.synchronize()
        for i in range(2):
            assert_equal(ckks.to_host32(out[i]), want[i], "galois %d into %s, half %d" % (g, layout, i))
    ctx.close()
