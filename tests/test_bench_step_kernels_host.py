"""Host check of the bench line's step kernels (CPU): the committed counter
summary names the launches of HMult+relin and the rotation's inner product, with
the algorithmic bytes that follow from their operands, and the bench reads it."""
import os

from test_bench_host import ROOT, _bench

LIMB = 65536 * 8
PROFILE = os.path.join(ROOT, "profiles", "step_kernels_logn16_l30_hbm_counters.md")


def test_step_kernels_and_their_bytes():
    # l = 30, K = 4: 31 rows, digits of 11, 11 and 9, 74 converted rows, 35 extended rows
    want = {
        "k_inv_row_tensor": (2 * 31 + 31) * LIMB,            # a1, b1 read, ModUp's input written
        "k16_cols<0>": (31 + 74) * LIMB,                     # sources read, converted rows written
        "k16_ip_rows<1>": (31 * (2 + 6 + 4) + 4 * (3 + 6) + 2 * 35) * LIMB,
        "k16_cols<1>": (8 + 62) * LIMB,
        "k_fwd_row_moddown": 3 * 62 * LIMB,                  # converted rows, sums, outputs
        "k16_ip_rows<0>": (35 * (3 + 6) + 2 * 35) * LIMB,
    }
    got = {}
    for line in open(PROFILE).read().splitlines():
        if line.startswith("step_kernel:"):
            name, _, *kv = line.split(":", 1)[1].split()
            f = dict(x.split("=") for x in kv)
            got[name.replace("_w8", "").replace("_w4", "")] = int(f["algorithmic_bytes"])
            assert int(f["traffic_bytes"]) >= int(f["algorithmic_bytes"]) and float(f["avg_us"]) > 0
    assert got == want


def test_bench_reads_them():
    out = _bench().step_inner_products()
    if out is not None:  # None while the kernel sources differ from the profiled ones
        assert len(out) == 6 and all(0.0 < e["frac"] < 1.0 and e["traffic"] > 0 for e in out)
