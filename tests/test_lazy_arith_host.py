"""Host-side check of the integer NTT path's lazy butterflies (modarith.h) on
the CPU, against 128-bit arithmetic: product ranges, residues and word limits
for moduli up to 2^61 - 1."""
import os
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))


def test_lazy_butterflies_stay_in_range_and_exact():
    src = os.path.join(HERE, "host", "lazy_arith_check.cpp")
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "lazycheck")
        subprocess.check_call(["/opt/rocm/bin/hipcc", "-O2", "-std=c++17", src, "-o", exe],
                              stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
        r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.strip().endswith("ok")
