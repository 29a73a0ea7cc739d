"""Host-side check of the base conversions' constant rows and sums (conv_row.h,
modarith.h) on the CPU: FoldSum's two columns and MacSplit's four against exact
128-bit sums, for 1 to 16 source rows of 30 to 61 bits, plain and shifted
inputs at their limits, and targets of 20 to 50 bits."""
import os
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))


def test_conversion_rows_and_sums_are_exact():
    src = os.path.join(HERE, "host", "conv_row_check.cpp")
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "convcheck")
        subprocess.check_call(["/opt/rocm/bin/hipcc", "-O2", "-std=c++17", "-ffp-contract=off", src, "-o", exe],
                              stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
        r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.strip().endswith("ok")
