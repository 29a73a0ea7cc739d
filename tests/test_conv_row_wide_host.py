"""Host-side check of the base conversions whose sums take exact 128 bits
(conv_row.h, modarith.h): 1 to 16 source primes just below 2^61 into targets of
51 and 61 bits, plain and shifted inputs at their limits."""
import os
import subprocess

import pytest

from paper_2507_04775_amd import inputs

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("conv") / "check")
    subprocess.check_call(["/opt/rocm/bin/hipcc", "-O2", "-std=c++17", os.path.join(HERE, "host", "conv_row_wide_check.cpp"),
                           "-o", out], stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    return out


@pytest.mark.parametrize("target_bits", [51, 61])
def test_wide_sums_are_exact(exe, target_bits):
    big = inputs.ntt_primes(61, 17, 16)
    target = big[16] if target_bits == 61 else inputs.ntt_primes(target_bits, 1, 16)[0]
    r = subprocess.run([exe, str(target)] + [str(p) for p in big[:16]], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.strip().endswith("ok")
