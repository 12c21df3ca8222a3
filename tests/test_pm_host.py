"""Host check of the signed transforms' arithmetic (modarith.h: pm_mul,
pm_red, pm_canon; pm_form.h) and of the bounds that the passes rely on: the
headers compiled as plain C++ and run against exact 128-bit arithmetic, for
the workloads' primes, others of 50 to 60 bits, and the largest delta and
d60 that the form accepts."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CXX = "/opt/rocm/llvm/bin/clang++" if os.path.exists("/opt/rocm/llvm/bin/clang++") else shutil.which("clang++")

# 60-bit workload primes; 2^60 - delta with delta just below 2^24 (any odd
# modulus serves: nothing here needs a prime); 55, 50 and 40 bits, the last
# with d60 just below 2^31
MODULI = [1152921504606830593, 1152921504606748673, 1152921504606683137, 2 ** 60 - 2 ** 24 + 1, 2 ** 55 - 2 ** 24 + 3,
          1125899906826241, 2 ** 50 - 2 ** 21 + 1, 2 ** 40 - 2 ** 11 + 1]


@pytest.fixture(scope="module")
def pm_bin(tmp_path_factory):
    if CXX is None:
        pytest.skip("no clang++ for the host build")
    out = str(tmp_path_factory.mktemp("pm") / "pm_host")
    subprocess.run([CXX, "-O2", "-std=c++17", "-I",
                    os.path.join(HERE, "host_shim"), "-I", os.path.join(ROOT, "paper_2506_11586_amd", "csrc"),
                    os.path.join(HERE, "pm_host.cpp"), "-o", out], check=True)
    return out


@pytest.mark.parametrize("q", MODULI)
def test_signed_transform_arithmetic(pm_bin, q):
    r = subprocess.run([pm_bin, str(q), "400000"], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr
