"""Host check of the compiled key-switching inner product (csrc/rotate.hip):
its operands come from beyond L2, so a term's loads have to be in flight
together.  The compiler, held to 64 registers, once waited for each pair of
words before it issued the next: rotation of a few ciphertexts at N = 2048 took
a tenth longer for it (four digits: a fifth).  Counted in the assembly: the
buffer loads issued and not yet waited for."""
import os
import re
import subprocess

import pytest

from paper_2506_11586_amd import build

MIN_IN_FLIGHT = 8  # four points' digit and key words


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    out = str(tmp_path_factory.mktemp("ks") / "rotate.s")
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    subprocess.run([build.HIPCC, *flags, "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, "-S",
                    "--cuda-device-only", os.path.join(build.CSRC, "rotate.hip"), "-o", out], check=True,
                   capture_output=True)
    with open(out) as f:
        return f.read()


def most_in_flight(code):
    most = pending = 0
    for line in code.splitlines():
        op = line.split(";")[0].strip()
        if op.startswith("buffer_load"):
            pending += 1
            most = max(most, pending)
        elif op.startswith("s_waitcnt") and (m := re.search(r"vmcnt\((\d+)\)", op)):
            pending = min(pending, int(m.group(1)))
    return most


@pytest.mark.parametrize("logn", [10, 11, 12, 13])
def test_general_inner_product_keeps_loads_in_flight(assembly, logn):
    # inner_intt_kernel<logn, PM = false, ...>
    m = re.search(r"^_ZN6heconv17inner_intt_kernelILi%dELb0E\S*:.*?\n(.*?)s_endpgm" % logn, assembly, re.S | re.M)
    assert m, "kernel not found"
    assert most_in_flight(m.group(1)) >= MIN_IN_FLIGHT
