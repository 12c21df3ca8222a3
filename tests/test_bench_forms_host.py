"""Host checks of the transforms' rooflines that bench.py prints: the ceiling is
that of the butterfly that the context's primes take, and which form that is
follows the library's own rule (csrc/pm_form.h)."""
import os
import re
import shutil
import subprocess

import pytest

import bench
import oracle
from tests.test_bench_host import _grids

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CXX = "/opt/rocm/llvm/bin/clang++" if os.path.exists("/opt/rocm/llvm/bin/clang++") else shutil.which("clang++")


@pytest.mark.parametrize("signed,inv,fwd", [(False, 21, 21), (True, 296 / 24, 272 / 24)])
def test_transform_ceiling_follows_the_form(signed, inv, fwd):
    kavg, alg = _grids(6.0, 84.0, 119.0)
    roof, _, _, ntt = bench.headline_rooflines(kavg, alg, {"grid": 1, "lds": 3}, None, lambda k: None, signed)
    assert roof is ntt["batch_inv"]
    for k, insts in (("batch_inv", inv), ("batch_fwd", fwd)):
        assert abs(ntt[k]["peak"] - 256 * 64 * 2.4 / insts) < 0.1
        assert abs(ntt[k]["frac"] - ntt[k]["achieved"] / ntt[k]["peak"]) < 1e-3
        assert ("signed" in ntt[k]["peak_derivation"]) == signed


def test_form_rule_is_the_librarys(tmp_path):
    if CXX is None:
        pytest.skip("no clang++ for the host build")
    qs = [q for N in (1024, 8192, 16384) for b in (36, 40, 45, 50, 55, 60) for q in oracle.find_primes(N, b, 3)]
    qs += [2 ** 60 - 2 ** 24 + 1, 2 ** 60 - 2 ** 24 - 1, 2 ** 40 - 2 ** 11 + 1, 2 ** 40 - 2 ** 11 - 1, 2 ** 59 + 2 ** 57 + 1,
           2 ** 34 - 1, 2 ** 33 - 1, 2 ** 60 - 1]
    src, out = tmp_path / "form.cpp", tmp_path / "form"
    src.write_text('#include <cstdio>\n#include "pm_form.h"\nint main() {\n' +
                   "".join(f'  std::printf("%d", (int)heconv::pm_form({q}ull).ok);\n' for q in qs) + "}\n")
    subprocess.run([CXX, "-O1", "-std=c++17", "-I", os.path.join(ROOT, "tests", "host_shim"), "-I",
                    os.path.join(ROOT, "paper_2506_11586_amd", "csrc"), str(src), "-o", str(out)], check=True)
    got = subprocess.run([str(out)], capture_output=True, text=True, check=True).stdout
    assert got == "".join(str(int(bench.signed_form([q]))) for q in qs)
    assert "0" in got and "1" in got
    assert bench.signed_form(qs[:0]) and not bench.signed_form([qs[-1], 2 ** 59 + 2 ** 57 + 1])


def test_instruction_counts_are_the_probes():
    """The counts are those of the compiled loops of the butterfly probes."""
    from paper_2506_11586_amd import build
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    asm = subprocess.run([build.HIPCC, *flags, "-I", os.path.join(ROOT, "include"), "-I", build.CSRC, "-S",
                          "--cuda-device-only", os.path.join(build.CSRC, "probe.hip"), "-o", "-"], check=True,
                         capture_output=True, text=True).stdout
    for kernel, per, table in (("probe_pass_kernel", 24, bench.BFLY_VALU_INSTS_SIGNED),
                               ("probe_bfly_kernel", 32, bench.BFLY_VALU_INSTS)):
        for inverse, name in ((1, "batch_inv"), (0, "batch_fwd")):
            body = re.search(r"^_ZN\S*%sILb%d\S*:.*?\n(.*?)s_endpgm" % (kernel, inverse), asm, re.S | re.M).group(1)
            loop = max(len(re.findall(r"^\tv_", b, re.M)) for b in re.split(r"\n(?=\.LBB)", body))
            assert loop == round(table[name] * per), (kernel, name)
