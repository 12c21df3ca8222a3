"""Host check of the transforms' exchange chain: NTT-form words are stored
and loaded in the mapping at bit 6, every exchange starts in the mapping in
which the one before ended (each thread then overwrites only entries that it
read itself, so one barrier orders a cross-wave exchange), and the padded
LDS index of an element is that of the thread's part plus that of the
register's, within the array, with no two elements at one place.  Also the
twiddle tables' order (csrc/tw_layout.h): every entry of a stage has a place of
its own, and a stage read by lanes of different blocks puts the entries of 64
consecutive blocks side by side."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CXX = "/opt/rocm/llvm/bin/clang++" if os.path.exists("/opt/rocm/llvm/bin/clang++") else shutil.which("clang++")


def elem(loge, lo, t, k):
    return (t & ((1 << lo) - 1)) | (k << lo) | ((t >> lo) << (lo + loge))


def pad(j):
    return j + (j >> 4)


def passes(logn, loge):
    return [logn - loge * (p + 1) for p in range(logn // loge)] + ([0] if logn % loge else [])


def chain(mappings):
    return list(zip(mappings, mappings[1:]))


@pytest.mark.parametrize("logn", range(10, 15))
@pytest.mark.parametrize("loge", [3, 4])
def test_exchange_chain(logn, loge):
    threads, e = (1 << logn) >> loge, 1 << loge
    if threads > 1024:
        pytest.skip("more threads than a workgroup holds: not instantiated")
    fwd = passes(logn, loge) + [6]
    for seq in (chain(fwd), chain(fwd[::-1])):
        for (_, to), (frm, _) in zip(seq, seq[1:]):
            assert to == frm
        for frm, to in seq:
            for lo in (frm, to):
                words = [elem(loge, lo, t, k) for t in range(threads) for k in range(e)]
                assert sorted(words) == list(range(1 << logn))
                at = [pad(elem(loge, lo, t, 0)) + pad(k << lo) for t in range(threads) for k in range(e)]
                assert at == [pad(w) for w in words]
                assert max(at) < (1 << logn) + (1 << logn) // 16
            if frm <= 6 and to <= 6:  # wave-local: each wave's own block on both sides
                for w in range(threads // 64):
                    ts = range(64 * w, 64 * w + 64)
                    block = set(range(w * 64 * e, (w + 1) * 64 * e))
                    assert {elem(loge, frm, t, k) for t in ts for k in range(e)} == block
                    assert {elem(loge, to, t, k) for t in ts for k in range(e)} == block


TABLE_CHECK = """
#include <cstdio>
#include <vector>
#include "tw_layout.h"
int main() {
  for (int n = 10; n <= 14; n++)
    for (int s = 0; s < n; s++) {
      std::vector<int> seen(1u << s, 0);
      const int u = heconv::tw_u(n, s);
      if (u > s) return std::printf("u %d %d", n, s), 1;
      for (unsigned i = 0; i < 1u << s; i++) {
        const unsigned p = heconv::tw_place(n, s, i);
        if (p < 1u << s || p >= 2u << s || seen[p - (1u << s)]++) return std::printf("place %d %d %u", n, s, i), 1;
        if (u && (i >> u) % 64 && p != heconv::tw_place(n, s, i - (1u << u)) + 1) return std::printf("run %d %d", n, s), 1;
      }
    }
  std::printf("ok");
}
"""


def test_twiddle_places(tmp_path):
    if CXX is None:
        pytest.skip("no clang++ for the host build")
    src, out = tmp_path / "tw.cpp", tmp_path / "tw"
    src.write_text(TABLE_CHECK)
    subprocess.run([CXX, "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2506_11586_amd", "csrc"), str(src), "-o",
                    str(out)], check=True)
    r = subprocess.run([str(out)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout == "ok", r.stdout
