"""Host rules of the library that need no device, compiled from its headers."""

import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2009_12009_amd", "csrc")

TAIL = r"""
#include <cstdio>
#include "host.hpp"
int main() {
  const std::vector<long long> halved = {1ll << 30, 1ll << 27, 1ll << 24, 1ll << 21, 1ll << 18,
                                         1ll << 15, 1ll << 12, 1ll << 9, 1ll << 6, 8};
  auto f = [&](int lo, long long limit) {
    std::printf("%d ", amrmg::first_tail_level(halved, lo, limit, 6));
  };
  f(1, 0);            // nothing small enough
  f(1, 64);           // one level above the bottom
  f(1, 1024);
  f(1, 1ll << 40);    // everything is: no more than the tables hold
  f(2, 1ll << 40);
  f(8, 1ll << 40);    // not before lo
  f(9, 1ll << 40);
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")
def test_tail_levels_stay_within_the_tables(tmp_path):
    src = tmp_path / "tail.cpp"
    src.write_text(TAIL)
    exe = tmp_path / "tail"
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()
    assert [int(x) for x in out] == [-1, 8, 7, 3, 3, 8, -1]
