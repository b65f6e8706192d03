"""The host threads of the batched eigenproblems (csrc/host_parallel.hpp), compiled here with the host compiler."""

import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_15775_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <new>
#include "host_parallel.hpp"
int main() {
  for (int count : {0, 1, 3, 4, 7, 8, 33, 1000}) {
    std::vector<std::atomic<int>> calls(count);
    if (!almbm::host_parallel(count, [&](int t) { calls[t]++; })) return 1;
    for (auto& c : calls)
      if (c != 1) return 2;
  }
  for (int bad : {0, 5, 63}) {  // on the caller's thread or on another
    std::vector<std::atomic<int>> calls(64);
    if (almbm::host_parallel(64, [&](int t) {
          calls[t]++;
          if (t >= bad) throw std::bad_alloc();
        }))
      return 3;
    for (auto& c : calls)
      if (c > 1) return 4;
  }
  std::puts("ok");
  return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_every_call_once_and_exceptions_stay_inside(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++20", "-O1", "-pthread", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout.strip() == "ok", (out.returncode, out.stderr)
