"""The library's process-wide host tables are made once, also when the first calls
come from several threads at once (contexts are per thread, these tables are not):
the header that holds them, built for the CPU under the thread sanitizer."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2304_11002_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <thread>
#include <vector>
#include "stencil_pairs.h"
int main() {
  const uint32_t masks[4] = {fmm::kFullMask, 1u << fmm::kCentreBit, 0x0000ffffu, 0x07ffe000u};
  int64_t got[8][4];
  std::vector<std::thread> ts;
  for (int t = 0; t < 8; ++t)
    ts.emplace_back([&, t] {
      for (int m = 0; m < 4; ++m) got[t][m] = fmm::pairs_of_mask(masks[(m + t) % 4]);
    });
  for (auto& t : ts) t.join();
  int64_t centre = 0;   // pairs whose source is in the target block, counted directly
  const std::vector<int>& s = fmm::stencil_host();
  for (size_t i = 0; i < s.size(); i += 3) {
    int64_t n = 1;
    for (int a = 0; a < 3; ++a) n *= 8 - (s[i + a] < 0 ? -s[i + a] : s[i + a]);
    centre += n;
  }
  for (int t = 0; t < 8; ++t)
    for (int m = 0; m < 4; ++m)
      if (got[t][m] != fmm::pairs_of_mask(masks[(m + t) % 4])) return 2;
  if (fmm::pairs_of_mask(fmm::kFullMask) != 512 * 892 || fmm::pairs_of_mask(1u << fmm::kCentreBit) != centre) return 3;
  std::puts("ok");
  return 0;
}
"""


def test_pair_counts_from_several_threads(tmp_path):
    src, exe = tmp_path / "threads.cpp", tmp_path / "threads"
    src.write_text(PROGRAM)
    flags = ["-std=c++17", "-O1", "-g", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I", "/opt/rocm/include"]
    r = subprocess.run(["g++", "-fsanitize=thread"] + flags + [str(src), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    if "unexpected memory mapping" in r.stderr:
        pytest.skip("the thread sanitizer does not run under this kernel's address layout")
    assert r.returncode == 0 and r.stdout == "ok\n" and "data race" not in r.stderr, r.stderr[-2000:]
