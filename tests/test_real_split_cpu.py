"""The work split of the real-space kernel (host rule, compiled with g++).

Which of the two scans a system gets, and how many work-groups: a work-group of
four wavefronts per charge (grids with far more cells than charges), few blocks
for the one member of a batch, and a share's whole neighbourhood staged for a
handful of charges were all slower than a wavefront per charge.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADERS = ["-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_1303_4523_amd", "csrc"),
           "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include"]

PROGRAM = r"""
#include "enuf_internal.h"
#include <cstdio>
#include <cstdlib>
using namespace enuf;
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s (n %d nq %d blocks %d)\n", __LINE__, #x, n, nq, blocks); \
                                  std::exit(1); } } while (0)
int main() {
  for (int blocks : {0, kRealTargetBlocks / kRealBatchMembers, kRealDpdBlocks, kRealTargetBlocks})
    for (int n = 1; n <= 40; ++n) {
      bool wave = true;
      for (int nq = 0; nq <= 300 * n * n * n && nq <= 400000; nq += 1 + nq / 40) {
        const RealSplit s = real_split(nq, n, blocks, blocks);
        // a scan taken for some count is taken for every smaller one
        CHECK(wave || !s.wave);
        wave = s.wave;
        if (s.wave) CHECK(s.items == (nq + 3) / 4);
        // fewer than 2 charges per cell never take a work-group each
        if (nq < 2 * n * n * n) CHECK(s.wave);
        if (s.wave) continue;
        // segments cover the column, a share its part of a cell, within the block's charges
        CHECK(s.seg >= 1 && s.seg <= kRealSegMax && s.seg <= n && s.nseg * s.seg >= n && (s.nseg - 1) * s.seg < n);
        CHECK(s.group >= 1 && s.group <= kRealOwn && s.shares >= 1 && (s.seg == 1 || s.shares == 1));
        CHECK(s.items == n * n * s.nseg * s.shares);
      }
      // 3 and 4 cells per side: no shares of a few charges beside the whole box as candidates
      const int nq = 60 * n * n * n;
      if (blocks == kRealTargetBlocks && (n == 3 || n == 4)) CHECK(real_split(nq, n, blocks, blocks).wave);
      if (n >= 7) CHECK(!real_split(nq, n, blocks, blocks).wave);
    }
  return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"), reason="no host toolchain")
def test_real_split(tmp_path):
    src = tmp_path / "split.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "split"
    subprocess.run(["g++", "-std=c++17", "-O1", *HEADERS, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
