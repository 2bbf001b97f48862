"""The slabs a work-group of the persistent GEMM loads, walked on the CPU with the kernel's own cursor
(csrc/gemm_cursor.h): every row of a tile that exists is fetched at every slab, and no lane that the buffer's range check
lets through reads past the operand, up to the loads after the last tile that are issued for the waits to count.  The
check lets a lane through whose offset is below size - scalar offset, taken without a sign."""
import ctypes
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_04802_amd", "csrc")
WALK = r"""
#include <cstdint>
#include "gemm_cursor.h"
// panels of one operand: `count` of them, `panel` rows each, `rows` rows of K in all; one tile per panel in the list.
// 0, or what went wrong: 1 a lane reads past the operand, 2 a row that exists is not read, 3 a load past the last tile reads
extern "C" int walk(int rows, int K, int panel, int work_groups) {
  const int count = (rows + panel - 1) / panel, nk = K / 64;
  const int64_t end = static_cast<int64_t>(rows) * K * 2;
  for (int slot = 0; slot < work_groups && slot < count; ++slot) {
    reslim::SlabCursor at{slot, 0, nk, count, work_groups};
    // the loads run two slabs ahead of the multiplication: two slabs past the work-group's last one
    const int own = (count - slot + work_groups - 1) / work_groups;
    for (int s = 0; s < own * nk + 2; ++s, at.next()) {
      const bool exists = at.tile < count;
      if (exists != (s < own * nk)) return 4;
      const int first = exists ? at.tile * panel : 0;
      const uint32_t size = at.buffer_bytes(first, panel, rows, K), off = at.scalar_offset();
      for (int r = 0; r < panel; ++r)
        for (uint32_t c = 0; c < 128; c += 16) {
          const uint32_t lane = static_cast<uint32_t>(r) * K * 2 + c;
          if (lane < size - off) {
            if (!exists) return 3;
            if (static_cast<int64_t>(first) * K * 2 + lane + off + 16 > end) return 1;
          } else if (exists && first + r < rows) {
            return 2;
          }
        }
    }
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    d = tmp_path_factory.mktemp("walk")
    src, so = d / "walk.cpp", d / "walk.so"
    src.write_text(WALK)
    cxx = shutil.which("g++") or shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so)).walk


@pytest.mark.parametrize("K", [64, 128, 192, 512])
@pytest.mark.parametrize("rows", [1, 32, 64, 100, 127, 128, 129, 255, 256, 257, 700, 1000])
def test_loads_stay_in_the_operand(walk, rows, K):
    for panel in (128, 256):
        for work_groups in (1, 2, 3, 256):
            assert walk(rows, K, panel, work_groups) == 0, (panel, work_groups)
