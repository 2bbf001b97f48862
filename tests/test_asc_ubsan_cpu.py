"""The quad-tree builder under the undefined-behaviour sanitizer: no overflow at any largest leaf that it accepts."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2505_04802_amd", "csrc")
DRIVE = r"""
#include <cmath>
#include <cstdio>
#include <vector>
#include "reslim.h"
// the tiled builder's, not called here
extern "C" int tiles_partition(int32_t, int32_t, int32_t, int32_t, int32_t, tile_desc *, int32_t *, int32_t *, int64_t *) { return -1; }
int main() {
  for (int patch : {1, 2, 4})
    for (int leaf : {1, 16, 1 << 20, 1 << 30}) {
      const int H = 12 * patch, W = 20 * patch, n = 12 * 20;
      std::vector<float> img(static_cast<size_t>(H) * W);
      for (size_t i = 0; i < img.size(); ++i) img[i] = std::sin(0.7f * static_cast<float>(i % W)) + 0.3f * static_cast<float>(i / W % 5);
      std::vector<int32_t> y(n), x(n), s(n), off(2), of(n);
      int64_t leaves = 0;
      const int rc = reslim_asc_build(img.data(), 1, H, W, patch, leaf, 1, 10, 40, 0.05f, y.data(), x.data(), s.data(), off.data(), of.data(), &leaves);
      if (rc != 0 || leaves < 1 || leaves > n) return std::printf("patch %d leaf %d: rc %d, %ld leaves\n", patch, leaf, rc, static_cast<long>(leaves)), 1;
    }
  return 0;
}
"""


def test_largest_leaves(tmp_path):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no g++")
    (tmp_path / "drive.cpp").write_text(DRIVE)
    exe = tmp_path / "drive"
    subprocess.run([cxx, "-std=c++17", "-O0", "-w", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "include"), str(tmp_path / "drive.cpp"),
                    os.path.join(CSRC, "asc_host.cpp"), "-o", str(exe)], check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout + run.stderr
