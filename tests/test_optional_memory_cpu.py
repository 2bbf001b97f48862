"""Memory that a context is faster with and can do without (csrc/optional_memory.h, the packed matrices of reslim_create), compiled for
the CPU with a runtime that has none: no memory and no error left behind."""
import os
import shutil
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_04802_amd", "csrc")
MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "optional_memory.h"
static size_t room = 0;
static bool error = false;      // as a runtime keeps its last error
static bool allocate(void **p, size_t n) {
  if (n > room) { error = true; return false; }
  *p = std::malloc(n);
  return true;
}
int main() {
  auto forget = []() { error = false; };
  void *p = reslim::optional_memory(64, allocate, forget);
  if (p || error) return 1;
  room = 64;
  p = reslim::optional_memory(64, allocate, forget);
  if (!p || error) return 2;
  error = true;                  // of an earlier call: not this function's to take
  void *q = reslim::optional_memory(64, allocate, forget);
  if (!q || !error) return 3;
  std::free(p);
  std::free(q);
  return 0;
}
"""


def test_without_memory(tmp_path):
    (tmp_path / "main.cpp").write_text(MAIN)
    cxx = shutil.which("g++") or shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, str(tmp_path / "main.cpp"), "-o", str(tmp_path / "a")], check=True)
    assert subprocess.run([str(tmp_path / "a")]).returncode == 0
