"""When tile attention splits the keys over the waves (csrc/attention_plan.h), compiled for the CPU and held against measured times: the
kernel a launch gets never takes much longer than the other.  Microseconds on MI355X (256 compute units), one tile a sample, head
dimension 64, launches in a graph with each kernel forced in turn; two runs of one kernel differ by up to 2 %."""
import ctypes
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_04802_amd", "csrc")
# tokens, units of 128 queries, time without and with the split
TIMES = [(512, 16, 11.64, 6.59), (512, 64, 11.77, 6.98), (512, 112, 11.92, 8.41), (512, 128, 12.03, 9.19), (512, 144, 11.98, 12.33),
         (512, 192, 12.16, 13.11), (512, 224, 12.22, 14.57), (512, 256, 12.83, 15.04), (512, 512, 17.08, 26.32), (640, 40, 13.86, 8.32),
         (640, 100, 13.86, 9.33), (640, 120, 14.27, 10.55), (640, 140, 14.10, 13.84), (640, 180, 14.31, 14.11), (640, 200, 14.56, 16.58),
         (640, 240, 14.74, 16.60), (640, 320, 17.47, 21.05), (768, 96, 16.13, 10.83), (768, 144, 16.29, 15.68), (768, 192, 16.34, 16.19),
         (768, 216, 16.49, 18.19), (768, 240, 16.81, 18.45), (1024, 32, 20.18, 9.53), (1024, 128, 20.41, 12.90), (1024, 160, 20.44, 18.90),
         (1024, 192, 20.64, 18.66), (1024, 224, 20.64, 21.85), (1024, 256, 21.06, 22.82), (1024, 512, 26.34, 40.47), (1440, 108, 27.69, 15.93),
         (1440, 132, 27.76, 23.70), (1440, 192, 27.72, 26.85), (1440, 240, 28.11, 29.38), (1440, 384, 32.49, 40.23), (1806, 150, 33.96, 31.67),
         (1806, 180, 34.02, 31.61), (1806, 210, 34.20, 33.49), (1806, 240, 34.01, 34.69), (2300, 18, 40.60, 16.36), (2300, 72, 41.06, 21.59),
         (2300, 144, 41.08, 34.06), (2300, 198, 40.96, 39.30), (2300, 252, 41.66, 39.91), (2300, 288, 46.71, 49.39), (2300, 576, 66.24, 85.32),
         (3000, 192, 52.73, 42.99), (3000, 240, 53.06, 51.36), (3840, 60, 65.98, 27.11), (3840, 240, 66.18, 61.33), (3840, 480, 77.30, 116.56),
         (5040, 200, 86.35, 75.66), (6400, 100, 107.57, 51.03), (6400, 250, 107.72, 96.85), (6400, 400, 120.23, 167.67), (6400, 800, 268.80, 304.33)]


@pytest.fixture(scope="module")
def splits(tmp_path_factory):
    d = tmp_path_factory.mktemp("attention")
    src, so = d / "plan.cpp", d / "plan.so"
    src.write_text('#include "attention_plan.h"\nextern "C" int ask(int units, int cus, int tokens) { return reslim::attn_split_keys(units, cus, tokens); }\n')
    cxx = shutil.which("g++") or shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so)).ask


def test_never_much_slower_than_the_other(splits):
    for tokens, units, without, split in TIMES:
        got = split if splits(units, 256, tokens) else without
        assert got <= 1.03 * min(without, split), (tokens, units, got)


def test_only_where_it_was_measured(splits):
    """Shorter tiles and more units than compute units keep the kernel that they had."""
    assert not any(splits(u, 256, 511) for u in (1, 64, 256)) and not any(splits(257, 256, n) for n in (512, 4096, 10 ** 6))
    assert splits(1, 256, 512) and not splits(2 ** 31 - 1, 256, 10 ** 6)
