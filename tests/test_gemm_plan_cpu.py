"""The rule that gives a bf16 product its kernel (csrc/gemm_plan.h), compiled for the CPU and held against measured times: a
product is never given a kernel that takes much longer than the best of the three.  The times (microseconds, launches of
a forward or of a block's training with each kernel forced in turn, MI355X) are of products that the rule was not
fitted to: 48 drawn at random and 24 at random of those where an earlier rule lost more than 12 %."""
import ctypes
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_04802_amd", "csrc")
ASK = r"""
#include "gemm_plan.h"
extern "C" int choose(int M, int N, int K, int epi, int cus) { return reslim::gemm_choose(M, N, K, static_cast<reslim::GemmEpi>(epi), cus); }
"""
ACT, GELU, TWO, F32, STREAM = range(5)
# M, N, K, epilogue, time with 128 x 128, 256 x 256 and 128 x 256 tiles
TIMES = [
    (120, 576, 1728, ACT, 22.9, 32.4, 20.4), (120, 1792, 1792, STREAM, 26.1, 39.0, 26.0),
    (128, 128, 320, F32, 8.8, 12.9, 9.8), (128, 128, 384, F32, 9.2, 15.0, 10.9),
    (128, 640, 320, TWO, 10.5, 20.4, 14.0), (128, 1536, 384, ACT, 9.3, 13.8, 10.5),
    (242, 320, 320, STREAM, 9.5, 16.8, 11.4), (242, 384, 384, ACT, 9.2, 14.2, 10.6),
    (242, 576, 576, STREAM, 12.4, 20.5, 13.7), (242, 960, 320, ACT, 8.8, 14.0, 10.4),
    (242, 1152, 576, TWO, 14.1, 27.4, 18.0), (253, 2304, 768, ACT, 14.2, 21.7, 14.6),
    (253, 3072, 768, GELU, 15.2, 26.6, 17.2), (253, 6144, 1536, GELU, 23.2, 37.2, 23.5),
    (364, 128, 384, F32, 9.9, 16.1, 11.1), (364, 384, 384, ACT, 9.2, 15.0, 10.4),
    (364, 384, 384, STREAM, 10.2, 18.0, 13.1), (364, 1536, 768, TWO, 15.9, 28.8, 19.2),
    (392, 320, 320, STREAM, 9.2, 16.0, 11.6), (405, 384, 128, ACT, 6.6, 11.1, 9.0),
    (405, 1728, 576, ACT, 11.6, 18.6, 13.2), (665, 320, 320, STREAM, 9.2, 16.3, 11.8),
    (760, 6144, 1536, GELU, 31.5, 38.3, 25.1), (1080, 576, 576, STREAM, 13.0, 20.7, 15.2),
    (1080, 576, 576, STREAM, 12.8, 22.6, 15.0), (1104, 768, 768, STREAM, 14.7, 23.1, 16.6),
    (1125, 128, 256, STREAM, 8.9, 16.7, 11.3), (1456, 576, 576, STREAM, 12.6, 20.5, 14.5),
    (1508, 4096, 4096, ACT, 66.8, 74.3, 58.4), (1537, 384, 384, STREAM, 11.0, 20.5, 13.8),
    (1980, 576, 576, ACT, 11.5, 17.2, 12.6), (2176, 320, 320, STREAM, 9.8, 17.6, 13.1),
    (2205, 704, 704, STREAM, 14.2, 22.1, 16.1), (2304, 3072, 384, TWO, 17.4, 24.4, 17.9),
    (2698, 1152, 384, ACT, 11.7, 16.6, 13.1), (2847, 128, 128, STREAM, 8.2, 16.4, 11.1),
    (3034, 320, 640, STREAM, 13.5, 21.1, 15.2), (3234, 768, 768, STREAM, 15.8, 23.5, 16.9),
    (4089, 704, 2112, ACT, 32.4, 44.4, 34.5), (4224, 3072, 384, ACT, 21.6, 18.0, 20.0),
    (5141, 576, 2304, STREAM, 31.0, 43.6, 30.0), (5141, 2304, 576, ACT, 23.0, 22.1, 28.5),
    (5928, 4608, 1536, ACT, 99.8, 83.3, 92.7), (7424, 1792, 1792, GELU, 67.4, 50.6, 59.6),
    (8763, 128, 576, F32, 12.3, 18.2, 13.3), (8763, 1920, 960, GELU, 47.7, 55.4, 48.1),
    (9709, 320, 2560, ACT, 39.6, 56.8, 45.0), (10920, 1536, 6144, STREAM, 262.8, 231.2, 226.7),
    (11988, 576, 1152, ACT, 26.2, 31.4, 34.2), (12616, 768, 768, STREAM, 37.0, 38.2, 40.2),
    (12768, 128, 1024, STREAM, 18.0, 28.2, 18.6), (12936, 1536, 384, ACT, 26.8, 30.4, 27.6),
    (13005, 2112, 704, ACT, 52.6, 48.2, 50.6), (14168, 4608, 1536, ACT, 242.3, 163.3, 191.4),
    (14924, 1152, 576, GELU, 33.5, 43.6, 38.2), (17542, 4096, 16384, STREAM, 2839.1, 1835.7, 2322.4),
    (18382, 576, 2304, STREAM, 77.6, 72.8, 80.4), (21276, 4096, 4096, STREAM, 815.3, 621.4, 714.8),
    (23370, 576, 576, STREAM, 34.9, 42.9, 37.4), (26040, 384, 1152, ACT, 37.2, 32.7, 38.9),
    (28500, 2880, 960, ACT, 195.8, 155.0, 157.5), (35420, 5376, 1792, ACT, 775.7, 541.4, 636.4),
    (37180, 1536, 384, GELU, 66.0, 71.5, 68.2), (70132, 2112, 704, ACT, 267.1, 218.9, 268.9),
    (79800, 320, 320, STREAM, 52.0, 68.2, 60.2), (80010, 128, 384, F32, 25.8, 32.7, 30.2),
    (80010, 384, 768, ACT, 65.7, 68.5, 63.0), (90720, 2560, 320, GELU, 232.2, 244.6, 284.2),
    (96327, 2304, 576, ACT, 324.1, 278.5, 342.1), (105512, 768, 768, STREAM, 224.7, 197.7, 222.7),
    (105512, 6144, 768, ACT, 1304.6, 963.2, 1255.1), (108290, 704, 2112, ACT, 399.8, 268.4, 306.7),
]


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    d = tmp_path_factory.mktemp("choose")
    src, so = d / "choose.cpp", d / "choose.so"
    src.write_text(ASK)
    cxx = shutil.which("g++") or shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so)).choose


def test_choice_against_measured_times(choose):
    """Two timings of one launch differ by up to 5 % (medians of 3 x 5 launches at different times of a run), so a choice within
    10 % of the best is none that timing shows to be wrong; a rule has such ones at its lines, and few of them."""
    ratios = {(M, N, K, epi): times[choose(M, N, K, epi, 256) - 2] / min(times) for M, N, K, epi, *times in TIMES}
    slow = {k: round(v, 2) for k, v in ratios.items() if v > 1.10}
    assert len(slow) <= len(TIMES) // 24 and all(v <= 1.20 for v in slow.values()), slow
    assert sum(ratios.values()) / len(ratios) < 1.015
