"""GELU of the bf16 path (csrc/gelu.h), compiled for the CPU, against erfc in fp64: the bounds that its comment states."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest
from scipy.special import erfc

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_04802_amd", "csrc")
# what the header takes from the device compiler
DEVICE = """#include <cmath>
#include <cstdint>
#define __device__
#define __forceinline__ inline
#define __builtin_amdgcn_exp2f exp2f
#define __builtin_amdgcn_fmed3f(a, lo, hi) fminf(fmaxf(a, lo), hi)
"""
MAIN = """#include "gelu.h"
extern "C" void ask(const float *x, float *y, int n) { for (int i = 0; i < n; ++i) y[i] = reslim::gelu_erf_fast(x[i]); }
"""


@pytest.fixture(scope="module")
def gelu(tmp_path_factory):
    d = tmp_path_factory.mktemp("gelu")
    shutil.copy(os.path.join(CSRC, "gelu.h"), d)
    (d / "common.h").write_text(DEVICE)
    (d / "main.cpp").write_text(MAIN)
    cxx = shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"      # vector types that g++ does not have
    subprocess.run([cxx, "-std=c++17", "-O1", "-ffp-contract=off", "-shared", "-fPIC", str(d / "main.cpp"), "-o", str(d / "gelu.so")], check=True)
    lib = ctypes.CDLL(str(d / "gelu.so"))

    def call(x):
        x, y = np.ascontiguousarray(x, np.float32), np.empty(len(x), np.float32)
        lib.ask(x.ctypes.data_as(ctypes.c_void_p), y.ctypes.data_as(ctypes.c_void_p), len(x))
        return y.astype(np.float64)

    return call


def test_error_bounds(gelu):
    x = np.concatenate([np.linspace(-12, 12, 480001), np.geomspace(1e-30, 1, 4001), -np.geomspace(1e-30, 1, 4001)]).astype(np.float32)
    want = 0.5 * x.astype(np.float64) * erfc(-x.astype(np.float64) / np.sqrt(2.0))
    off = np.abs(gelu(x) - want)
    inside = (np.abs(x) <= 5) & (x != 0)
    assert (off[inside] / np.abs(want[inside])).max() <= 1.5e-5      # 130 times below the bf16 rounding, 2^-9
    assert off.max() <= 2e-6
    assert off[x < -5].max() <= 1.5e-6 and (off[x > 5] / want[x > 5]).max() <= 3e-7


def test_ends(gelu):
    big = np.float32(3.0e38)
    assert gelu(np.array([0.0, big], np.float32)).tolist() == [0.0, float(big)]
    far = gelu(np.array([-big, -np.inf, -20.0], np.float32))
    assert np.all(np.abs(far) <= 1.5e-6)
    assert gelu(np.array([np.inf], np.float32))[0] >= np.finfo(np.float32).max      # rounds to infinity in bf16
