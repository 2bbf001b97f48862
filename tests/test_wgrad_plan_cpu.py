"""The rule that gives the weight gradients a tile and slices of the tokens (csrc/wgrad_plan.h), compiled for the CPU: the
slices cover the tokens, the partial sums stay within what the header states, and the shapes of the GPU test reach both
kernels at every edge that it claims."""
import ctypes
import os
import random
import shutil
import subprocess

import pytest
from test_gpu_wgrad_tiles import SHAPES

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_04802_amd", "csrc")
ASK = r"""
#include "wgrad_plan.h"
extern "C" void plan(const int *nk, int n_op, int M, int cus, long long *out) {
  reslim::WgradOp op[reslim::kWgradMax] = {};
  for (int i = 0; i < n_op; ++i) { op[i].N = nk[2 * i]; op[i].K = nk[2 * i + 1]; }
  const reslim::WgradPlan p = reslim::wgrad_plan(op, n_op, M, cus);
  out[0] = p.kind == reslim::kWgrad256; out[1] = p.tiles; out[2] = p.splits; out[3] = p.m_per_split;
  out[4] = p.splits > 1 ? p.splits * reslim::wgrad_slice(op, n_op) * 4 : 0;
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, so = d / "plan.cpp", d / "plan.so"
    src.write_text(ASK)
    cxx = shutil.which("g++") or shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)], check=True)
    lib = ctypes.CDLL(str(so))

    def ask(products, M, cus=256):
        nk = (ctypes.c_int * (2 * len(products)))(*[v for p in products for v in p])
        out = (ctypes.c_longlong * 5)()
        lib.plan(nk, len(products), M, cus, out)
        return dict(zip(("tile", "tiles", "slices", "tokens", "bytes"), (256 if out[0] else 128, *out[1:])))

    return ask


def test_slices_cover_the_tokens_within_the_stated_bytes(plan):
    r = random.Random(3)
    for _ in range(400):
        D = 8 * r.randint(1, 1024)
        products = r.choice([[(3 * D, D)], [(D, D)], [(D, 4 * D), (4 * D, D)], [(D, 4 * D), (4 * D, D), (D, D), (3 * D, D)]])
        M = int(2 ** r.uniform(0, 19))
        p = plan(products, M)
        assert p["tokens"] % 64 == 0 and (p["slices"] - 1) * p["tokens"] < M <= p["slices"] * p["tokens"]
        assert p["tiles"] == sum(-(-n // p["tile"]) * -(-k // 256) for n, k in products)
        assert p["slices"] == 1 or p["slices"] * p["tiles"] <= 1024
        assert p["bytes"] <= 257 << 20


def test_shapes_of_the_gpu_test_reach_both_kernels_at_their_edges(plan):
    seen = {128: set(), 256: set()}
    for D, which, rows in SHAPES:
        n, k = ((3 * D, D), (D, D), (2 * D, D), (D, 2 * D))[which]
        p = plan([(n, k)], rows)
        slabs = -(-min(rows, p["tokens"]) // 64)
        seen[p["tile"]] |= {"one slab" if slabs == 1 else "odd slabs" if slabs % 2 else "even slabs",
                            "one slice" if p["slices"] == 1 else "slices", "whole slices" if rows % p["tokens"] == 0 else "ragged slice",
                            "one token" if rows == 1 else "tokens", "whole rows" if n % p["tile"] == 0 else "ragged rows",
                            "whole columns" if k % 256 == 0 else "ragged columns", "many slices" if p["slices"] >= 16 else "few slices"}
    for tile, s in seen.items():
        assert len(s) == 15, (tile, sorted(s))
