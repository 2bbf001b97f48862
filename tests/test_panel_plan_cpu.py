"""How many rows a work-group of the panel kernel takes (csrc/panel_plan.h), compiled for the CPU."""
import ctypes
import os
import shutil
import subprocess

import pytest
from test_gpu_panel import LARGE, SMALL

from oracle import reslim_oracle as O

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_04802_amd", "csrc")


@pytest.fixture(scope="module")
def row_blocks(tmp_path_factory):
    d = tmp_path_factory.mktemp("panel")
    src, so = d / "plan.cpp", d / "plan.so"
    src.write_text('#include "panel_plan.h"\nextern "C" int ask(int M, int cus, int most) { return reslim::panel_row_blocks(M, cus, most); }\n')
    cxx = shutil.which("g++") or shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so)).ask


def test_one_round_while_it_suffices(row_blocks):
    for rows, rb in [(1, 1), (8192, 1), (8193, 2), (16384, 2), (16385, 3), (24576, 3)]:
        assert row_blocks(rows, 256, 3) == rb and row_blocks(rows, 256, 2) == min(rb, 2), rows
    for rows in (1, 1000, 10 ** 6, 2 ** 31 - 1):
        assert 1 <= row_blocks(rows, 256, 2) <= 2 and 1 <= row_blocks(rows, 1, 3) <= 3


def test_the_gpu_tests_reach_every_height(row_blocks):
    rows = lambda c: c.batch * O.tiles_partition(c.Hp, c.Wp, c.tiles_y, c.tiles_x, c.halo)[3]
    most = lambda c: {256: 3, 512: 2}[c.embed_dim]
    assert {row_blocks(rows(c), 256, most(c)) for c in SMALL} == {1}
    assert [row_blocks(rows(c), 256, most(c)) for c in LARGE] == [2, 2, 3]
