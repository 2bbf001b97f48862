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
    src.write_text('#include "panel_plan.h"\nextern "C" int ask(int M, int cus, int most) { return reslim::panel_row_blocks(M, cus, most); }\n'
                   'extern "C" int from(int D, int R) { return reslim::panel_rows_from(D, R); }\n')
    cxx = shutil.which("g++") or shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)], check=True)
    lib = ctypes.CDLL(str(so))
    ask = lib.ask
    ask.rows_from = getattr(lib, "from")
    return ask


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
    assert all(c.batch * c.n_tokens >= row_blocks.rows_from(c.embed_dim, c.embed_dim * c.mlp_ratio) for c in SMALL + LARGE)


# rows, time of a launch (microseconds, MI355X) in panels of one, two and, at 256 features, three row blocks
TIMES = {256: [(2304, 25.8, 31.3, 39.5), (8192, 31.3, 34.6, 42.2), (8250, 49.1, 33.9, 40.9), (12288, 50.4, 37.0, 43.5), (16384, 55.6, 40.7, 45.5),
               (16500, 74.2, 64.3, 45.7), (19552, 75.1, 64.8, 48.8), (24576, 81.1, 68.7, 53.8), (24700, 99.3, 70.2, 83.8), (32768, 105.9, 76.5, 90.8),
               (33000, 125.2, 101.3, 91.9), (42560, 149.7, 107.3, 100.8), (49152, 156.5, 112.5, 105.3), (65536, 211.5, 153.1, 152.5),
               (100000, 337.2, 255.3, 243.7), (200000, 656.2, 475.4, 449.2)],
         512: [(2304, 71.5, 78.6), (8192, 85.7, 83.4), (8250, 152.3, 84.1), (12288, 151.9, 92.2), (16384, 167.3, 113.5), (16500, 226.4, 179.7),
               (19552, 230.7, 181.9), (24576, 248.1, 195.5), (24700, 312.2, 194.5), (32768, 348.8, 232.3), (42560, 499.7, 325.0), (65536, 689.1, 464.6),
               (100000, 1057.3, 742.9), (200000, 1958.0, 1377.7)]}
# hidden layer over features, rows, time of a block (microseconds) in separate launches and in one, at 512 features
FROM = [(1, 512, 54.3, 51.7), (1, 1024, 57.0, 51.9), (1, 4096, 72.3, 56.7), (2, 512, 58.8, 59.7), (2, 1024, 62.3, 59.3), (2, 2304, 69.8, 60.8),
        (3, 768, 68.2, 69.9), (3, 1024, 69.3, 69.8), (3, 1536, 72.3, 69.8), (3, 3072, 80.8, 72.6), (4, 512, 68.6, 78.3), (4, 1024, 71.3, 77.6),
        (4, 1536, 73.3, 77.3), (4, 2048, 75.5, 77.8), (4, 2304, 80.3, 78.5), (4, 4096, 87.0, 80.7), (6, 1024, 81.7, 97.0), (6, 3072, 98.4, 99.0),
        (6, 4096, 100.7, 100.4), (6, 6144, 119.8, 105.4), (8, 1024, 88.2, 114.8), (8, 2304, 102.1, 115.3), (8, 4096, 112.7, 117.8), (8, 6144, 132.9, 123.0)]


@pytest.mark.parametrize("D", [256, 512])
def test_panels_near_the_fastest(row_blocks, D):
    for rows, *t in TIMES[D]:
        assert t[row_blocks(rows, 256, len(t)) - 1] <= 1.03 * min(t), rows


def test_one_launch_only_where_it_gains(row_blocks):
    """Never more than 1 % slower than the launches it replaces, and taken wherever it is 10 % faster."""
    for ratio, rows, separate, panel in FROM:
        taken = rows >= row_blocks.rows_from(512, 512 * ratio)
        assert (panel <= 1.01 * separate) if taken else (separate <= 1.10 * panel), (ratio, rows)
    assert all(row_blocks.rows_from(256, 256 * r) == 1 for r in (2, 4, 16)) and 0 < row_blocks.rows_from(512, 512 * 256) < 2 ** 20
