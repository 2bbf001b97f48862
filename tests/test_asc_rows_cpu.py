"""The quad-tree builder's row loops where they can go wrong: widths around the vector lengths, images of one row or
column, fields whose range is a denormal number, negative zeros, boxes cut out of a wider field."""
import numpy as np
import pytest

from oracle import asc_oracle as A
from oracle import reslim_oracle as O
from paper_2505_04802_amd import binding as B

KEYS = ("leaf_y0", "leaf_x0", "leaf_s", "sample_off", "patch_leaf")


def same(got, ref):
    return all(np.array_equal(np.asarray(got[k]), np.asarray(ref[k])) for k in KEYS)


@pytest.mark.parametrize("W", [1, 2, 7, 8, 9, 15, 16, 17, 31, 33, 48, 65])
def test_widths(W):
    r = np.random.default_rng(W)
    for H in (1, 2, 3, 5, 20):
        img = np.cumsum(r.standard_normal((1, H, W)), axis=-1).astype(np.float32)
        e = B.reslim_asc_edges(img[0], 10, 40)
        assert np.array_equal(e.astype(bool), A.canny_edges(A.quantise_u8(img[0]), 10, 40)), (H, W)
        assert same(B.reslim_asc_build(img, 1, 8, 1, 10, 40, 0.1), A.build(img, 1, 8, 1, 10, 40, 0.1)), (H, W)


def test_extreme_ranges():
    r = np.random.default_rng(3)
    base = r.integers(0, 2, (5, 24, 40)).astype(np.float32)
    base[0] *= np.float32(1e-44)                      # 255 / range overflows to infinity
    base[1] = np.where(base[1] > 0, np.float32(0.0), np.float32(-0.0))      # two zeros: a constant field
    base[2] = (2 * base[2] - 1) * np.float32(3e38)    # the range overflows
    base[3] -= 7.0                                    # negative values only
    base[4] = (base[4] - 0.5) * np.float32(3e38)      # the largest range that does not overflow, nearly
    with np.errstate(all="ignore"):
        for b in (0, 1, 3, 4):
            got, ref = B.reslim_asc_build(base[b:b + 1], 2, 8, 1, 20, 60, 0.05), A.build(base[b:b + 1], 2, 8, 1, 20, 60, 0.05)
            assert same(got, ref), b
    # 255 / infinity is 0 and every product is 0 or the NaN of 0 * infinity, which counts as 0: the tree of a constant field
    assert not B.reslim_asc_edges(base[2], 20, 60).any()
    flat = A.build(np.zeros_like(base[2:3]), 2, 8, 1, 20, 60, 0.05)
    assert same(B.reslim_asc_build(base[2:3], 2, 8, 1, 20, 60, 0.05), flat)


def test_boxes_of_a_wide_field():
    r = np.random.default_rng(5)
    img = np.cumsum(np.cumsum(r.standard_normal((2, 40, 94)), axis=-1), axis=-2).astype(np.float32)
    tiles = O.tiles_partition(20, 47, 3, 4, 2)[0]
    assert same(B.reslim_asc_build_tiles(img, 2, 3, 4, 2, 8, 1, 15, 45, 0.05), A.build_tiles(img, 2, tiles, 8, 1, 15, 45, 0.05, Wp=47))


@pytest.mark.parametrize("max_leaf", [32, 64, 1 << 20, 1 << 30])
def test_leaves_limited_by_the_grid_alone(max_leaf):
    """A largest leaf beyond the grid: nodes that stick out split, and no table has its size."""
    img = np.cumsum(np.random.default_rng(6).standard_normal((2, 46, 70)), axis=-1).astype(np.float32)
    assert same(B.reslim_asc_build(img, 2, max_leaf, 1, 15, 45, 0.05), A.build(img, 2, max_leaf, 1, 15, 45, 0.05))
