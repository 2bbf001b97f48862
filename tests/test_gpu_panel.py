"""The kernel that takes whole rows through a block's products and LayerNorms in one launch (csrc/panel.hip), where it can go
wrong: fewer rows than a panel, a remainder of one row, one, two and three row blocks a panel, two to six chunks of the hidden layer (an even number), skip rows through the gather list and the stitch map, a block alone and blocks in a chain that leave each other's qkv."""
import numpy as np
import pytest
import torch

from oracle import reslim_oracle as O
from paper_2505_04802_amd import binding as B
from paper_2505_04802_amd import workloads as WL
from parity_checks import assert_parity

pytestmark = pytest.mark.gpu
BASE = WL.ReslimConfig("panel", batch=1, in_vars=2, out_vars=2, H=8, W=16, scale=2, patch=2, embed_dim=256, heads=4, mlp_ratio=4, depth=2,
                       tiles_y=1, tiles_x=1, halo=0, dtype=1, seed=71)
SMALL = [BASE,                                                                                # 32 rows: one panel
         BASE.with_(name="rows_33", H=6, W=22, mlp_ratio=2, depth=1),                         # a second panel of one row
         BASE.with_(name="halo", batch=2, H=20, W=28, tiles_y=2, tiles_x=2, halo=1, mlp_ratio=6, depth=3),      # gather list, stitch map
         BASE.with_(name="dh128", H=18, W=26, heads=2, tiles_y=1, tiles_x=2, halo=2),
         BASE.with_(name="d512", batch=4, H=30, W=36, embed_dim=512, heads=8, tiles_y=2, tiles_x=1, halo=1, mlp_ratio=3, depth=3),      # 1080 patches
         BASE.with_(name="d512_rows_1025", H=10, W=410, embed_dim=512, heads=4, tiles_x=5, mlp_ratio=1, depth=1)]
LARGE = [BASE.with_(name="d512_two_blocks", batch=2, H=128, W=130, embed_dim=512, heads=8, tiles_y=4, tiles_x=4, depth=1),
         BASE.with_(name="two_blocks", batch=2, H=128, W=130, tiles_y=4, tiles_x=4),          # 8320 rows: panels of 64
         BASE.with_(name="three_blocks", batch=4, H=126, W=134, tiles_y=4, tiles_x=5, halo=1)]     # 16,884 patches and more rows: panels of 96


@pytest.fixture
def separate_kernels():
    """Pins the GEMM kernel, which keeps every product a launch of its own."""
    yield lambda on: B.reslim_debug_set_gemm_tile(2 if on else -1)
    B.reslim_debug_set_gemm_tile(-1)


@pytest.mark.parametrize("cfg", SMALL, ids=lambda c: c.name)
def test_against_the_oracle(cfg):
    print(f"panel {cfg.name}", flush=True)
    w, x = WL.make_weights(cfg, std=0.1), WL.make_fields(cfg)
    y_ref, inter = O.reslim_forward(x, w, cfg, return_intermediates=True)
    with B.Reslim(cfg, w) as m:
        prev = inter["tokens"]
        for l in range(cfg.depth):
            t = torch.from_numpy(prev.astype(np.float32)).cuda()
            m.block(l, t)
            assert_parity(t.cpu().numpy(), inter[f"block{l}"], 2e-2, f"block{l}", print)
            prev = inter[f"block{l}"]
        assert_parity(m.forward(torch.from_numpy(x).cuda()).cpu().numpy(), y_ref, 2e-2, "forward", print)


@pytest.mark.parametrize("cfg", SMALL + LARGE, ids=lambda c: c.name)
def test_against_the_separate_kernels(separate_kernels, cfg):
    """Both round the same values to bf16; sums that start from the bias instead of ending with it move some of them to the neighbouring
    bf16, 2^-8 of the value at most: that is the bound in the 2-norm for a block, over the output and over every row.  Through a whole
    forward what either half of a block rounds differently is independent of the rest and adds up in quadrature: 2^-8 sqrt(2 depth)."""
    print(f"panel against separate kernels {cfg.name}", flush=True)
    w, x = WL.make_weights(cfg, std=0.1), torch.from_numpy(WL.make_fields(cfg)).cuda()
    with B.Reslim(cfg, w) as m:
        y = m.forward(x).cpu().numpy()
        tok = m.embed(x)
        chain = tok.clone()
        for l in range(cfg.depth):
            m.block(l, chain)
        separate_kernels(True)
        y_sep = m.forward(x).cpu().numpy()
        m.block(0, tok)
        separate_kernels(False)
        again = m.embed(x)
        m.block(0, again)
        y_chain = m.head(x, chain).cpu().numpy()
    assert np.array_equal(y, y_chain)                    # the chain of entry points, qkv by separate kernels
    assert_parity(again.cpu().numpy(), tok.cpu().numpy(), 2.0 ** -8, "block", print, k_elem=0.05)
    assert_parity(y, y_sep, 2.0 ** -8 * (2 * cfg.depth) ** 0.5, "forward", print, k_elem=0.05)
