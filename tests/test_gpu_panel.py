"""The kernel that takes whole rows through a block's products and LayerNorms in one launch (csrc/panel.hip), where it can go
wrong: fewer rows than a panel, a remainder of one row, one, two and three row blocks a panel, two to six chunks of the hidden layer (an even number), skip rows through the gather list and the stitch map, a block alone and blocks in a chain that leave each other's qkv."""
import numpy as np
import pytest
import torch

from oracle import asc_oracle as A
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
def test_same_bits_as_the_separate_kernels(separate_kernels, cfg):
    """Every sum runs over k upwards from zero, then comes the bias, then the skip connection: as in the separate kernels, to the bit."""
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
        chain_sep = tok.clone()
        for l in range(cfg.depth):
            m.block(l, chain_sep)
        separate_kernels(False)
        y_chain = m.head(x, chain).cpu().numpy()
    assert np.array_equal(y, y_chain)                    # the chain of entry points, qkv by separate kernels
    assert torch.equal(chain, chain_sep) and np.array_equal(y, y_sep)


@pytest.mark.parametrize("cfg", [BASE, SMALL[4], *LARGE], ids=lambda c: c.name)
def test_a_stream_far_larger_than_the_update(separate_kernels, cfg):
    """Rows around 4096, updates of order one: summed by themselves and added once, in either form, so the same bits."""
    print(f"panel, large stream {cfg.name}", flush=True)
    with B.Reslim(cfg, WL.make_weights(cfg, std=0.1)) as m:
        g = torch.Generator(device="cuda").manual_seed(5)
        x = 4096.0 + torch.randn((cfg.batch, m.n_h, cfg.embed_dim), generator=g, device="cuda", dtype=torch.float32)
        got, sep = x.clone(), x.clone()
        m.block(0, got)
        separate_kernels(True)
        m.block(0, sep)
    assert torch.equal(got, sep) and not torch.equal(got, x)


def test_a_stream_that_is_not_aligned(separate_kernels):
    """Four bytes off 16: the separate kernels take it; the same bits as the aligned one, so a chain of entry points on any stream gives
    what a whole forward gives."""
    for cfg in (SMALL[2], SMALL[4]):
        print(f"stream off 16 bytes {cfg.name}", flush=True)
        with B.Reslim(cfg, WL.make_weights(cfg, std=0.1)) as m:
            x = torch.from_numpy(WL.make_fields(cfg)).cuda()
            tok = m.embed(x)
            off = torch.empty(tok.numel() + 1, dtype=torch.float32, device="cuda")[1:].view(tok.shape)
            assert tok.data_ptr() % 16 == 0 and off.data_ptr() % 16 == 4
            off.copy_(tok)
            for l in range(cfg.depth):
                m.block(l, tok)
                m.block(l, off)
            assert torch.equal(tok, off)
            assert torch.equal(m.forward(x), m.head(x, tok))


def test_compressed_and_plain_forward_choose_apart():
    """One patch per leaf at D = 512, 1008 patches owned and 1280 with halo copies: the compressed forward counts the leaves, copies included,
    and takes the kernel; the plain forward counts the patches and does not.  The outputs are the same bits all the same."""
    cfg = BASE.with_(H=72, W=56, in_vars=1, out_vars=1, embed_dim=512, heads=8, mlp_ratio=2, tiles_y=2, tiles_x=2, halo=2)
    w, x = WL.make_weights(cfg, std=0.05), WL.make_fields(cfg)
    tiles, _, _, n_h = O.tiles_partition(cfg.Hp, cfg.Wp, cfg.tiles_y, cfg.tiles_x, cfg.halo)
    assert cfg.batch * cfg.n_tokens < 1024 <= cfg.batch * n_h, "the case is meant to lie across the line"
    tab = A.build_tiles(np.ascontiguousarray(x[:, 0]), cfg.patch, tiles, 1, 1, 10, 20, 0.05, Wp=cfg.Wp)
    with B.Reslim(cfg, w) as m:
        xd = torch.from_numpy(x).cuda()
        plain = m.forward(xd)
        y = torch.empty_like(plain)
        plan = B.reslim_asc_plan_create(m.ctx, cfg.batch, tab)
        try:
            B.reslim_asc_forward(m.ctx, plan, xd, y, m.ws)
        finally:
            B.reslim_asc_plan_destroy(plan)
    assert torch.equal(y, plain)


def test_a_sample_does_not_depend_on_its_batch():
    """D = 512 with 900 patches a sample: alone they are separate launches, two of them are panels."""
    cfg = BASE.with_(batch=2, H=60, W=60, embed_dim=512, heads=8, mlp_ratio=2, tiles_y=2, tiles_x=2, halo=1)
    w = WL.make_weights(cfg, std=0.1)
    x = torch.from_numpy(WL.make_fields(cfg)).cuda()
    assert cfg.n_tokens < 1024 <= 2 * cfg.n_tokens
    with B.Reslim(cfg, w) as m:
        both = m.forward(x)
    with B.Reslim(cfg.with_(batch=1), w) as m:
        assert torch.equal(both, torch.cat([m.forward(x[i:i + 1].contiguous()) for i in range(2)]))
