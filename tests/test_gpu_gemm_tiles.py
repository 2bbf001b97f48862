"""The persistent bf16 GEMM kernels (256 x 256 and 128 x 256 tiles, two wave groups half a phase apart) forced where
they can go wrong: one, two, an odd and an even number of 64-deep slabs per tile (the buffer a tile starts in then
alternates), fewer and more tiles than compute units, row counts at the edges of both tiles, a column edge, every
epilogue.  Reference: the same product in fp32 by PyTorch on the CPU; the small-tile kernel must agree bit for bit,
since all three add k in the same order."""
import numpy as np
import pytest
import torch

from paper_2505_04802_amd import binding as B
from paper_2505_04802_amd import workloads as WL

pytestmark = pytest.mark.gpu
BASE = WL.ReslimConfig("gemm", batch=1, in_vars=2, out_vars=2, H=8, W=16, scale=2, patch=2, embed_dim=64, heads=1, mlp_ratio=1,
                       depth=1, tiles_y=1, tiles_x=1, halo=0, dtype=1, seed=91)


@pytest.fixture
def forced_tile():
    yield B.reslim_debug_set_gemm_tile
    B.reslim_debug_set_gemm_tile(-1)


@pytest.mark.parametrize("D,which,rows", [(64, 1, 1), (64, 1, 127), (64, 1, 70001), (64, 0, 257), (128, 1, 70000), (128, 2, 384),
                                          (320, 1, 1000), (320, 0, 128), (192, 0, 33003)], ids=str)
def test_input_gradient_of_a_linear_layer(forced_tile, D, which, rows):
    print(f"gemm tiles D={D} which={which} rows={rows}", flush=True)
    cfg = BASE.with_(embed_dim=D, heads=D // 64, mlp_ratio=2)
    w = WL.make_weights(cfg, std=0.1)
    n, k, name = ((3 * D, D, "w_qkv"), (D, D, "w_proj"), (2 * D, D, "w_fc1"), (D, 2 * D, "w_fc2"))[which]
    g = torch.Generator().manual_seed(rows)
    dy = torch.randn((rows, n), generator=g).to(torch.bfloat16)
    ref = dy.float() @ torch.from_numpy(w[name][0])
    with B.Reslim(cfg, w) as m:
        B.reslim_train_prepare(m.ctx)
        x = torch.zeros((rows, k), dtype=torch.bfloat16, device="cuda")
        dw = torch.empty((n, k), dtype=torch.float32, device="cuda")
        db = torch.empty(n, dtype=torch.float32, device="cuda")
        ws = torch.empty(B.reslim_linear_bwd_workspace_bytes(m.ctx, which, rows), dtype=torch.uint8, device="cuda")
        out = {}
        for tile in (2, 3, 4):
            dx = torch.full((rows, k), float("nan"), dtype=torch.bfloat16, device="cuda")
            forced_tile(tile)
            B.reslim_linear_bwd(m.ctx, 0, which, x, dy.cuda(), dx, dw, db, rows, ws)
            out[tile] = dx.cpu()
        forced_tile(-1)
    err = float((out[3].float() - ref).norm() / ref.norm())
    assert err <= 5e-3, err
    assert torch.equal(out[3], out[2]) and torch.equal(out[4], out[2])


@pytest.mark.parametrize("D", [64, 320])
def test_every_epilogue_bit_identical_to_the_small_tiles(forced_tile, D):
    """A training forward (GELU keeping both outputs, skip connection from another buffer), a whole forward with halo
    copies (skip through the gather list and the stitch map, position table, fp32 head) and the chained block (skip in
    place, q-scaled and GELU outputs); about a thousand rows, no multiple of a tile."""
    cfg = BASE.with_(batch=2, H=36, W=44, embed_dim=D, heads=D // 64, mlp_ratio=3, depth=3, tiles_y=2, tiles_x=2, halo=1, scale=4)
    w = WL.make_weights(cfg, std=0.1)
    x = torch.from_numpy(WL.make_fields(cfg)).cuda()
    with B.Reslim(cfg, w) as m:
        B.reslim_train_prepare(m.ctx)
        sb, wb = B.reslim_block_train_bytes(m.ctx, cfg.batch)
        ws = torch.empty(wb, dtype=torch.uint8, device="cuda")
        res = {}
        for tile in (2, 3, 4):
            print(f"gemm tiles epilogues D={D} tile={tile}", flush=True)
            forced_tile(tile)
            y = m.forward(x)
            tok = m.embed(x)
            out = torch.empty_like(tok)
            saved = torch.zeros(sb, dtype=torch.uint8, device="cuda")
            B.reslim_block_fwd_train(m.ctx, 0, tok, out, saved, cfg.batch, ws)
            m.block(1, tok)
            res[tile] = [t.cpu() for t in (y, tok, out, saved)]
        forced_tile(-1)
    for tile in (3, 4):
        assert all(torch.equal(a, b) for a, b in zip(res[tile], res[2]))
    assert np.isfinite(res[2][0].numpy()).all()
