"""Parameter gradients of linear layers where the tiled kernel can go wrong: one token, one less and one more than the 64
tokens of a slab, an odd and an even number of slabs, a last slice that is not whole, feature counts at the edges of both
tiles (128 and 256; test_wgrad_plan_cpu.py asks the library's own rule which one each shape takes).  Reference: the same
sums in float64 on the CPU."""
import numpy as np
import pytest
import torch

from paper_2505_04802_amd import binding as B
from paper_2505_04802_amd import workloads as WL

pytestmark = pytest.mark.gpu
BASE = WL.ReslimConfig("wgrad", batch=1, in_vars=2, out_vars=2, H=8, W=16, scale=2, patch=2, embed_dim=64, heads=1, mlp_ratio=2,
                       depth=1, tiles_y=1, tiles_x=1, halo=0, dtype=1, seed=17)


SHAPES = [(64, 1, 1), (64, 0, 63), (64, 2, 65), (128, 1, 128), (128, 3, 4097), (256, 1, 192), (256, 2, 19551), (320, 0, 1000), (320, 1, 70001),
          (1024, 2, 2000),
          (1984, 0, 1), (1984, 0, 65), (1984, 0, 129), (2048, 0, 63), (2048, 0, 192), (1088, 0, 4001), (1024, 0, 8000), (320, 0, 64001)]


@pytest.mark.parametrize("D,which,rows", SHAPES, ids=str)
def test_weight_and_bias_gradient(D, which, rows):
    print(f"wgrad D={D} which={which} rows={rows}", flush=True)
    cfg = BASE.with_(embed_dim=D, heads=D // 64)
    n, k = ((3 * D, D), (D, D), (2 * D, D), (D, 2 * D))[which]
    g = torch.Generator().manual_seed(rows)
    x = torch.randn((rows, k), generator=g).to(torch.bfloat16)
    dy = torch.randn((rows, n), generator=g).to(torch.bfloat16)
    with B.Reslim(cfg, WL.make_weights(cfg, std=0.1)) as m:
        B.reslim_train_prepare(m.ctx)
        dw = torch.full((n, k), float("nan"), dtype=torch.float32, device="cuda")
        db = torch.full((n,), float("nan"), dtype=torch.float32, device="cuda")
        ws = torch.full((B.reslim_linear_bwd_workspace_bytes(m.ctx, which, rows),), 255, dtype=torch.uint8, device="cuda")
        B.reslim_linear_bwd(m.ctx, 0, which, x.cuda(), dy.cuda(), None, dw, db, rows, ws)
        dw2, db2 = torch.empty_like(dw), torch.empty_like(db)
        B.reslim_linear_bwd(m.ctx, 0, which, x.cuda(), dy.cuda(), None, dw2, db2, rows, ws)
        assert torch.equal(dw, dw2) and torch.equal(db, db2)      # fixed order of summation
    cols = np.unique(np.concatenate([np.arange(min(k, 8)), np.arange(k - 8, k), np.random.default_rng(1).integers(0, k, 48)]))
    ref = dy.double().t() @ x[:, cols].double()
    err = float((dw.cpu()[:, cols].double() - ref).norm() / ref.norm())
    assert err <= 2e-6, err
    ref = dy.double().sum(0)
    assert float((db.cpu().double() - ref).norm() / ref.norm()) <= 2e-6
