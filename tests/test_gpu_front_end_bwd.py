"""The front end's gradient at the edges of its kernels: value tables of one to several 128-row chunks (variables times
pixels), every patch size, heads wider than 64 features or narrower than 32, more heads than a 32-row tile holds,
embedding widths that end inside a tile, token counts that end inside a group."""
import pytest
import torch

from oracle import train_oracle as TO
from paper_2505_04802_amd import binding as B
from paper_2505_04802_amd import workloads as WL
from test_gpu_train_step import FRONT, case, check_grads, cuda, grad_buffers, u8

pytestmark = pytest.mark.gpu
BASE = WL.ReslimConfig("fe", batch=1, in_vars=3, out_vars=1, H=12, W=20, scale=2, patch=2, embed_dim=48, heads=2, mlp_ratio=1, depth=1,
                       tiles_y=1, tiles_x=2, halo=1, dtype=0, seed=61)


@pytest.mark.parametrize("cfg", [
    BASE.with_(name="v30", in_vars=30, embed_dim=100, heads=5),              # 150 table rows, dh 20
    BASE.with_(name="v7p1", in_vars=7, patch=1, H=9, W=15, batch=2),         # 14 rows
    BASE.with_(name="v2p4", in_vars=2, patch=4, H=16, W=24),                 # 34 rows
    BASE.with_(name="v9p4", in_vars=9, patch=4, H=16, W=24),                 # 153 rows
    BASE.with_(name="h40", embed_dim=160, heads=40),                         # dh 4
    BASE.with_(name="dh150", embed_dim=300, heads=2),
    BASE.with_(name="bf", in_vars=13, out_vars=3, scale=4, embed_dim=192, heads=3, dtype=1, batch=3),
], ids=lambda c: c.name)
def test_front_end(cfg):
    w, x, target, lat_w = case(cfg, 0.1)
    print(f"front end {cfg.name}: oracle ...", flush=True)
    _, ref, inter = TO.reslim_loss_and_grads(x, target, w, cfg, lat_w, 0.5)
    with B.Reslim(cfg, w) as m:
        B.reslim_train_prepare_model(m.ctx, w)
        g = grad_buffers(w, FRONT)
        B.reslim_embed_bwd(m.ctx, cuda(x), cuda(inter["d_tokens_in"]), g, cfg.batch, u8(B.reslim_embed_bwd_workspace_bytes(m.ctx, cfg.batch)))
        torch.cuda.synchronize()
        check_grads(g, ref, FRONT, cfg, "front end")
