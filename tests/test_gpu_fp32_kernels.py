"""The fp32 matrix kernels where they can go wrong: head dimensions around the 32-feature blocks and beyond 256 or no
multiple of four, tiles of one token up to several blocks of 32 keys, products whose rows or columns end inside a tile,
split over waves or not, operands that are not 16-byte aligned."""
import numpy as np
import pytest
import torch

from oracle import reslim_oracle as O
from paper_2505_04802_amd import binding as B
from paper_2505_04802_amd import workloads as WL

pytestmark = pytest.mark.gpu
BASE = WL.ReslimConfig("f32k", batch=2, in_vars=1, out_vars=1, H=10, W=26, scale=2, patch=2, embed_dim=64, heads=2, mlp_ratio=1,
                       depth=1, tiles_y=1, tiles_x=1, halo=0, dtype=0, seed=23)


@pytest.mark.parametrize("dh,heads", [(2, 2), (6, 2), (20, 3), (36, 1), (64, 2), (130, 2), (300, 1), (516, 1)], ids=str)
@pytest.mark.parametrize("grid", [(5, 13, 5, 13, 0), (5, 13, 1, 1, 0), (10, 26, 2, 3, 1)], ids=str)
def test_attention(dh, heads, grid):
    hp, wp, ty, tx, halo = grid
    print(f"fp32 attention dh={dh} heads={heads} grid={grid}", flush=True)
    D = dh * heads
    cfg = BASE.with_(H=2 * hp, W=2 * wp, embed_dim=D, heads=heads, tiles_y=ty, tiles_x=tx, halo=halo)
    tiles = O.tiles_partition(hp, wp, ty, tx, halo)[0]
    r = np.random.default_rng(dh)
    with B.Reslim(cfg, WL.make_weights(cfg)) as m:
        qkv = r.standard_normal((cfg.batch, m.n_h, 3 * D)).astype(np.float32)
        qkv[..., : 2 * D] *= 2.0
        out, lse = m.attention_with_lse(torch.from_numpy(qkv).cuda())
        out, lse = out.cpu().numpy(), lse.cpu().numpy()
    for b in range(cfg.batch):
        for t in tiles:
            o, n = t["tok_off"], t["n_tok"]
            z = qkv[b, o:o + n].astype(np.float64)
            assert O.rel_l2(out[b, o:o + n], O.self_attention(z[:, :D], z[:, D:2 * D], z[:, 2 * D:], heads)) <= 1e-5
            for h in range(heads):
                s = z[:, h * dh:(h + 1) * dh] @ z[:, D + h * dh:D + (h + 1) * dh].T / np.sqrt(dh)
                ref = np.log(np.exp(s - s.max(1, keepdims=True)).sum(1)) + s.max(1)
                assert np.abs(lse[b, h, o:o + n] - ref).max() <= 1e-4


@pytest.mark.parametrize("D,which,rows,offset", [(4, 1, 1, 0), (36, 0, 33, 0), (36, 2, 65, 1), (100, 1, 31, 0), (128, 2, 20000, 0),
                                                 (100, 0, 9001, 1)], ids=str)
def test_input_gradient_of_a_linear_layer(D, which, rows, offset):
    cfg = BASE.with_(embed_dim=D, heads=1, mlp_ratio=2)
    w = WL.make_weights(cfg, std=0.1)
    n, k, name = ((3 * D, D, "w_qkv"), (D, D, "w_proj"), (2 * D, D, "w_fc1"))[which]
    buf = torch.randn(rows * n + 8, dtype=torch.float32, generator=torch.Generator().manual_seed(rows))
    dy = buf[offset:offset + rows * n].view(rows, n)
    ref = dy.double() @ torch.from_numpy(w[name][0]).double()
    with B.Reslim(cfg, w) as m:
        B.reslim_train_prepare(m.ctx)
        dyd = buf.cuda()[offset:offset + rows * n].view(rows, n)
        x = torch.zeros((rows, k), dtype=torch.float32, device="cuda")
        dx = torch.full((rows, k), float("nan"), dtype=torch.float32, device="cuda")
        dw, db = torch.empty((n, k), dtype=torch.float32, device="cuda"), torch.empty(n, dtype=torch.float32, device="cuda")
        ws = torch.empty(B.reslim_linear_bwd_workspace_bytes(m.ctx, which, rows), dtype=torch.uint8, device="cuda")
        B.reslim_linear_bwd(m.ctx, 0, which, x, dyd, dx, dw, db, rows, ws)
    assert float((dx.cpu().double() - ref).norm() / ref.norm()) <= 1e-5


def test_attention_with_infinities():
    """Scores that overflow to -inf have weight zero, also where a whole block of 32 keys does; an infinite value whose key
    has weight is an infinite output in its own feature and nowhere else, also at the ragged end of a tile."""
    cfg = BASE.with_(H=2 * 9, W=2 * 15)                     # 135 keys: the last block holds seven
    n, D, dh = 135, 64, 32
    r = np.random.default_rng(9)
    qkv = r.standard_normal((cfg.batch, n, 3 * D)).astype(np.float32)
    qkv[0, :, :dh] = np.abs(qkv[0, :, :dh])
    qkv[0, 32:64, D:D + dh] = -np.inf                       # head 0, second block of keys
    qkv[0, 128:, D:D + dh] = -np.inf                        # head 0, last block: after the first of the same wave
    qkv[0, :32, D:D + dh] = -np.inf                         # and that one too
    qkv[1, n - 1, 2 * D + 3] = np.inf
    with B.Reslim(cfg, WL.make_weights(cfg)) as m:
        assert m.n_h == n
        out = m.attention_with_lse(torch.from_numpy(qkv).cuda())[0].cpu().numpy()
    z = qkv[0].astype(np.float64)
    keys = [k for k in range(n) if 64 <= k < 128]
    s = z[:, :dh] @ z[keys, D:D + dh].T / np.sqrt(dh)
    p = np.exp(s - s.max(1, keepdims=True))
    assert O.rel_l2(out[0, :, :dh], p @ z[keys, 2 * D:2 * D + dh] / p.sum(1, keepdims=True)) <= 1e-5
    assert np.isposinf(out[1, :, 3]).all()
    assert np.isfinite(np.delete(out[1], 3, axis=1)).all()
