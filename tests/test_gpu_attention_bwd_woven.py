"""Gradient of tile attention at head dimensions 64 and 128 (attn_bwd_woven and attn_bwd_wide in csrc/attention_bwd.hip): one block of 32 streamed tokens, odd and even
numbers of them, as many as the ring has and more, a last block of one token, waves without tokens, tiles of several lengths in a
launch, more units of work than compute units, logits so low that the zeros past a tile's end would outweigh them."""
import numpy as np
import pytest
import torch

from oracle import reslim_oracle as O
from paper_2505_04802_amd import binding as B
from paper_2505_04802_amd import workloads as WL
from parity_checks import GRAD_BF16, assert_parity

pytestmark = pytest.mark.gpu
BASE = WL.ReslimConfig("woven", batch=1, in_vars=1, out_vars=1, H=2, W=2, scale=4, patch=2, embed_dim=128, heads=2, mlp_ratio=1, depth=1,
                       tiles_y=1, tiles_x=1, halo=0, dtype=1, seed=43)
# patches of the grid, tiles, halo: 1, 31, 32, 33, 64, 65, 96 tokens; 7, 8, 9 and 10 blocks; 128, 129 and 257 tokens; 12 to 49; 36 to 56 in 576 units; 672 to 784, 392 units of 448 slots
GRIDS = [(1, 3, 1, 3, 0), (31, 2, 1, 2, 0), (8, 8, 1, 2, 0), (3, 22, 1, 2, 0), (8, 16, 1, 2, 0), (5, 26, 1, 2, 0), (8, 12, 1, 1, 0), (8, 28, 1, 1, 0),
         (15, 17, 1, 1, 0), (16, 18, 1, 1, 0), (10, 30, 1, 1, 0), (8, 16, 1, 1, 0), (3, 43, 1, 1, 0), (1, 257, 1, 1, 0), (10, 14, 3, 4, 2),
         (60, 66, 12, 12, 1), (50, 170, 2, 8, 3)]


@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: "x".join(map(str, g)))
@pytest.mark.parametrize("kind", ["normal", "low"])
@pytest.mark.parametrize("dh", [64, 128])
def test_against_the_oracle(grid, kind, dh):
    print(f"woven attention gradient {grid} {kind} {dh}", flush=True)
    h, w, ty, tx, halo = grid
    cfg = BASE.with_(H=2 * h, W=2 * w, tiles_y=ty, tiles_x=tx, halo=halo, batch=2, embed_dim=2 * dh)
    tiles, _, _, n_h = O.tiles_partition(h, w, ty, tx, halo)
    D = cfg.embed_dim
    qkv = WL.make_qkv(2 * n_h, D, seed=8, peaked=kind == "normal", bf16=True).reshape(2, n_h, 3 * D).copy()
    first = np.arange(D) % dh < 4
    if kind == "low":                # every logit about 92 (65 at dimension 128) lower in base 2.  The gradients of those features are sums of dS, which add up to nothing,
        qkv[..., :D][..., first], qkv[..., D:2 * D][..., first] = 16.0, -8.0      # times a constant: rounding noise, left out below
    d_out = np.ascontiguousarray(WL.make_qkv(2 * n_h, D, seed=108, bf16=True)[:, :D]).reshape(2, n_h, D)
    ref = O.tiles_attention_bwd(qkv, d_out, tiles, cfg.heads)
    with B.Reslim(cfg, WL.make_weights(cfg)) as m:
        q, g = (torch.from_numpy(a.astype(np.float32)).cuda().to(m.act_dtype) for a in (qkv, d_out))
        out, lse = m.attention_with_lse(q)
        got, again = m.attention_bwd(q, out, lse, g), m.attention_bwd(q, out, lse, g)
    assert torch.equal(got, again)
    got = got.float().cpu().numpy()
    for name, s in (("dq", slice(0, D)), ("dk", slice(D, 2 * D)), ("dv", slice(2 * D, 3 * D))):
        keep = ~first if kind == "low" else slice(None)
        got_s, ref_s = got[..., s][..., keep], ref[..., s][..., keep]
        if np.abs(ref_s).max() < 1e-12:
            # one token a tile: P = 1 and the output is v, so dS = dP - delta is two fp32 sums of the same dh products in another order.  Of products of at most M
            # each of the dh additions is off by 2^-24 dh M at most, in either; dQ and dK are that times k or q, over sqrt(dh), rounded to bf16 twice.
            other = qkv[..., D:2 * D] if name == "dq" else qkv[..., :D]
            m = np.abs(d_out).max() * np.abs(qkv[..., 2 * D:]).max()
            bound = 2 * dh * dh * 2.0 ** -24 * m * np.abs(other[..., keep]).max() / np.sqrt(dh) * 1.01
            print(f"  {name}: {np.abs(got_s).max():.2e} (<= {bound:.2e})")
            assert np.abs(got_s).max() <= bound, name
        else:
            assert_parity(got_s, ref_s, 2e-2, name, print, **GRAD_BF16)
