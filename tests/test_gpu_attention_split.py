"""Tile attention with the keys split over the waves (csrc/attention.hip), taken for few queries and at least 512 tokens: blocks of 32
keys that do not divide among four waves, a last block of one key, a wave whose keys have far smaller logits than the others',
the log-sum-exp, halo copies (stitched output).  The neighbours of the rule run the other kernel."""
import numpy as np
import pytest
import torch

from oracle import reslim_oracle as O
from paper_2505_04802_amd import binding as B
from paper_2505_04802_amd import workloads as WL
from parity_checks import assert_parity

pytestmark = pytest.mark.gpu
BASE = WL.ReslimConfig("split", batch=1, in_vars=1, out_vars=1, H=32, W=64, scale=4, patch=2, embed_dim=128, heads=2, mlp_ratio=2, depth=2,
                       tiles_y=1, tiles_x=1, halo=0, dtype=1, seed=33)
CASES = [BASE,                                                              # 512 tokens: 16 blocks
         BASE.with_(name="t513", H=54, W=38),                               # 27 x 19 = 513: a last block of one key
         BASE.with_(name="t627_b2", batch=2, H=66, W=38),                   # 33 x 19 = 627: 20 blocks
         BASE.with_(name="ragged_tiles", H=70, W=66, tiles_y=1, tiles_x=2, halo=1),      # 35 x 17 = 595 and 35 x 18 = 630
         BASE.with_(name="long", H=120, W=124)]                             # 3720 tokens, 60 units


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
@pytest.mark.parametrize("kind", ["normal", "peaked", "one_quarter"])
def test_against_the_oracle(cfg, kind):
    print(f"split attention {cfg.name} {kind}", flush=True)
    tiles, _, _, n_h = O.tiles_partition(cfg.Hp, cfg.Wp, cfg.tiles_y, cfg.tiles_x, cfg.halo)
    D = cfg.embed_dim
    qkv = WL.make_qkv(cfg.batch * n_h, D, seed=5, peaked=kind == "peaked", bf16=True).reshape(cfg.batch, n_h, 3 * D)
    if kind == "one_quarter":      # only the keys of one wave of the four count: 29 in base-2 logits above the rest
        qkv[..., :D] = 4.0
        blk = np.arange(n_h) // 32 % 4
        qkv[..., D:2 * D] = np.where(blk == 2, 0.5, -0.125)[None, :, None]
    ref = O.tiles_attention(qkv, tiles, cfg.heads)
    with B.Reslim(cfg, WL.make_weights(cfg)) as m:
        act = torch.from_numpy(qkv.astype(np.float32)).cuda().to(m.act_dtype)
        out = m.attention(act)
        out2, lse = m.attention_with_lse(act)
        B.reslim_debug_set_attention_variant(1)                            # the kernel without the split
        try:
            other = m.attention(act)
        finally:
            B.reslim_debug_set_attention_variant(0)
        again = m.attention(act)
    assert torch.equal(out, out2) and torch.equal(out, again)
    assert_parity(out.float().cpu().numpy(), ref, 2e-2, "attention", print)
    # both kernels round P and the output to bf16 relative to other references: 2^-8 each at most
    assert_parity(other.float().cpu().numpy(), out.float().cpu().numpy(), 2.0 ** -7, "against the kernel without the split", print)
    scale = 1.0 / np.sqrt(D // cfg.heads)
    for t in tiles[:1]:
        s = slice(int(t["tok_off"]), int(t["tok_off"]) + int(t["n_tok"]))
        for h in range(cfg.heads):
            f = slice(h * 64, h * 64 + 64)
            logits = (qkv[0, s, :D][:, f].astype(np.float64) @ qkv[0, s, D:2 * D][:, f].astype(np.float64).T) * scale
            want = np.log(np.exp(logits - logits.max(1, keepdims=True)).sum(1)) + logits.max(1)
            # the sum is of probabilities rounded to bf16 (8 significant bits: up to 2^-8 of each), beside 1e-5 of the fp32 arithmetic
            assert np.abs(lse[0, h, s].cpu().numpy() - want).max() <= 2.0 ** -8 + 1e-5 * np.abs(want).max()


def test_whole_forward_with_halo_copies():
    """Stitched output, q scaled by the QKV epilogue; the chain of entry points runs the same kernel unstitched."""
    cfg = CASES[3]
    w, x = WL.make_weights(cfg, std=0.1), WL.make_fields(cfg)
    y_ref = O.reslim_forward(x, w, cfg)
    with B.Reslim(cfg, w) as m:
        xd = torch.from_numpy(x).cuda()
        tok = m.embed(xd)
        for l in range(cfg.depth):
            m.block(l, tok)
        y_chain, y = m.head(xd, tok).cpu().numpy(), m.forward(xd).cpu().numpy()
    assert np.array_equal(y, y_chain)
    assert_parity(y, y_ref, 2e-2, "forward", print)
