"""Tile attention with two query groups a wave (csrc/attention.hip), taken for launches of many blocks of queries: waves and groups without
queries, one block of keys and several, a last block of one key, references that move in the middle, keys past the end that
would outweigh the real ones, the log-sum-exp, halo copies (stitched output)."""
import numpy as np
import pytest
import torch

from oracle import reslim_oracle as O
from paper_2505_04802_amd import binding as B
from paper_2505_04802_amd import workloads as WL
from parity_checks import assert_parity

pytestmark = pytest.mark.gpu
BASE = WL.ReslimConfig("pair", batch=1, in_vars=1, out_vars=1, H=2, W=2, scale=4, patch=2, embed_dim=1024, heads=16, mlp_ratio=1, depth=1,
                       tiles_y=1, tiles_x=1, halo=0, dtype=1, seed=41)


def tiled(h, w, ty, tx, **other):
    """ty x tx tiles; h x w patches each where they divide"""
    return BASE.with_(name=f"{h}x{w}_{ty}x{tx}_{'_'.join(map(str, other.values()))}", H=2 * h, W=2 * w, tiles_y=ty, tiles_x=tx, **other)


# 768 blocks of 128 queries and more, in tiles that fill blocks of 256 as well, or leave a tenth of the waves idle at most: four waves in a work-group
FOUR = [tiled(3, 43 * 25, 1, 25),                           # 129: no query for the fourth wave, one for the third
        tiled(8, 20 * 25, 1, 25),                           # 160: five whole blocks of keys, none in the third wave's second group
        tiled(7, 23 * 25, 1, 25),                           # 161: a last block of one key
        tiled(15, 15 * 25 + 9, 1, 25),                      # 225 and 240: one query in the last group
        tiled(16, 16 * 13, 1, 13, batch=2),                 # 256
        tiled(60, 84, 2, 3, batch=3, halo=2)]               # 32 by 30 to 32
# 8192 blocks and more, a twentieth fewer waves than with four at least: two, where a tile has more than 40 tokens (tests/test_attention_plan_cpu.py holds both lists against the rule)
TWO = [tiled(n, 128, 1, 128, embed_dim=4096, heads=64) for n in (1, 33, 65)] + [tiled(257, 43, 1, 43, embed_dim=4096, heads=64)]


def qkv_of(cfg, n_h, kind):
    D = cfg.embed_dim
    x = WL.make_qkv(cfg.batch * n_h, D, seed=6, peaked=kind == "peaked", bf16=True).reshape(cfg.batch, n_h, 3 * D).copy()
    tok = np.arange(n_h)
    if kind == "moving":           # every seventh query meets a logit 13 times as large at every 37th key, 104 in base 2
        x[:, tok % 7 == 3, :D] = 3.0
        x[:, :, D:2 * D] *= 0.25
        x[:, tok % 37 == 36, D:2 * D] = 3.0
    if kind == "low":              # every logit is about -100 in base 2: a zero would be all there is
        x[..., :D], x[..., D:2 * D] = 3.0, -3.0 + 0.25 * np.sign(x[..., D:2 * D])
    if kind == "stairs":           # queries that meet a logit 11 above their last largest (base 2) every 64 keys: in the first 32 of them, in the others, in both
        f = np.arange(D) % 64
        x[..., :D][..., f < 2] = x[..., D:2 * D][..., f < 2] = 0.0
        for first, key, queries in ((0, 8, (1, 3)), (1, 40, (2, 3))):
            x[:, np.ix_(np.isin(tok % 5, queries), f == first)[0], np.flatnonzero(f == first)] = 8.0
            at = tok[tok % 64 == key]
            x[:, at[:, None], D + np.flatnonzero(f == first)] = (8.0 * (1 + at // 64))[None, :, None]
    return x


@pytest.mark.parametrize("cfg,kind", [(c, k) for c in FOUR for k in ("normal", "peaked", "moving", "low")] +
                         [(c, k) for c in TWO for k in ("moving", "low")], ids=lambda v: v if isinstance(v, str) else v.name)
def test_against_the_oracle(cfg, kind):
    print(f"pair attention {cfg.name} {kind}", flush=True)
    tiles, _, _, n_h = O.tiles_partition(cfg.Hp, cfg.Wp, cfg.tiles_y, cfg.tiles_x, cfg.halo)
    D = cfg.embed_dim
    qkv = qkv_of(cfg, n_h, kind)
    with B.Reslim(cfg, WL.make_weights(cfg)) as m:
        act = torch.from_numpy(qkv.astype(np.float32)).cuda().to(m.act_dtype)
        out = m.attention(act)
        out2, lse = m.attention_with_lse(act)
        B.reslim_debug_set_attention_variant(1)                            # one query group a wave
        try:
            other = m.attention(act)
        finally:
            B.reslim_debug_set_attention_variant(0)
    assert torch.equal(out, out2)
    some = tiles if cfg in FOUR else tiles[:2]                             # tiles never interact
    rows = slice(0, int(some[-1]["tok_off"]) + int(some[-1]["n_tok"]))
    ref = O.tiles_attention(qkv[:, rows], some, cfg.heads)
    # an element: the usual 0.05 rms, and half a unit in the last place of the largest output (2^-8 of it; a query whose softmax falls on one
    # key has outputs 12 times the rms of those that average over 384)
    elem = 0.05 + 2.0 ** -8 * np.abs(ref).max() / np.sqrt((ref ** 2).mean())
    assert_parity(out[:, rows].float().cpu().numpy(), ref, 2e-2, "attention", print, k_elem=elem)
    # both kernels round P and the output to bf16 relative to other references: 2^-8 each at most
    assert_parity(other.float().cpu().numpy(), out.float().cpu().numpy(), 2.0 ** -7, "against one group a wave", print, k_elem=elem)
    t = some[-1]
    s = slice(int(t["tok_off"]), int(t["tok_off"]) + int(t["n_tok"]))
    for h in (0, cfg.heads - 1):
        f = slice(h * 64, h * 64 + 64)
        logits = (qkv[-1, s, :D][:, f].astype(np.float64) @ qkv[-1, s, D:2 * D][:, f].astype(np.float64).T) / 8.0
        want = np.log(np.exp(logits - logits.max(1, keepdims=True)).sum(1)) + logits.max(1)
        # the sum is of probabilities rounded to bf16 (8 significant bits: up to 2^-8 of each), beside 1e-5 of the fp32 arithmetic
        assert np.abs(lse[-1, h, s].cpu().numpy() - want).max() <= 2.0 ** -8 + 1e-5 * np.abs(want).max()


def test_stitched_output_is_the_same_bits():
    """The last block of a whole forward writes the owned queries alone; the chain of entry points runs the same kernel unstitched."""
    cfg = FOUR[-1].with_(depth=2)
    w, x = WL.make_weights(cfg, std=0.1), torch.from_numpy(WL.make_fields(cfg)).cuda()
    with B.Reslim(cfg, w) as m:
        tok = m.embed(x)
        for l in range(cfg.depth):
            m.block(l, tok)
        assert torch.equal(m.forward(x), m.head(x, tok))


@pytest.mark.parametrize("scale", [0.3, 3.0, 9.0])      # no reference moves after the first keys; some do; most do
def test_the_same_bits_as_with_one_group_a_wave(scale):
    """A batch takes the kernel with two groups, its samples one by one the kernel with one: what a query gets does not depend on it."""
    cfg = BASE.with_(batch=4, H=128, W=256, tiles_y=4, tiles_x=4, halo=2, embed_dim=512, heads=8)
    _, _, _, n_h = O.tiles_partition(cfg.Hp, cfg.Wp, 4, 4, 2)
    qkv = WL.make_qkv(cfg.batch * n_h, 512, seed=9, bf16=True).reshape(cfg.batch, n_h, 1536).astype(np.float32)
    qkv[..., :512] *= scale
    with B.Reslim(cfg, WL.make_weights(cfg)) as m:
        act = torch.from_numpy(qkv).cuda().to(m.act_dtype)
        out, lse = m.attention_with_lse(act)
        parts = [m.attention_with_lse(act[b:b + 1].contiguous()) for b in range(cfg.batch)]
    assert torch.equal(out, torch.cat([p[0] for p in parts])) and torch.equal(lse, torch.cat([p[1] for p in parts]))


SHORT = [tiled(n, 3 * 16, 1, 48) for n in (1, 31, 32, 33, 63, 64, 65, 96, 97, 128)]
EDGES = SHORT + [tiled(n, 25, 1, 25) for n in (129, 160, 161, 255, 256, 257)] + [FOUR[-1]]


@pytest.mark.parametrize("kind", ["normal", "moving", "low", "stairs"])
@pytest.mark.parametrize("cfg", EDGES, ids=lambda c: c.name)
def test_the_same_bits_in_every_kernel(cfg, kind):
    """One query group a wave and two, in work-groups of two waves and of four: by the rule, launches of one size or another get them."""
    print(f"attention kernels beside each other {cfg.name} {kind}", flush=True)
    _, _, _, n_h = O.tiles_partition(cfg.Hp, cfg.Wp, cfg.tiles_y, cfg.tiles_x, cfg.halo)
    with B.Reslim(cfg, WL.make_weights(cfg)) as m:
        act = torch.from_numpy(qkv_of(cfg, n_h, kind).astype(np.float32)).cuda().to(m.act_dtype)
        try:
            got = []
            for variant in (2, 3, 4):
                B.reslim_debug_set_attention_variant(variant)
                got.append(m.attention_with_lse(act))
        finally:
            B.reslim_debug_set_attention_variant(0)
    assert all(torch.isfinite(t.float()).all() for t in got[0])
    for other in got[1:]:
        assert all(torch.equal(a, b) for a, b in zip(got[0], other))


@pytest.mark.parametrize("std", [0.02, 0.3])
@pytest.mark.parametrize("cfg", [FOUR[-1].with_(depth=2, embed_dim=256, heads=4, batch=2), tiled(9, 42, 1, 3, halo=2, embed_dim=128, heads=2).with_(depth=2)],
                         ids=lambda c: c.name)
def test_a_forward_is_the_same_bits_with_every_kernel(cfg, std):
    """q scaled by the QKV epilogue; the last block's output stitched."""
    print(f"forward with each attention kernel {cfg.name} {std}", flush=True)
    w, x = WL.make_weights(cfg, std=std), torch.from_numpy(WL.make_fields(cfg)).cuda()
    with B.Reslim(cfg, w) as m:
        try:
            got = []
            for variant in (2, 3, 4):
                B.reslim_debug_set_attention_variant(variant)
                got.append(m.forward(x).clone())
        finally:
            B.reslim_debug_set_attention_variant(0)
    assert torch.isfinite(got[0]).all() and torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])


@pytest.mark.parametrize("dh", [128, 256])
@pytest.mark.parametrize("n", [1, 8, 31, 33, 40, 64, 65, 100, 129])
def test_wide_heads_in_short_tiles(n, dh):
    """Blocks of keys that the tile ends in (rows past its end are its last row again), beside whole ones; logits so low that anything else there would be all there is."""
    print(f"attention at head dimension {dh}, tiles of {n} tokens", flush=True)
    cfg = tiled(n, 4, 1, 4, embed_dim=2 * dh, heads=2)
    tiles, _, _, n_h = O.tiles_partition(cfg.Hp, cfg.Wp, 1, 4, 0)
    for kind in ("normal", "low"):
        qkv = qkv_of(cfg, n_h, kind)
        with B.Reslim(cfg, WL.make_weights(cfg)) as m:
            out = m.attention(torch.from_numpy(qkv.astype(np.float32)).cuda().to(m.act_dtype)).float().cpu().numpy()
        ref = O.tiles_attention(qkv, tiles, 2)
        elem = 0.05 + 2.0 ** -8 * np.abs(ref).max() / np.sqrt((ref ** 2).mean())      # as above
        assert_parity(out, ref, 2e-2, "attention", print, k_elem=elem)
