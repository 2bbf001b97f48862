"""Tile attention with a query that is not finite (csrc/attention.hip): its own row is not a number, every other row keeps its bits, in every
bf16 kernel.  A query that shares a column of the row sums' matrix instruction with it (16 further on) is the one that would show.  And a query whose
first 32 or 64 logits overflow to -inf: it gets the softmax over the other keys."""
import numpy as np
import pytest
import torch

from oracle import reslim_oracle as O
from paper_2505_04802_amd import binding as B
from paper_2505_04802_amd import workloads as WL

pytestmark = pytest.mark.gpu
BASE = WL.ReslimConfig("nonfinite", batch=1, in_vars=1, out_vars=1, H=2, W=2, scale=4, patch=2, embed_dim=128, heads=2, mlp_ratio=1, depth=1,
                       tiles_y=1, tiles_x=1, halo=0, dtype=1, seed=47)


def tiled(name, h, w, tx, dh, heads):
    return BASE.with_(name=name, H=2 * h, W=2 * w, tiles_x=tx, embed_dim=dh * heads, heads=heads)


# a tile has more than 64 tokens, so that a reference is set in one block and used in another, and ends within a block
ONE = tiled("one_group", 70, 2, 2, 64, 2)
KERNELS = [(ONE, 0), (tiled("two_groups_four_waves", 7, 23 * 25, 25, 64, 16), 0), (tiled("two_groups_two_waves", 65, 128, 128, 64, 64), 0),
           (tiled("keys_split", 27, 19, 1, 64, 2), 0), (tiled("blocks_of_128", 70, 2, 2, 64, 2), 1), (tiled("dh128", 70, 2, 2, 128, 2), 0),
           (tiled("dh256", 70, 2, 2, 256, 2), 0)]
QUERIES = (5, 21, 37)       # partners in the row sums, and one of another wave or group


def run(cfg, variant, *inputs):
    """(output, log-sum-exp) of each"""
    with B.Reslim(cfg, WL.make_weights(cfg)) as m:
        B.reslim_debug_set_attention_variant(variant)
        try:
            return [tuple(t.float().cpu().numpy() for t in m.attention_with_lse(torch.from_numpy(x).cuda().to(m.act_dtype))) for x in inputs]
        finally:
            B.reslim_debug_set_attention_variant(0)


def inputs(cfg):
    _, _, _, n_h = O.tiles_partition(cfg.Hp, cfg.Wp, cfg.tiles_y, cfg.tiles_x, cfg.halo)
    return WL.make_qkv(n_h, cfg.embed_dim, seed=12, bf16=True).reshape(1, n_h, 3 * cfg.embed_dim).astype(np.float32)


@pytest.mark.parametrize("kind", ["nan", "overflow"])
@pytest.mark.parametrize("cfg,variant", KERNELS, ids=lambda v: getattr(v, "name", None))
def test_a_query_that_is_not_finite_keeps_to_itself(cfg, variant, kind):
    print(f"attention, a query {kind}: {cfg.name}", flush=True)
    qkv, dh = inputs(cfg), cfg.embed_dim // cfg.heads
    spoilt = []
    for query in QUERIES:
        spoilt.append(qkv.copy())
        spoilt[-1][0, query, dh] = np.nan if kind == "nan" else 3e38      # of head 1; with 3e38 the logits of keys above 1.2 there are +inf
    clean, *others = run(cfg, variant, qkv, *spoilt)
    assert np.isfinite(clean[0]).all() and np.isfinite(clean[1]).all()
    for query, (out, lse) in zip(QUERIES, others):
        own, own_lse = np.zeros(out.shape, bool), np.zeros(lse.shape, bool)
        own[0, query, dh:2 * dh] = own_lse[0, 1, query] = True
        assert np.isnan(out[own]).all() and np.isnan(lse[own_lse]).all(), query
        assert np.array_equal(out[~own], clean[0][~own]) and np.array_equal(lse[~own_lse], clean[1][~own_lse]), query


@pytest.mark.parametrize("dead", [32, 64])
@pytest.mark.parametrize("cfg,variant", [k for k in KERNELS if k[0].name != "keys_split"], ids=lambda v: getattr(v, "name", None))
def test_first_keys_that_overflow_downwards_have_no_weight(cfg, variant, dead):
    """The kernel that splits the keys gives each wave a reference of its own and needs a finite logit among a wave's first 32 keys."""
    print(f"attention, first {dead} keys at -inf: {cfg.name}", flush=True)
    qkv, D, dh, n = inputs(cfg), cfg.embed_dim, cfg.embed_dim // cfg.heads, cfg.Hp * (cfg.Wp // cfg.tiles_x)
    qkv[..., dh] = qkv[..., D + dh] = 0.0                      # feature 0 of head 1 decides alone
    qkv[0, :dead, D + dh] = -3e38
    calm = qkv.copy()
    qkv[0, QUERIES[0], dh] = 3e38
    clean, (out, lse) = run(cfg, variant, calm, qkv)
    own, own_lse = np.zeros(out.shape, bool), np.zeros(lse.shape, bool)
    own[0, QUERIES[0], dh:2 * dh] = own_lse[0, 1, QUERIES[0]] = True
    assert np.array_equal(out[~own], clean[0][~own]) and np.array_equal(lse[~own_lse], clean[1][~own_lse])
    q, k, v = (qkv[0, :n, i * D + dh:i * D + 2 * dh].astype(np.float64) for i in range(3))
    logits = k[dead:] @ q[QUERIES[0]] / np.sqrt(dh)
    p = np.exp(logits - logits.max())
    want = p @ v[dead:] / p.sum()
    # probabilities and the output are rounded to bf16: 2^-9 of each at most, of a row whose probabilities are positive
    assert np.abs(out[own] - want).max() <= 2.0 ** -8 * np.abs(v).max()
    assert abs(lse[own_lse][0] - (np.log(p.sum()) + logits.max())) <= 2.0 ** -8
