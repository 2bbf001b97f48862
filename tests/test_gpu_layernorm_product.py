"""The fp32 product that normalises its rows itself (csrc/gemm.hip, gemm_f32_kernel with LN): rows of one step and of the most a
wave holds, lengths that leave a half step or whole waves without work, one row and a remainder of rows, rows through a map (the head
under tiles), and the neighbours that keep a LayerNorm launch (more than 256 features).  Every stage against the oracle."""
import numpy as np
import pytest
import torch

from oracle import reslim_oracle as O
from paper_2505_04802_amd import binding as B
from paper_2505_04802_amd import workloads as WL
from parity_checks import assert_parity

pytestmark = pytest.mark.gpu
BASE = WL.ReslimConfig("lnp", batch=1, in_vars=2, out_vars=1, H=10, W=14, scale=2, patch=2, embed_dim=64, heads=1, mlp_ratio=2, depth=1,
                       tiles_y=1, tiles_x=1, halo=0, dtype=0, seed=17)


@pytest.mark.parametrize("D", [4, 12, 36, 128, 252, 256, 260])
@pytest.mark.parametrize("grid", [dict(H=2, W=2), dict(), dict(H=22, W=26, batch=2, tiles_y=2, tiles_x=2, halo=1)], ids=["one_row", "35_rows", "tiles"])
def test_block_and_head(D, grid):
    cfg = BASE.with_(embed_dim=D, **grid)
    print(f"fp32 product with LayerNorm D={D} {grid}", flush=True)
    w, x = WL.make_weights(cfg, std=0.1), WL.make_fields(cfg)
    y_ref, inter = O.reslim_forward(x, w, cfg, return_intermediates=True)
    with B.Reslim(cfg, w) as m:
        t = torch.from_numpy(inter["tokens"].astype(np.float32)).cuda()
        m.block(0, t)
        assert_parity(t.cpu().numpy(), inter["block0"], 1e-5, "block", print)
        xd = torch.from_numpy(x).cuda()
        assert_parity(m.head(xd, torch.from_numpy(inter["block0"].astype(np.float32)).cuda()).cpu().numpy(), y_ref, 1e-5, "head", print)
        assert_parity(m.forward(xd).cpu().numpy(), y_ref, 1e-5, "forward", print)


@pytest.mark.parametrize("cfg", [WL.CONFIGS["c0"], WL.CONFIGS["m9m"]], ids=lambda c: c.name)
def test_every_launch_record_has_a_time(cfg):
    """A launch that does several steps leaves a record for each, and a rate is computed from every record's time: none may be zero."""
    w, x = WL.make_weights(cfg), torch.from_numpy(WL.make_fields(cfg)).cuda()
    with B.Reslim(cfg, w) as m:
        B.reslim_profile_enable(m.ctx, 256)
        m.forward(x)
        torch.cuda.synchronize()
        recs, launch = B.reslim_profile_read(m.ctx), B.reslim_profile_launches(m.ctx)
        B.reslim_profile_enable(m.ctx, 0)
    assert recs and all(ms > 0 for _, ms, _, _ in recs), recs
    # records of one launch are adjacent and named; the launches are those of a forward
    assert len(launch) == len(recs) and launch[0] == 0 and all(b - a in (0, 1) for a, b in zip(launch, launch[1:]))
    names = ["+".join(r[0] for r, k in zip(recs, launch) if k == i) for i in range(launch[-1] + 1)]
    if cfg.dtype == 0:
        block = ["layernorm+gemm_qkv", "tiles_attention", "gemm_proj", "layernorm+gemm_fc1", "gemm_fc2"]
        assert names == ["embed_agg", "gemm_agg_out", "gather"] + block * cfg.depth + ["layernorm_final+gemm_head", "residual_unpatchify"]
    else:
        mlp = "gemm_proj+layernorm+gemm_fc1+gemm_fc2"
        assert names == (["embed_agg", "gemm_agg_out", "layernorm", "gemm_qkv"] + ["tiles_attention", mlp + "+layernorm+gemm_qkv"] * (cfg.depth - 1) +
                         ["tiles_attention", mlp, "layernorm_final", "gemm_head", "residual_unpatchify"])
