"""More slots of work than one launch takes work-groups (2^32 threads a grid dimension): the forward with two query groups a wave and the gradient at
head dimension 64 (csrc/attention_plan.h)."""
import pytest
import torch

from paper_2505_04802_amd import binding as B
from paper_2505_04802_amd import workloads as WL

pytestmark = pytest.mark.gpu
CFG = WL.ReslimConfig("many", batch=1, in_vars=1, out_vars=1, H=128, W=256, scale=4, patch=2, embed_dim=2048, heads=32, mlp_ratio=1, depth=1,
                      tiles_y=64, tiles_x=128, halo=0, dtype=1, seed=3)


@pytest.mark.parametrize("batch", [64, 128])        # 2^24 slots: one work-group too many for the gradient's 256 threads; 2^25: for the forward's 128 as well
def test_tiles_of_one_token(batch):
    """A token alone is its own softmax: the output is v, its gradient passes to v, and nothing passes to q and k."""
    print(f"attention of {batch} x 8192 tiles of one token, 32 heads", flush=True)
    D = CFG.embed_dim
    g = torch.Generator(device="cuda").manual_seed(batch)
    with B.Reslim(CFG, WL.make_weights(CFG)) as m:
        assert batch * m.n_h * CFG.heads >= 2 ** 24
        qkv = torch.empty((batch, m.n_h, 3 * D), dtype=m.act_dtype, device="cuda").normal_(generator=g)
        d_out = torch.empty((batch, m.n_h, D), dtype=m.act_dtype, device="cuda").normal_(generator=g)
        out = torch.empty_like(d_out)
        lse = torch.empty((batch, CFG.heads, m.n_h), dtype=torch.float32, device="cuda")
        for variant in (0, 3, 4):                    # by the rule; two query groups a wave, in work-groups of two waves and of four
            B.reslim_debug_set_attention_variant(variant)
            try:
                B.tiles_attention_fwd_lse(m.ctx, qkv, out.zero_(), lse, batch)
            finally:
                B.reslim_debug_set_attention_variant(0)
            assert torch.equal(out, qkv[..., 2 * D:]), variant
        d_qkv = torch.empty_like(qkv)
        ws = torch.empty(B.tiles_attention_bwd_workspace_bytes(m.ctx, batch), dtype=torch.uint8, device="cuda")
        B.tiles_attention_bwd(m.ctx, qkv, out, lse, d_out, d_qkv, batch, ws)
        assert torch.equal(d_qkv[..., 2 * D:], d_out)
        # dS = P (dO . V - delta), two fp32 sums of the same 64 products of at most 6^2 in another order: off by 64 * 36 * 64 * 2^-24 at most, times q or k of at most 6
        assert all(d_qkv[b, :, :2 * D].abs().max() <= 6 * 64 * 36 * 64 * 2.0 ** -24 for b in range(0, batch, 9))
