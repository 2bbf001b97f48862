"""The folded aggregation on fp32 matrix instructions (csrc/elementwise.hip), where it can go wrong: patches that fill a
work-group of 32 or 64 and one more or less, one variable, odd and even numbers, heads taken in several groups with fewer at the end, the
three head dimensions, features that leave waves idle, variables so many that the vector kernel takes over."""
import pytest
import torch

from oracle import reslim_oracle as O
from paper_2505_04802_amd import binding as B
from paper_2505_04802_amd import workloads as WL
from parity_checks import assert_parity

pytestmark = pytest.mark.gpu


def _cfg(hp, wp, batch, variables, heads, dh):
    return WL.ReslimConfig(f"embed_{batch}x{hp}x{wp}_v{variables}_h{heads}x{dh}", batch=batch, in_vars=variables, out_vars=1, H=2 * hp, W=2 * wp,
                           scale=8, patch=2, embed_dim=heads * dh, heads=heads, mlp_ratio=1, depth=1, tiles_y=1, tiles_x=1, halo=0, dtype=1, seed=83)


CASES = [_cfg(4, 8, 1, 1, 1, 64), _cfg(3, 11, 1, 2, 2, 64), _cfg(1, 31, 3, 3, 5, 64), _cfg(8, 8, 1, 23, 4, 64),
         _cfg(5, 13, 1, 30, 11, 64), _cfg(5, 7, 2, 7, 3, 128), _cfg(9, 7, 1, 33, 5, 128), _cfg(4, 9, 1, 6, 2, 256), _cfg(5, 9, 1, 150, 4, 64),
         _cfg(3, 5, 1, 200, 4, 64), _cfg(128, 512, 1, 3, 2, 64), _cfg(255, 257, 1, 4, 3, 64), _cfg(257, 257, 1, 1, 1, 128),
         _cfg(129, 509, 1, 9, 5, 64),
         # both sides of the rule that chooses the kernel (csrc/embed_plan.h): at 192, 256, 512 and 1024 features, the last by the patches too
         _cfg(1, 31, 3, 3, 3, 64), _cfg(4, 8, 1, 2, 1, 64), _cfg(5, 9, 1, 1, 4, 64), _cfg(4, 9, 1, 6, 4, 128), _cfg(4, 9, 1, 7, 2, 256),
         _cfg(7, 9, 2, 8, 8, 128), _cfg(3, 21, 1, 32, 16, 64), _cfg(125, 128, 1, 8, 16, 64), _cfg(5, 11, 1, 23, 24, 128)]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_embedding_against_the_oracle(cfg):
    """Tokens = aggregation times W_o plus tables: the aggregation's output and W_o are rounded to bf16, 2^-9 of a value at most
    each, so 2^-8 bounds the 2-norm of plane and rows with room for fp32 sums."""
    print(f"embed {cfg.name}", flush=True)
    w, x = WL.make_weights(cfg, std=0.1), WL.make_fields(cfg)
    with B.Reslim(cfg, w) as m:
        got = m.embed(torch.from_numpy(x).cuda()).cpu().numpy()
    ref = O.embed_tokens(x, w, cfg.patch, cfg.heads, cfg.res_idx)
    assert_parity(got, ref, 2.0 ** -8, "embedding", print)
