"""The loss and its gradient on rows of every remainder and alignment, for each number of rows a thread of the gradient takes
(one, two, eight), in one work-group a row and in several; the gradient writes its own elements and no others."""
import numpy as np
import pytest
import torch

from oracle import reslim_oracle as O
from oracle import train_oracle as TO
from paper_2505_04802_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [0, 1, 2, 3])
@pytest.mark.parametrize("shape", [(1, 1, 1, 1), (1, 2, 3, 3), (1, 1, 9, 6), (2, 1, 5, 1027), (1, 2, 9, 2050), (1, 24, 300, 7), (2, 12, 299, 258),
                                   (1, 24, 701, 131), (1, 24, 702, 132)], ids=str)
def test_rows(shape, offset):
    print(f"loss rows {shape} offset {offset}", flush=True)
    r = np.random.default_rng([offset, *shape])
    n = int(np.prod(shape))
    pred = (r.integers(-8, 9, shape) / 4).astype(np.float32)            # many equal neighbours
    target = r.standard_normal(shape).astype(np.float32)
    lw = O.lat_weights(shape[2], -80.0, 85.0).astype(np.float32)
    def place(a):
        buf = torch.zeros(n + 8, dtype=torch.float32, device="cuda")
        buf[offset:offset + n] = torch.from_numpy(a).cuda().flatten()
        return buf[offset:offset + n].view(shape)
    p, t, l = place(pred), place(target), torch.from_numpy(lw).cuda()
    out = torch.zeros(3, dtype=torch.float64, device="cuda")
    ws = torch.empty(max(B.reslim_bayes_loss_workspace_bytes(*shape), 8), dtype=torch.uint8, device="cuda")
    B.reslim_bayes_loss_fwd(p, t, l, 0.25, out, ws)
    ref = O.bayes_loss(pred, target, lw, tv_weight=0.25)
    assert np.allclose(out.cpu().numpy(), np.asarray(ref, dtype=np.float64), rtol=1e-5)      # 32-bit sums of up to 32 terms a thread
    d = torch.full((n + 8,), float("nan"), dtype=torch.float32, device="cuda")
    B.reslim_bayes_loss_bwd(p, t, l, 0.25, 8.0, d[offset:offset + n].view(shape))
    d = d.cpu().numpy()
    assert np.isnan(d[:offset]).all() and np.isnan(d[offset + n:]).all()
    assert O.rel_l2(d[offset:offset + n].reshape(shape), TO.bayes_loss_bwd(pred, target, lw, 0.25) * 8.0) <= 1e-6


@pytest.mark.parametrize("shape", [(1, 3072, 2, 3), (1, 3073, 8, 4), (2, 2047, 2, 4), (1, 4096, 3, 4), (1, 4097, 8, 4), (1, 7168, 2, 3), (1, 8191, 3, 5),
                                   (4, 2049, 1, 2)], ids=str)
def test_many_partial_sums(shape):
    """A partial sum a plane: from 3073 of them on a thread of the last kernel takes four at once while there is a fourth, then up to
    three singly.  One of them left out or taken twice is 1e-4 of the value."""
    print(f"loss partial sums {shape}", flush=True)
    r = np.random.default_rng(shape)
    pred = (r.integers(-8, 9, shape) / 4).astype(np.float32)
    target = (pred + 1.0 + 0.25 * r.standard_normal(shape)).astype(np.float32)
    lw = O.lat_weights(shape[2], -80.0, 85.0).astype(np.float32)
    assert B.reslim_bayes_loss_workspace_bytes(*shape) == 16 * shape[0] * shape[1]
    out = torch.zeros(3, dtype=torch.float64, device="cuda")
    ws = torch.empty(16 * shape[0] * shape[1], dtype=torch.uint8, device="cuda")
    B.reslim_bayes_loss_fwd(torch.from_numpy(pred).cuda(), torch.from_numpy(target).cuda(), torch.from_numpy(lw).cuda(), 0.25, out, ws)
    ref = np.asarray(O.bayes_loss(pred, target, lw, tv_weight=0.25), dtype=np.float64)
    assert np.allclose(out.cpu().numpy(), ref, rtol=1e-5)
