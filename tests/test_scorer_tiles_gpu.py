"""Scorer gradients at the edges of the row tiles (32 rows up to 16,384, 64
beyond) and of the chunks the weight gradients are summed in, against the FP64
reference with the same BF16 rounding points.

Tolerance: FP32 sums in another order move a product by ~1e-6 of its size,
which now and then tips one BF16 rounding (2^-8 of that value); with up to one
in 16 values tipped a block's error stays below 2^-8 / 4 = 1e-3 of its norm,
and one element's below 2^-8 of the block's largest."""
import numpy as np
import pytest

from oracle import mlp as M
from tests.test_scorer_gpu import BLOCKS, _setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 31, 32, 33, 127, 2049, 16384, 16385])
def test_gradient_at_tile_edges(rows):
    import torch
    net, p, X, y, Xd, yd = _setup(rows, 500 + rows)
    g, loss = net.grad(Xd, yd)
    losses = torch.zeros(1, device="cuda")
    net.train_epoch(Xd, yd, rows, 1e-3, seed=1, epoch=0, losses=losses)   # its sums are taken by the optimizer step
    g = g.cpu().numpy().astype(np.float64)
    gr, lr = M.grad(p.astype(np.float64), X.astype(np.float64), y.astype(np.float64), bf=True)
    assert float(loss.cpu()) == pytest.approx(lr, rel=1e-4) and float(losses.cpu()[0]) == pytest.approx(lr, rel=1e-4)
    moved = net.get_params().astype(np.float64) - p
    for name, sl in BLOCKS.items():
        assert np.linalg.norm(g[sl] - gr[sl]) <= 1e-3 * np.linalg.norm(gr[sl]) + 1e-12, name
        assert np.abs(g[sl] - gr[sl]).max() <= 2.0 ** -8 * np.abs(gr[sl]).max() + 1e-12, name
        # the first Adam step: lr against the gradient's sign wherever it is clear of the rounding
        clear = np.abs(gr[sl]) > np.maximum(2.0 ** -6 * np.abs(gr[sl]).max(), 1e-6)
        assert (np.abs(moved[sl][clear] + 1e-3 * np.sign(gr[sl][clear])) <= 2e-5).all(), name
