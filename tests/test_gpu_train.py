"""The training kernels at the edges of their tiles (16 samples a tile, at
most 256 workgroups): loss and gradient against the FP64 oracle, and a
train_step against gradient + adam, bitwise."""
import numpy as np
import pytest

from oracle import sensor as S
from paper_1503_00707_amd import dvm as D
from paper_1503_00707_amd import inputs as I
from tests.test_gpu_sensor import _net_and_data

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 16, 17, 4095, 4096, 4097, 9000])
def test_gradient_and_train_step_at_tile_edges(n):
    import torch
    p, x, y = _net_and_data(seed=n, n=n)
    xt, yt = torch.as_tensor(x).cuda(), torch.as_tensor(y).cuda()
    a, b = D.MLP(p, max_batch=n), D.MLP(p, max_batch=n + 40)
    lo, go = S.loss_and_grad(p.astype(np.float64), x.astype(np.float64), y.astype(np.float64), 3.0)
    for _ in range(2):  # the second pass with weights moved by Adam
        a.gradient(xt, yt, pos_weight=3.0)
        g, loss = a.grads_and_loss()
        if lo is not None:  # FP32 layers of 64-term sums: 64 x 2^-24 of the terms, as for the other sizes tested
            assert loss == pytest.approx(lo, rel=1e-5)
            assert np.abs(g.double().cpu().numpy() - go).max() <= 1e-5 * np.abs(go).max()
            lo = None
        a.adam(1e-2)
        b.train_step(xt, yt, lr=1e-2, pos_weight=3.0)
        gb, lb = b.grads_and_loss()
        assert torch.equal(g, gb) and loss == lb
        assert torch.equal(a.params, b.params)
    assert not np.array_equal(a.params.cpu().numpy()[:I.MLP_WEIGHTS], p[:I.MLP_WEIGHTS])
