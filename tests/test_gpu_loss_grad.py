"""Standalone epipolar loss and gradient over graphs whose pairs fill one and
many workgroups and whose cameras have no pair, fewer and more than 64 of
them: against the oracle, and each output alone against both together."""
import numpy as np
import pytest
import torch

from oracle import ea
from tests import helpers

pytestmark = pytest.mark.gpu


# cameras, pairs per camera
@pytest.mark.parametrize("N,reach", [(2, 1), (5, 3), (30, 29), (90, 70), (700, 40)])
@pytest.mark.parametrize("wdt", [torch.float32, torch.float64])
def test_loss_and_gradient(N, reach, wdt):
    from paper_2505_04612_amd import api
    ctx = api.default_context()
    rng = np.random.default_rng(N + reach)
    pairs = np.array([(i, i + k) for i in range(N) for k in range(1, reach + 1) if i + k < N], dtype=np.int32)
    P, per = len(pairs), 9
    uv = rng.normal(scale=0.5, size=(per * P, 4))
    # one more camera, in no pair
    s = api.Scene.from_numpy(ctx, N + 1, pairs, (np.arange(P + 1) * per).astype(np.int64), uv, torch.float64)
    W = api.build_pair_grams(s)[0 if wdt == torch.float64 else 1]
    th = rng.normal(size=(N + 1, 9)).astype(np.float32)
    p = torch.from_numpy(th).to(ctx.device)
    iz = 1.0 / (per * P)
    loss, grad = api.epipolar_loss_grad(s, W, p, inv_Z=iz)
    L, g = ea.loss_grad(th.astype(np.float64), pairs, helpers.expand36(W.double().cpu().numpy()), iz)
    # float64 loss; gradient: float32 records (2^-24 of each) summed in float64,
    # rounded once; the largest entry bounds the records' size
    assert abs(float(loss) - L) <= 1e-12 * abs(L)
    got = grad.cpu().numpy()
    assert np.abs(got - g).max() <= 4 * 2.0 ** -24 * np.sqrt(2 * reach) * np.abs(g).max()
    assert np.all(got[N] == 0.0)
    only_loss, none = api.epipolar_loss_grad(s, W, p, inv_Z=iz, want_grad=False)
    nil, only_grad = api.epipolar_loss_grad(s, W, p, inv_Z=iz, want_loss=False)
    assert none is None and nil is None
    assert torch.equal(only_loss, loss) and torch.equal(only_grad, grad)
