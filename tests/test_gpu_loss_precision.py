"""The standalone gradient is float64 up to its one rounding to float32: the
pairs' records carry no rounding of their own, which the cancellation in a
camera's sum would magnify.  Against the oracle in float64."""
import numpy as np
import pytest
import torch

from oracle import ea
from tests import helpers

pytestmark = pytest.mark.gpu


# cameras (and one in no pair, the last or the first), pairs to each side
@pytest.mark.parametrize("N,reach,first", [(2, 1, 0), (4, 3, 1), (40, 20, 0), (120, 70, 1), (700, 40, 0)])
def test_gradient_is_rounded_once(N, reach, first):
    from paper_2505_04612_amd import api
    ctx = api.default_context()
    rng = np.random.default_rng(N + reach)
    pairs = np.array([(i, i + k) for i in range(N) for k in range(1, reach + 1) if i + k < N], dtype=np.int32) + first
    P, per = len(pairs), 9
    uv = rng.normal(scale=0.5, size=(per * P, 4))
    s = api.Scene.from_numpy(ctx, N + 1, pairs, (np.arange(P + 1) * per).astype(np.int64), uv, torch.float64)
    W = api.build_pair_grams(s)[0]
    th = rng.normal(size=(N + 1, 9)).astype(np.float32)
    iz = 1.0 / (per * P)
    _, grad = api.epipolar_loss_grad(s, W, torch.from_numpy(th).to(ctx.device), inv_Z=iz)
    _, g = ea.loss_grad(th.astype(np.float64), pairs, helpers.expand36(W.cpu().numpy()), iz)
    got = grad.cpu().numpy().astype(np.float64)
    # half a float32 unit of the entry, and the float64 rounding of the terms
    # and of their sums (a few hundred operations deep)
    assert np.all(np.abs(got - g) <= 2.0 ** -24 * np.abs(g) + 1e-12 * np.abs(g).max())
    assert np.all(got[0 if first else N] == 0.0)
