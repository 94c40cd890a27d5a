"""MLP backward at the edges of a 16-match tile and of a workgroup's four
tiles: what stands behind the last match (NaN here) must not reach the
gradients, so these equal, bit by bit, those with zeros behind it."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 16, 17, 63, 64, 65, 32_769])
def test_nothing_behind_the_last_match_is_used(M):
    from paper_2505_04612_amd import api
    ctx = api.default_context()
    rng = np.random.default_rng(M)
    w = api.MlpWeights(ctx.device, mean=torch.zeros(3, device=ctx.device), std=torch.ones(3, device=ctx.device))
    for k, shp in api.MLP_SHAPES.items():
        w.views[k].copy_(torch.from_numpy(rng.normal(0.0, 0.5, size=shp).astype(np.float32)))
    feats = torch.from_numpy(rng.normal(size=(M, 3)).astype(np.float32)).to(ctx.device)
    dout = torch.from_numpy(rng.normal(size=M).astype(np.float32)).to(ctx.device)
    _, act = api.mlp_forward(ctx, w, feats, keep_act=True)
    got = []
    for fill in (0.0, float("nan")):
        def behind(t):
            buf = torch.full((M + 64, *t.shape[1:]), fill, dtype=t.dtype, device=t.device)
            buf[:M] = t
            return buf[:M]
        got.append(api.mlp_backward(ctx, w, behind(feats), behind(act), behind(dout)).flat.clone())
    assert torch.isfinite(got[0]).all() and float(got[0].abs().max()) > 0
    assert torch.equal(got[0], got[1])
