"""MLP forward around its 64-match steps and 16-match tiles, the precision of
its first layer (float32 MFMA: the kept activations against float64, also where
the products cancel), non-finite features, and weights at any float alignment."""
import numpy as np
import pytest
import torch

from oracle import mlp

pytestmark = pytest.mark.gpu


def _net(seed, scale=1.0):
    p = mlp.init_params(seed)
    rng = np.random.default_rng(seed + 9)
    return {k: ((v + rng.normal(0.0, 0.05, v.shape)) * scale).astype(np.float32) for k, v in p.items()}


def _weights(api, ctx, p, mean, std, shift=0):
    n = sum(v.size for v in p.values())
    base = torch.zeros(n + shift, dtype=torch.float32, device=ctx.device)
    w = api.MlpWeights(ctx.device, flat=base[shift:])
    w.load_numpy(p, mean, std)
    return w


@pytest.mark.parametrize("M", [1, 16, 31, 63, 64, 65, 127, 129, 255, 257, 131_072 + 17])
def test_forward_over_steps(M):
    from paper_2505_04612_amd import api
    ctx = api.default_context()
    rng = np.random.default_rng(M)
    f = (rng.normal(size=(M, 3)) * [2.0, 1.0, 0.1] + [-6.0, 5.0, 0.2]).astype(np.float32)
    mean, std = np.float32([-6.0, 5.0, 0.2]), np.float32([2.0, 1.0, 0.1])
    p = _net(M % 5)
    x = torch.from_numpy(f).to(ctx.device)
    got, act = api.mlp_forward(ctx, _weights(api, ctx, p, mean, std), x, out_scale=2.0, keep_act=True)
    plain, _ = api.mlp_forward(ctx, _weights(api, ctx, p, mean, std, shift=1), x, out_scale=2.0)
    assert torch.equal(got, plain)
    ref, _ = mlp.forward({k: v.astype(np.float64) for k, v in p.items()}, f.astype(np.float64), mean, std)
    assert np.abs(got.cpu().numpy() - 2.0 * ref).max() <= 4e-3   # float16 hidden layer
    assert act.shape == (M, 128) and bool(torch.isfinite(act).all())


@pytest.mark.parametrize("offset,scale", [(0.0, 1.0), (300.0, 1.0), (0.0, 1e-3), (40.0, 20.0)])
def test_first_layer_keeps_float32_precision(offset, scale):
    from paper_2505_04612_amd import api
    ctx = api.default_context()
    M = 5000
    rng = np.random.default_rng(17)
    x = (rng.normal(size=(M, 3)) * 0.3 + offset).astype(np.float32)
    p = _net(3, scale)
    # rows whose weights sum to 0: the offset cancels
    p["W1"][::2, 2] = -(p["W1"][::2, 0] + p["W1"][::2, 1])
    w = _weights(api, ctx, p, np.zeros(3, np.float32), np.ones(3, np.float32))
    _, act = api.mlp_forward(ctx, w, torch.from_numpy(x).to(ctx.device), keep_act=True)
    h1 = act[:, :64].cpu().numpy().astype(np.float64)
    W1, b1 = p["W1"].astype(np.float64), p["b1"].astype(np.float64)
    z = np.maximum(x.astype(np.float64) @ W1.T + b1, 0.0)
    size = np.abs(x).astype(np.float64) @ np.abs(W1).T + np.abs(b1)
    # float32 accumulation (a few units of 2^-24 of the terms' size), then the
    # float16 rounding (half a unit, or half the smallest subnormal)
    tol = 4 * 2.0 ** -24 * size + 2.0 ** -11 * z + 2.0 ** -25
    assert np.all(np.abs(h1 - z) <= tol), np.max(np.abs(h1 - z) / tol)


def test_non_finite_features():
    from paper_2505_04612_amd import api
    ctx = api.default_context()
    x = np.zeros((70, 3), np.float32)
    x[3, 0], x[20, 1], x[66, 2] = np.inf, -np.inf, np.nan
    p = {k: np.abs(v) + np.float32(0.01) for k, v in _net(2).items()}
    w = _weights(api, ctx, p, np.zeros(3, np.float32), np.ones(3, np.float32))
    run = lambda v: [t.cpu().numpy() for t in api.mlp_forward(ctx, w, torch.from_numpy(v).to(ctx.device),  # noqa: E731
                                                                keep_act=True)]
    out, act = run(x)
    bad = [3, 20, 66]
    # the infinity reaches every unit of its match (float16 infinity), -inf and
    # NaN leave ReLU at 0
    assert np.all(np.isposinf(act[3, :64])) and np.all(act[20, :64] == 0.0) and np.all(act[66, :64] == 0.0)
    # and no other match sees them
    clean = x.copy()
    clean[bad] = 0.0
    out0, act0 = run(clean)
    keep = np.setdiff1d(np.arange(70), bad)
    assert np.array_equal(out[keep], out0[keep]) and np.array_equal(act[keep], act0[keep])
    assert np.all(np.isfinite(out0)) and np.all(np.isfinite(out[[20, 66]]))
