"""Match features over pair sizes around the 1,024-match work items and over
the ranges of their logarithm and angle (every octant of atan2, the floor
delta, residuals above 1), against NumPy in float64 on the stored values."""
import numpy as np
import pytest
import torch

from oracle import ea

pytestmark = pytest.mark.gpu

SIZES = [1, 63, 64, 65, 0, 1023, 1024, 1025, 2500, 4096]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32, torch.bfloat16])
@pytest.mark.parametrize("spread", [1e-6, 0.3, 30.0])
def test_features_over_sizes_and_angles(dtype, spread):
    from paper_2505_04612_amd import api
    ctx = api.default_context()
    rng = np.random.default_rng(int(spread * 1e6) % 1000 + 1)
    N, P = 6, len(SIZES)
    pairs = np.array([(i, j) for i in range(N) for j in range(i + 1, N)][:P], np.int32)
    off = np.concatenate([[0], np.cumsum(SIZES)]).astype(np.int64)
    M = int(off[-1])
    base = rng.normal(scale=0.3, size=(M, 2))
    uv = np.concatenate([base, base + rng.normal(scale=spread, size=(M, 2))], 1)
    # cameras near one another (angles near 0), and one turned by 170 degrees
    th = np.zeros((N, 9), np.float32)
    th[:, 0], th[:, 4] = 1.0, 1.0
    th[:, 0:6] += rng.normal(scale=1e-3, size=(N, 6)).astype(np.float32)
    c, s_ = np.cos(np.radians(170.0)), np.sin(np.radians(170.0))
    th[2, 0:3] = [c, 0.0, -s_]
    th[:, 6:9] = rng.normal(size=(N, 3)).astype(np.float32)
    s = api.Scene.from_numpy(ctx, N, pairs, off, uv, dtype)
    delta = 1e-4
    got = api.match_features(s, torch.from_numpy(th).to(ctx.device), delta).cpu().numpy().astype(np.float64)

    x = s.uv.to(torch.float64).cpu().numpy()
    R, t = ea.poses_from_params(th.astype(np.float64))
    n = np.repeat(np.arange(P), SIZES)
    i, j = pairs[n, 0], pairs[n, 1]
    one = np.ones((M, 1))
    x1, x2 = np.concatenate([x[:, :2], one], 1), np.concatenate([x[:, 2:], one], 1)
    a = np.einsum("mba,mb->ma", R[i], x1)
    b = np.einsum("mba,mb->ma", R[j], x2)
    Rij = np.einsum("mab,mcb->mac", R[j], R[i])
    tt = t[j] - np.einsum("mab,mb->ma", Rij, t[i])
    tt /= np.linalg.norm(tt, axis=1, keepdims=True)
    r = np.abs(np.sum(x2 * np.cross(tt, np.einsum("mab,mb->ma", Rij, x1)), axis=1))
    f0 = np.log(np.maximum(r, np.float64(np.float32(delta))))
    f2 = np.arctan2(np.linalg.norm(np.cross(a, b), axis=1), np.sum(a * b, axis=1))
    scale = np.linalg.norm(x1, axis=1) * np.linalg.norm(x2, axis=1)
    # half a float32 unit, plus the float64 rounding of the residual (a few eps
    # of the rays' lengths) and of the angle
    tol0 = 6.1e-8 * np.abs(f0) + 1e-11 + 4e-15 * scale / np.maximum(r, delta)
    assert np.all(np.abs(got[:, 0] - f0) <= tol0), np.max(np.abs(got[:, 0] - f0) / tol0)
    assert np.allclose(got[:, 1], np.log(np.asarray(SIZES, np.float64)[n]), rtol=2e-7, atol=1e-7)
    tol2 = 6.1e-8 * f2 + 4e-15
    assert np.all(np.abs(got[:, 2] - f2) <= tol2), np.max(np.abs(got[:, 2] - f2) / tol2)
