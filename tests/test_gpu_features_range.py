"""The match features' angle past the range of its float64 estimates (float64
coordinates of 1e60 to 1e100, whose cross products' squares overflow), against
what atan2 of the square root gives in NumPy: infinities included."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


# magnitudes of the first and second point; the cross product's square is
# finite in float64, near its largest value, and infinite
@pytest.mark.parametrize("m1,m2", [(1e60, 1e60), (1.0, 1e74), (1e75, 1e75), (3e75, 3e76), (1e80, 1e80), (1e100, 1e100),
                                   (1e5, 1e152), (1.2e154, 1.2e154)])
def test_angle_of_huge_coordinates(m1, m2):
    from paper_2505_04612_amd import api
    ctx = api.default_context()
    rng = np.random.default_rng(5)
    M = 130
    d = rng.uniform(0.2, 0.9, size=(M, 4)) * np.where(rng.random((M, 4)) < 0.5, -1.0, 1.0)
    uv = d * np.array([m1, m1, m2, m2])
    if m1 > 1e150:
        # a dot product of +inf and of -inf beside a finite cross product
        uv[:] = [m1, m1, m2, 0.9 * m2]
        uv[::2, 2:] *= -1.0
    # two cameras with the identity rotation, one unit apart along x
    th = np.zeros((2, 9), np.float32)
    th[:, 0] = th[:, 4] = 1.0
    th[1, 6] = 1.0
    s = api.Scene.from_numpy(ctx, 2, np.array([[0, 1]], np.int32), np.array([0, M], np.int64), uv, torch.float64)
    got = api.match_features(s, torch.from_numpy(th).to(ctx.device), 1e-4).cpu().numpy().astype(np.float64)
    one = np.ones((M, 1))
    a, b = np.concatenate([uv[:, :2], one], 1), np.concatenate([uv[:, 2:], one], 1)
    with np.errstate(over="ignore"):
        c = np.cross(a, b)
        y2, x = np.sum(c * c, axis=1), np.sum(a * b, axis=1)
        angle = np.arctan2(np.sqrt(y2), x)
        r = np.abs(c[:, 0])   # t_hat = (1, 0, 0)
    assert np.all(np.isfinite(angle))
    # half a float32 unit, plus the float64 rounding of the cross product
    tol = 6.1e-8 * angle + 4e-15
    assert np.all(np.abs(got[:, 2] - angle) <= tol), (got[:3, 2], angle[:3])
    f0 = np.log(np.maximum(r, np.float64(np.float32(1e-4))))
    scale = 3e-14 * np.abs(a).max(axis=1) * np.abs(b).max(axis=1)
    assert np.all(np.abs(got[:, 0] - f0) <= 6.1e-8 * np.abs(f0) + 1e-11 + scale / r)


def test_a_nan_coordinate_stays_nan():
    from paper_2505_04612_amd import api
    ctx = api.default_context()
    uv = np.full((70, 4), 0.25)
    uv[3, 0] = uv[66, 3] = np.nan
    th = np.zeros((2, 9), np.float32)
    th[:, 0] = th[:, 4] = 1.0
    th[1, 6] = 1.0
    s = api.Scene.from_numpy(ctx, 2, np.array([[0, 1]], np.int32), np.array([0, 70], np.int64), uv, torch.float64)
    got = api.match_features(s, torch.from_numpy(th).to(ctx.device), 1e-4).cpu().numpy()
    assert np.array_equal(np.flatnonzero(np.isnan(got[:, 2])), [3, 66])
    assert np.all(np.abs(got[:, 0] - np.log(np.float64(np.float32(1e-4)))) <= 1e-6)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32, torch.bfloat16])
def test_infinite_coordinates(dtype):
    """No angle, and the residual of the form x2~^T (E x1~): infinite, or where
    its terms' infinities cancel the floor."""
    from paper_2505_04612_amd import api
    from oracle import ea
    ctx = api.default_context()
    rng = np.random.default_rng(8)
    M = 700
    uv = rng.normal(size=(M, 4))
    hit = rng.random((M, 4)) < 0.3
    uv[hit] = np.where(rng.random(hit.sum()) < 0.5, -np.inf, np.inf)
    th = rng.normal(size=(2, 9)).astype(np.float32)
    s = api.Scene.from_numpy(ctx, 2, np.array([[0, 1]], np.int32), np.array([0, M], np.int64), uv, dtype)
    got = api.match_features(s, torch.from_numpy(th).to(ctx.device), 1e-4).cpu().numpy().astype(np.float64)
    x = s.uv.to(torch.float64).cpu().numpy()
    R, t = ea.poses_from_params(th.astype(np.float64))
    Rij = R[1] @ R[0].T
    d = t[1] - Rij @ t[0]
    d /= np.linalg.norm(d)
    E = np.array([[0.0, -d[2], d[1]], [d[2], 0.0, -d[0]], [-d[1], d[0], 0.0]]) @ Rij
    with np.errstate(invalid="ignore"):
        e = [E[k, 0] * x[:, 0] + E[k, 1] * x[:, 1] + E[k, 2] for k in range(3)]
        r = np.abs(x[:, 2] * e[0] + x[:, 3] * e[1] + e[2])
    any_hit = hit.any(axis=1)
    f0 = np.log(np.where(r > np.float32(1e-4), r, np.float64(np.float32(1e-4))))
    assert np.array_equal(np.isnan(got[:, 2]), any_hit)
    assert np.array_equal(np.isinf(got[:, 0]), np.isinf(f0)) and np.isinf(f0).sum() > 100
    fin = any_hit & np.isfinite(f0)
    assert np.all(np.abs(got[fin, 0] - f0[fin]) <= 1e-6)
