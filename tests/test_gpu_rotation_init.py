"""Rotation initialisation over workgroup counts (basis wholly in LDS, partly
and mostly in memory), step budgets (the variant that keeps everything in
memory from 1,025 steps on) and small graphs, against the oracle's dense
eigendecompositions."""
import numpy as np
import pytest
import torch

from oracle import rotation as ra
from paper_2505_04612_amd import synth

pytestmark = pytest.mark.gpu


def _graph(N, reach, seed):
    rng = np.random.default_rng(seed)
    q = rng.normal(size=(N, 4))
    q /= np.linalg.norm(q, axis=1, keepdims=True)
    w, x, y, z = q.T
    R = np.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                  2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                  2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], -1).reshape(N, 3, 3)
    pairs = np.array([(i, i + d) for i in range(N) for d in range(1, reach + 1) if i + d < N], np.int32)
    sc = synth.Scene("graph", seed, R, np.zeros((N, 3)), R, np.zeros((N, 3)), pairs, np.zeros(len(pairs) + 1, np.int64),
                     np.zeros((0, 4)), np.zeros(0, bool), "f32", 0.0, 0.0)
    return sc, synth.rotation_inputs(sc).R_rel.reshape(-1, 9).astype(np.float32)


# cameras, pairs per camera, steps, workgroups; 2: two cameras in one pair
@pytest.mark.parametrize("N,reach,steps,blocks", [
    (2, 1, 300, 0), (3, 2, 300, 0), (16, 5, 300, 0), (17, 5, 300, 0), (17, 5, 300, 17), (33, 8, 9, 0), (33, 8, 10, 0),
    (200, 26, 300, 0), (200, 26, 300, 1), (200, 26, 300, 2), (200, 26, 300, 50), (200, 70, 300, 0), (400, 30, 1100, 0),
    (400, 30, 1100, 3)])
def test_initialisation_over_grids(N, reach, steps, blocks):
    from paper_2505_04612_amd import api
    ctx = api.default_context()
    sc, Q = _graph(N, reach, 7 * N + reach)
    s = api.Scene.from_numpy(ctx, N, sc.pairs, sc.offsets, sc.uv, torch.float32)
    start = torch.from_numpy(np.random.default_rng(3).normal(size=(2, 3 * N))).to(ctx.device)
    q = torch.from_numpy(Q).to(ctx.device)
    p, info = api.rotation_init(s, q, start, steps, blocks)
    p2, info2 = api.rotation_init(s, q, start, steps, blocks)
    assert s.barrier_failures() == 0
    assert torch.equal(p, p2) and torch.equal(info, info2)
    info = info.cpu().numpy()
    assert 1 <= info[1] <= min(steps, 3 * N) and 1 <= info[3] <= min(steps, 3 * N)
    got = p.cpu().numpy().astype(np.float64)
    R = ra.rotations(got)
    assert np.abs(np.einsum("nba,nbc->nac", R, R) - np.eye(3)).max() < 1e-6
    R_or, oinfo = ra.initialise(sc.pairs, Q.astype(np.float64).reshape(-1, 3, 3), N)
    w1, w2 = np.linalg.eigvalsh(oinfo["A"]), np.linalg.eigvalsh(oinfo["B"])
    if steps < 60 and steps < 3 * N:
        # a step budget too small to converge: a Ritz value lies above
        assert info[0] >= w1[0] - 1e-9 and info[1] == steps
        return
    # float64 rounding of matrices of this norm
    assert abs(info[0] - w1[0]) <= 1e-10 * w1[0] + 1e-13 * w1[-1], (info, w1[0])
    if w1[1] - w1[0] > 1e-3:   # else the first column is any vector of that space
        assert abs(info[2] - w2[0]) <= 1e-8 * w2[0] + 1e-13 * w2[-1], (info, w2[0])
        if w2[1] - w2[0] > 1e-3 * w2[-1]:
            e = ra.relative_rotation_errors(R, R_or, sc.pairs)
            assert e.max() < 1e-3, e.max()


def test_initialisation_takes_the_memory_it_needs_in_any_order():
    from paper_2505_04612_amd import api
    ctx = api.default_context()
    sc, Q = _graph(120, 10, 5)
    q = torch.from_numpy(Q).to(ctx.device)
    start = torch.from_numpy(np.random.default_rng(4).normal(size=(2, 360))).to(ctx.device)
    s = api.Scene.from_numpy(ctx, 120, sc.pairs, sc.offsets, sc.uv, torch.float32)
    order = [(40, 0), (300, 1), (300, 0), (360, 2), (300, 1)]
    got = [api.rotation_init(s, q, start, m, b)[0].clone() for m, b in order]
    assert torch.equal(got[1], got[4]) and s.barrier_failures() == 0
    fresh = api.Scene.from_numpy(ctx, 120, sc.pairs, sc.offsets, sc.uv, torch.float32)
    assert torch.equal(api.rotation_init(fresh, q, start, 300, 0)[0], got[2])
