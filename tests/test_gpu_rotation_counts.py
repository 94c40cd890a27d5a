"""A given workgroup count of the rotation initialisation is raised to one per
256 cameras: smaller counts are the same launch."""
import numpy as np
import pytest
import torch

from paper_2505_04612_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,least", [(256, 1), (257, 2), (600, 3)])
def test_small_counts_are_raised(N, least):
    from paper_2505_04612_amd import api
    ctx = api.default_context()
    rng = np.random.default_rng(N)
    pairs = np.array([(i, i + d) for i in range(N) for d in (1, 2, 3) if i + d < N], np.int32)
    q, _ = np.linalg.qr(rng.normal(size=(len(pairs), 3, 3)))
    q *= np.sign(np.linalg.det(q))[:, None, None]
    s = api.Scene.from_numpy(ctx, N, pairs, np.zeros(len(pairs) + 1, np.int64), np.zeros((0, 4)), torch.float32)
    Q = torch.from_numpy(q.reshape(-1, 9).astype(np.float32)).to(ctx.device)
    start = torch.from_numpy(rng.normal(size=(2, 3 * N))).to(ctx.device)
    want, info = api.rotation_init(s, Q, start, 40, least)
    for blocks in range(1, least):
        p, i = api.rotation_init(s, Q, start, 40, blocks)
        assert torch.equal(p, want) and torch.equal(i, info)
    assert s.barrier_failures() == 0 and torch.isfinite(want).all()


@pytest.mark.parametrize("steps", [1, 10, 40])
def test_a_nan_rotation_gives_nan_parameters(steps):
    from paper_2505_04612_amd import api
    ctx = api.default_context()
    rng = np.random.default_rng(1)
    for N, blocks in ((5, 0), (70, 0), (70, 70)):
        pairs = np.array([(i, i + 1) for i in range(N - 1)], np.int32)
        q, _ = np.linalg.qr(rng.normal(size=(N - 1, 3, 3)))
        q = (q * np.sign(np.linalg.det(q))[:, None, None]).reshape(-1, 9).astype(np.float32)
        q[N // 2, 4] = np.nan
        s = api.Scene.from_numpy(ctx, N, pairs, np.zeros(N, np.int64), np.zeros((0, 4)), torch.float32)
        start = torch.from_numpy(rng.normal(size=(2, 3 * N))).to(ctx.device)
        p, info = api.rotation_init(s, torch.from_numpy(q).to(ctx.device), start, steps, blocks)
        assert torch.isnan(p).all() and torch.isnan(info[0::2]).all() and s.barrier_failures() == 0
