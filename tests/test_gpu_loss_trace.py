"""The fused epipolar loops' loss trace against the standalone loss at the same
parameters, for iteration counts around the batches in which the loops sum
their per-iteration partials, on one and on many workgroups (flat and per-XCD
barrier), camera loop and pair loop."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _problem(N, reach, per=9):
    from paper_2505_04612_amd import api
    ctx = api.default_context()
    rng = np.random.default_rng(N)
    pairs = np.array([(i, i + k) for i in range(N) for k in range(1, reach + 1) if i + k < N], dtype=np.int32)
    P = len(pairs)
    uv = rng.normal(scale=0.5, size=(per * P, 4))
    s = api.Scene.from_numpy(ctx, N, pairs, (np.arange(P + 1) * per).astype(np.int64), uv, torch.float32)
    W, _ = api.build_pair_grams(s)
    a = rng.normal(size=(N, 9)).astype(np.float32)
    return api, s, W, torch.from_numpy(a).to(ctx.device), 1.0 / (per * P)


# cameras, pairs per camera, workgroups (0: the automatic camera loop)
@pytest.mark.parametrize("N,reach,blocks", [(5, 2, 0), (5, 2, 1), (70, 6, 0), (70, 6, 3), (600, 4, 0), (600, 4, 150)])
def test_trace_equals_the_loss_at_each_iteration(N, reach, blocks):
    api, s, W, theta, iz = _problem(N, reach)

    def solve(K):
        p = theta.clone()
        m, v = torch.zeros_like(p), torch.zeros_like(p)
        tr = torch.full((K,), float("nan"), dtype=torch.float64, device=p.device)
        api.epipolar_solve(s, W, p, m, v, K, 3e-3, 1e-2, 1e-2, 0, 64, inv_Z=iz, loss_trace=tr, blocks=blocks)
        return p, tr

    _, full = solve(50)
    # P float64 terms summed in two orders: a few P eps, P <= 2,390
    for K in (1, 2, 15, 16, 17, 31, 32, 33, 48, 49):
        p, tr = solve(K)
        assert torch.equal(tr, full[:K])
        loss, _ = api.epipolar_loss_grad(s, W, p, inv_Z=iz, want_grad=False)
        torch.testing.assert_close(full[K], loss[0], rtol=1e-11, atol=0)
    assert s.barrier_failures() == 0
