"""Graphs with one camera that is paired with very many: the gradient by rows of
16 lanes and by whole wavefronts, and the loops that the automatic grids take."""
import numpy as np
import pytest
import torch

from oracle import ea
from tests import helpers

pytestmark = pytest.mark.gpu


def _hub(N, deg, hub):
    """A ring of N cameras, and camera `hub` paired with `deg` of them in all."""
    pr = {tuple(sorted((i, (i + 1) % N))) for i in range(N)}
    for i in range(N):
        if sum(hub in p for p in pr) == deg:
            break
        if i != hub:
            pr.add(tuple(sorted((hub, i))))
    return np.array(sorted(pr), np.int32)


# on both sides of 1,024 pairs of a camera, the hub first, last and between
@pytest.mark.parametrize("N,deg,hub", [(1030, 1024, 0), (1030, 1025, 0), (1300, 1299, 1299), (1500, 1200, 700)])
def test_gradient(N, deg, hub):
    from paper_2505_04612_amd import api
    ctx = api.default_context()
    rng = np.random.default_rng(N + deg)
    pairs = _hub(N, deg, hub)
    P, per = len(pairs), 9
    assert np.bincount(pairs.reshape(-1)).max() == deg
    s = api.Scene.from_numpy(ctx, N, pairs, (np.arange(P + 1) * per).astype(np.int64),
                             rng.normal(scale=0.5, size=(per * P, 4)), torch.float64)
    W = api.build_pair_grams(s)[0]
    th = rng.normal(size=(N, 9)).astype(np.float32)
    iz = 1.0 / (per * P)
    loss, grad = api.epipolar_loss_grad(s, W, torch.from_numpy(th).to(ctx.device), inv_Z=iz)
    L, g = ea.loss_grad(th.astype(np.float64), pairs, helpers.expand36(W.cpu().numpy()), iz)
    got = grad.cpu().numpy().astype(np.float64)
    assert abs(float(loss) - L) <= 1e-12 * abs(L)
    # one rounding to float32, and the float64 rounding of up to 1,300 terms
    assert np.all(np.abs(got - g) <= 2.0 ** -24 * np.abs(g) + 1e-12 * np.abs(g).max())


# cameras, pairs of the hub, whether the automatic grid goes camera by camera; the
# last one's neighbours wait some 200 us for it, long enough to look at the clock
# that bounds their waits
@pytest.mark.parametrize("N,deg,cam", [(600, 250, True), (1000, 600, False), (1300, 1299, False),
                                       (5000, 4999, False)])
def test_loops(N, deg, cam):
    from paper_2505_04612_amd import api
    ctx = api.default_context()
    rng = np.random.default_rng(N)
    pairs = _hub(N, deg, 3)
    P, K = len(pairs), 5
    s = api.Scene.from_numpy(ctx, N, pairs, np.arange(P + 1, dtype=np.int64), rng.normal(scale=0.5, size=(P, 4)),
                             torch.float64)
    W = torch.randn((P, 36), device=ctx.device, generator=torch.Generator(ctx.device).manual_seed(1))
    th = torch.from_numpy(rng.normal(size=(N, 9)).astype(np.float32)).to(ctx.device)
    out = {}
    for blocks in (0, -1, 128):
        p = th.clone()
        m, v = torch.zeros_like(p), torch.zeros_like(p)
        tr = torch.zeros(K, dtype=torch.float64, device=ctx.device)
        api.epipolar_solve(s, W, p, m, v, K, 3e-3, 1e-2, 1e-2, 0, 20, inv_Z=1.0 / P, blocks=blocks, loss_trace=tr)
        out[blocks] = (p, m, v, tr)
    # (float64 traces: the same for every launch of the camera loop, and in their
    # last bits not the pair loop's)
    assert torch.equal(out[0][3], out[-1][3]) == cam
    assert all(torch.equal(x, y) for x, y in zip(out[0][:3], out[-1 if cam else 128][:3]))
    torch.testing.assert_close(out[0][3], out[-1][3], rtol=1e-9, atol=0)
    # the translation loop by mailbox (traced) and as the automatic grid takes it
    d = rng.normal(size=(P, 3))
    dirs = torch.from_numpy((d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)).to(ctx.device)
    for runs in (1, 3, 4):
        cen = torch.from_numpy(rng.normal(size=(runs, N, 3)).astype(np.float32)).to(ctx.device)
        res = []
        for trace in (None, torch.zeros((runs, K), dtype=torch.float64, device=ctx.device)):
            c = cen.clone()
            m, v = torch.zeros_like(c), torch.zeros_like(c)
            api.translation_solve(s, dirs, c, m, v, K, 3e-2, 1e-2, loss_trace=trace)
            res.append((c, m, v))
        assert all(torch.equal(x, y) for x, y in zip(*res))
    assert s.barrier_failures() == 0
