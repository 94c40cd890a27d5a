"""The grid search's two kernels against each other: a pair's result does not
depend on the graph around it, so the first pairs of a graph on which few
candidates run one lane per pair slice equal, to the bit, those of a graph small
enough for the batched kernel."""
import numpy as np
import pytest
import torch

from oracle import grid_search as gs

pytestmark = pytest.mark.gpu


# pairs of the large graph, candidates: one to sixteen lanes per pair, one and
# two LDS tiles, fewer candidates than lanes; the last two run the batched
# kernel on both
@pytest.mark.parametrize("P,C", [(140_000, 1), (140_000, 1025), (70_001, 63), (70_001, 700), (40_000, 1500),
                                 (20_000, 300), (15_000, 5), (15_000, 600), (15_000, 4000), (140_000, 3000)])
def test_few_candidates_on_a_large_graph(P, C):
    from paper_2505_04612_amd import api
    ctx = api.default_context()
    rng = np.random.default_rng(P + C)
    N, small = 600, 2003
    pairs = np.array([(i, j) for i in range(N) for j in range(i + 1, N)][:P], np.int32)
    counts = rng.integers(0, 3, size=P)
    uv = rng.uniform(-0.5, 0.5, size=(int(counts.sum()), 4))
    W36, prior = rng.normal(size=(P, 36)), rng.normal(size=(P, 3)).astype(np.float32)
    W36[1] = np.nan      # no candidate is the lowest
    W36[2] = 0.0         # every candidate is
    th = rng.normal(size=(N, 9)).astype(np.float32)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(ctx.device)  # noqa: E731
    out = []
    for n in (P, small):
        off = np.concatenate([[0], np.cumsum(counts[:n])]).astype(np.int64)
        s = api.Scene.from_numpy(ctx, N, pairs[:n], off, uv[:off[-1]], torch.float32)
        out.append(api.translation_search(s, dev(W36[:n]), dev(th), dev(gs.fibonacci_sphere(C)), dev(prior[:n])))
    for x, y in zip(*out):
        assert torch.equal(x[:small], y)
    assert int(out[0][1][1]) == -1 and int(out[0][1][2]) == (0 if counts[2] else -1)
