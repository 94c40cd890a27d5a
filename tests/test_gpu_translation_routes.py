"""The translation loop's two camera-by-camera forms: a traced launch exchanges by
mailbox, an untraced one of many runs goes through the grid barrier. They add in
the same order, so they agree to the bit; and with the pair loop to the
rounding of its records (6e-8 over a cancellation of 1e3, times lr = 3e-2, over
9 steps: 2e-5)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


# cameras, pairs to each side, runs: groups of four past the line of graphs below
# 128 cameras with few and more pairs, of one, two and three passes, and two on it
@pytest.mark.parametrize("N,reach,runs", [(3, 2, 5), (40, 6, 4), (40, 6, 7), (60, 20, 9), (127, 126, 10), (200, 26, 21),
                                          (200, 45, 9), (300, 90, 5), (700, 4, 28), (1024, 50, 17)])
def test_traced_and_untraced_agree(N, reach, runs):
    from paper_2505_04612_amd import api
    ctx = api.default_context()
    rng = np.random.default_rng(N + runs)
    pairs = np.array([(i, i + k) for i in range(N) for k in range(1, reach + 1) if i + k < N], dtype=np.int32)
    P, K = len(pairs), 9
    s = api.Scene.from_numpy(ctx, N, pairs, np.zeros(P + 1, np.int64), np.zeros((0, 4)), torch.float32)
    d = rng.normal(size=(P, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    dirs = torch.from_numpy(d.astype(np.float32)).to(ctx.device)
    cen = rng.normal(size=(runs, N, 3)).astype(np.float32)
    out = []
    for traced, blocks in ((True, 0), (False, 0), (True, 8)):
        c = torch.from_numpy(cen).to(ctx.device)
        m, v = torch.zeros_like(c), torch.zeros_like(c)
        tr = torch.zeros((runs, K), dtype=torch.float64, device=ctx.device) if traced else None
        api.translation_solve(s, dirs, c, m, v, K, 3e-2, 1e-2, loss_trace=tr, blocks=blocks)
        out.append((c, m, v, tr))
    assert s.barrier_failures() == 0
    for x, y in zip(out[0][:3], out[1][:3]):
        assert torch.equal(x, y)
    torch.testing.assert_close(out[0][0], out[2][0], rtol=0, atol=2e-5)
    torch.testing.assert_close(out[0][3], out[2][3], rtol=1e-6, atol=0)
