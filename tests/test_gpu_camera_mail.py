"""The epipolar camera loop's exchange between wavefronts: graphs of one to
three passes of 64 pairs per camera and of one to three cameras per wavefront,
with a camera in no pair, against the pair loop; and launches in a row, which
find the tags of the one before, against each other.

Both loops sum the same float32 records in float64 in different orders.  A
record's last bit (6e-8) moves a step by at most lr = 1e-2 times that over the
cancellation in a camera's sum (1e3 at the most here): 6e-7 a step, 1e-5 over
the 17 steps."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


# cameras (without the one in no pair), pairs to each side, iterations
@pytest.mark.parametrize("N,reach,K", [(2, 1, 1), (40, 39, 2), (70, 69, 17), (140, 139, 3), (511, 3, 4), (512, 3, 4),
                                       (1030, 2, 17), (2100, 1, 16)])
@pytest.mark.parametrize("wdt", [torch.float32, torch.float64])
def test_camera_loop_against_pair_loop(N, reach, K, wdt):
    from paper_2505_04612_amd import api
    ctx = api.default_context()
    rng = np.random.default_rng(N + K)
    pairs = np.array([(i, i + k) for i in range(N) for k in range(1, reach + 1) if i + k < N], dtype=np.int32)
    P, per = len(pairs), 9
    uv = rng.normal(scale=0.5, size=(per * P, 4))
    s = api.Scene.from_numpy(ctx, N + 1, pairs, (np.arange(P + 1) * per).astype(np.int64), uv, torch.float64)
    W = api.build_pair_grams(s)[0 if wdt == torch.float64 else 1]
    th = rng.normal(size=(N + 1, 9)).astype(np.float32)
    out = []
    for blocks in (-1, -1, -1, 8):
        p = torch.from_numpy(th).to(ctx.device)
        m, v = torch.zeros_like(p), torch.zeros_like(p)
        tr = torch.zeros(K, dtype=torch.float64, device=ctx.device)
        api.epipolar_solve(s, W, p, m, v, K, 3e-3, 1e-2, 1e-2, 0, 20, inv_Z=1.0 / (per * P), blocks=blocks,
                           loss_trace=tr)
        out.append((p, m, v, tr))
    assert s.barrier_failures() == 0
    for r in out[1:3]:
        for x, y in zip(out[0], r):
            assert torch.equal(x, y)
    torch.testing.assert_close(out[0][3], out[3][3], rtol=1e-7, atol=0)
    torch.testing.assert_close(out[0][0], out[3][0], rtol=0, atol=1e-5)
    # the camera in no pair stays where it was
    assert torch.equal(out[0][0][N].cpu(), torch.from_numpy(th[N]))
