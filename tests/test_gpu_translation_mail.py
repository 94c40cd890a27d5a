"""The translation loop's exchange between wavefronts: groups of four, two and
one run, one to three passes of 64 pairs per camera, the largest graph with a
wavefront per camera, a camera in no pair; against the pair loop, and launches
in a row, which find the tags of the one before, against each other.

Both loops sum the same float32 records in float64 in different orders: a
record's last bit (6e-8) over the cancellation in a camera's sum (1e3 at the
most here), times lr = 3e-2, over 17 steps: 3e-5."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


# cameras (without the one in no pair), pairs to each side, runs, iterations
@pytest.mark.parametrize("N,reach,runs,K", [(2, 1, 1, 1), (40, 39, 2, 2), (70, 69, 7, 17), (140, 90, 4, 3),
                                            (511, 3, 3, 4), (512, 3, 5, 4), (1023, 2, 6, 17)])
@pytest.mark.parametrize("traced", [False, True])
def test_mailbox_loop_against_pair_loop(N, reach, runs, K, traced):
    from paper_2505_04612_amd import api
    ctx = api.default_context()
    rng = np.random.default_rng(N + runs)
    pairs = np.array([(i, i + k) for i in range(N) for k in range(1, reach + 1) if i + k < N], dtype=np.int32)
    P = len(pairs)
    s = api.Scene.from_numpy(ctx, N + 1, pairs, np.zeros(P + 1, np.int64), np.zeros((0, 4)), torch.float32)
    d = rng.normal(size=(P, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    dirs = torch.from_numpy(d.astype(np.float32)).to(ctx.device)
    cen = rng.normal(size=(runs, N + 1, 3)).astype(np.float32)
    out = []
    for blocks in (0, 0, 0, 8):
        c = torch.from_numpy(cen).to(ctx.device)
        m, v = torch.zeros_like(c), torch.zeros_like(c)
        tr = torch.zeros((runs, K), dtype=torch.float64, device=ctx.device) if traced else None
        api.translation_solve(s, dirs, c, m, v, K, 3e-2, 1e-2, loss_trace=tr, blocks=blocks)
        out.append([c, m, v] + ([tr] if traced else []))
    assert s.barrier_failures() == 0
    for r in out[1:3]:
        for x, y in zip(out[0], r):
            assert torch.equal(x, y)
    torch.testing.assert_close(out[0][0], out[3][0], rtol=0, atol=3e-5)
    if traced:
        torch.testing.assert_close(out[0][3], out[3][3], rtol=1e-6, atol=0)
    # the camera in no pair stays where it was
    assert torch.equal(out[0][0][:, N].cpu(), torch.from_numpy(cen[:, N]))
