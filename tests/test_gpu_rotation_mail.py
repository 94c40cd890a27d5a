"""The rotation initialisation's two kinds of exchange between workgroups:
mailboxes up to 64 workgroups, grid barriers above, on one graph.  They sum the
same partials in the same order up to the grid's split, so the Ritz values
agree to the rounding of matrices of this norm (1e-13 of it, 1e-10 relative) and
the rotations to the residual bound the steps stop at (1e-11 of the norm over
the gap: below 1e-3 degrees, float32 output included)."""
import numpy as np
import pytest
import torch

from oracle import rotation as ra
from tests.test_gpu_rotation_init import _graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blocks", [63, 64, 65, 130])
def test_exchanges_agree(blocks):
    from paper_2505_04612_amd import api
    ctx = api.default_context()
    N = 200
    sc, Q = _graph(N, 26, 11)
    s = api.Scene.from_numpy(ctx, N, sc.pairs, sc.offsets, sc.uv, torch.float32)
    start = torch.from_numpy(np.random.default_rng(5).normal(size=(2, 3 * N))).to(ctx.device)
    q = torch.from_numpy(Q).to(ctx.device)
    p0, i0 = api.rotation_init(s, q, start, 300, 25)
    p, i = api.rotation_init(s, q, start, 300, blocks)
    again, _ = api.rotation_init(s, q, start, 300, blocks)
    assert s.barrier_failures() == 0 and torch.equal(p, again)
    R_or, oinfo = ra.initialise(sc.pairs, Q.astype(np.float64).reshape(-1, 3, 3), N)
    norms = [np.linalg.eigvalsh(oinfo[k])[-1] for k in ("A", "B")]
    for k, norm in enumerate(norms):
        a, b = float(i0[2 * k]), float(i[2 * k])
        assert abs(a - b) <= 1e-10 * abs(a) + 1e-13 * norm, (a, b)
    R0, R = (ra.rotations(x.cpu().numpy().astype(np.float64)) for x in (p0, p))
    assert ra.relative_rotation_errors(R, R0, sc.pairs).max() < 1e-3
