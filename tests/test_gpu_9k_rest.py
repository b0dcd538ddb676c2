"""Fields that come to rest and move again in the spectrally preconditioned
FP32 solve: a system whose first residual meets the tolerance takes no
increment, its field is not rewritten, and its increment buffers hold zeros.
Items that rest are mixed with items that do not, over more items than
workgroups, so that a slot's earlier contents would show."""
import numpy as np
import pytest

import oracle
from gpu_common import TAU, need_gpu

pytestmark = pytest.mark.gpu

# the first is at rest in the homogeneous fields u = a + b, v = b / u^2; the
# others are moved by their reaction, at different rates
THETAS = np.array([(0.1, 0.9, 200.0, 10.0), (0.1005, 0.9, 60.0, 10.0), (0.3, 0.6, 240.0, 50.0),
                   (0.1, 0.9001, 55.0, 5.0)])


@pytest.mark.parametrize("n,m", [(32, 4300), (64, 1700), (128, 600), (256, 140)])
@pytest.mark.parametrize("rtol,rate", [(1e-3, 0.0), (1e-5, 0.0), (1e-4, 0.05)])
def test_resting_and_moving_items_do_not_depend_on_their_neighbours(n, m, rtol, rate):
    import torch
    from paper_1605_04718_amd.api import Grid, Problem
    need_gpu()
    steps = 25
    x = (np.arange(n) + 0.5) / n
    wave = np.cos(2 * np.pi * x)[:, None] * np.cos(np.pi * x)[None, :]
    u0, v0 = np.full((n, n), 1.0), 0.9 + 1e-4 * wave
    g = Grid(n=n, u0=u0, v0=v0, growth=int(rate != 0.0), growth_rate=rate)
    p = Problem(g, TAU, steps, rtol, max_batch=m)
    pick = np.random.default_rng(n).integers(0, 4, m)
    pick[:4] = range(4)
    u, v, st, it = p.forward_solve(torch.tensor(THETAS[pick], device="cuda"))
    assert p.check_solves() == 0
    first = torch.tensor(pick.copy(), device="cuda", dtype=torch.long)  # items 0 .. 3
    for t in (u, v, it):
        assert torch.equal(t, t[first])
    u, v = u[:4].double().cpu().numpy(), v[:4].double().cpu().numpy()
    p.close()
    for k, th in enumerate(THETAS):
        uo, vo, _, so = oracle.forward_solve(th, u0, v0, TAU, steps, rtol=1e-12,
                                             growth=int(rate != 0.0), rate=rate)
        assert so == 0
        # as the other field tests: at most 1.2 rtol |x| a step, 4 for its growth
        tol = 2.0 ** -24 + 4 * 1.2 * steps * rtol
        for got, want in ((u[k], uo), (v[k], vo)):
            assert np.linalg.norm(got - want) <= tol * np.linalg.norm(want)
