"""The one-dimensional solve at the edges of its lane layout: 16 lanes per
item with ceil(n / 16) rows each and four items per wavefront, so n around
multiples of 16, batches that do not fill the last wavefront, and items that
end early (non-positive growth) beside items that do not."""
import numpy as np
import pytest

from oracle import growth1d as og
from gpu_common import need_gpu, rel_l2
from paper_1605_04718_amd import inputs

pytestmark = pytest.mark.gpu

THETA1, TAU, RHO_T = (0.1, 0.9, 1000.0, 10.0), 1e-4, 1.8


@pytest.mark.parametrize("n,m", [(3, 1), (15, 5), (16, 4), (17, 3), (33, 6), (80, 7), (96, 2),
                                 (97, 9), (113, 1), (127, 5)])
def test_fields_at_the_edges_of_the_lane_layout(n, m):
    import torch
    from paper_1605_04718_amd.api import Growth1D
    need_gpu()
    steps = 120
    u0, v0 = inputs.initial_fields_1d(n)
    g = Growth1D(n, steps, TAU, THETA1, u0, v0, rho_T=RHO_T, max_batch=16)
    B = inputs.box_draws(m, (-0.5, -0.5, -0.5), (1.5, 1.0, 1.0), seed=n)
    dead = np.arange(m) % 3 == 1     # rho turns negative on the way
    B[dead] = (-30.0, 0.0, 0.0)
    u, v, st = g.forward(torch.tensor(B, device="cuda"))
    u, v, st = u.cpu().numpy(), v.cpu().numpy(), st.cpu().numpy()
    g.close()
    for k in range(m):
        assert og.growth_positive(B[k], RHO_T, TAU, steps) == (not dead[k])
        assert st[k] == (8 if dead[k] else 0)
        if not dead[k]:
            uo, vo = og.forward_beta(THETA1, B[k], RHO_T, u0, v0, TAU, steps)
            # as the other field tests: direct solves of systems with condition
            # numbers below 1e4 in FP64, 120 steps
            assert rel_l2(u[k], uo) < 1e-11 and rel_l2(v[k], vo) < 1e-11
