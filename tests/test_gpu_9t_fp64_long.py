"""FP64 solves over hundreds of steps, where an error of a step has time to grow:
the refined solves against the oracle (64 x 64, 128 x 128) and against the streamed
plain CG of the same size (256 x 256)."""
import numpy as np
import pytest

import oracle
from gpu_common import THETA_TRUE, TAU, need_gpu, rel_l2
from paper_1605_04718_amd import inputs

pytestmark = pytest.mark.gpu

THETAS = np.array([THETA_TRUE, (0.3, 0.6, 55.0, 5.0), (0.15, 0.8, 240.0, 50.0)])
RTOL = 1e-11


# fastest growth of a perturbation of the rest state, over gamma: the largest real
# part of an eigenvalue of J - q diag(1, d) over q >= 0 (J the reaction's Jacobian)
RATES = (0.058, 0.0, 0.361)


def _tol(k, steps):
    # 1.2 rtol |x| enters at each step (as the other field tests) and grows
    return 1.2 * steps * RTOL * np.exp(RATES[k] * THETAS[k, 2] * steps * TAU)


def _fields(n, cpt, steps):
    import torch
    from paper_1605_04718_amd.api import FP64, Grid, Problem
    u0, v0 = inputs.initial_fields(n, THETA_TRUE[0], THETA_TRUE[1])
    p = Problem(Grid(n=n, u0=u0, v0=v0), TAU, steps, RTOL, precision=FP64, max_batch=4)
    p.set_tile(0, cpt)
    print(f"FP64 {n}^2 tile {cpt}: {steps} steps", flush=True)
    u, v, st, _ = p.forward_solve(torch.tensor(THETAS, device="cuda"))
    assert not st.any() and p.check_solves() == 0
    out = u.cpu().numpy(), v.cpu().numpy()
    p.close()
    return u0, v0, out


@pytest.mark.parametrize("n,cpt,steps", [(64, 16, 300), (128, 32, 200)])
def test_against_the_oracle(n, cpt, steps):
    need_gpu()
    u0, v0, (u, v) = _fields(n, cpt, steps)
    for k, th in enumerate(THETAS):
        uo, vo, _, so = oracle.forward_solve(th, u0, v0, TAU, steps, rtol=1e-13)
        assert so == 0
        assert rel_l2(u[k], uo) <= _tol(k, steps) and rel_l2(v[k], vo) <= _tol(k, steps)


def test_groups_against_the_streamed_tile():
    need_gpu()
    steps = 200
    _, _, (u, v) = _fields(256, 32, steps)
    _, _, (us, vs) = _fields(256, 128, steps)
    for k in range(len(THETAS)):
        assert rel_l2(u[k], us[k]) <= 2 * _tol(k, steps) and rel_l2(v[k], vs[k]) <= 2 * _tol(k, steps)
