"""Caps on the CG iterations: below 16 they bound plain CG (a solve that plain CG
finishes within the cap is not stopped, whatever the precision), from 16 on the
preconditioned iteration, in FP64 over all corrections of a system."""
import numpy as np
import pytest

import oracle
from gpu_common import THETA_TRUE, TAU, need_gpu, rel_l2

pytestmark = pytest.mark.gpu

ALL = [(32, 0), (64, 0), (128, 0), (256, 0), (64, 1), (128, 1), (256, 1)]


def _rough(n):
    rng = np.random.default_rng(9)
    return rng.uniform(0.5, 1.5, (n, n)), rng.uniform(0.5, 1.5, (n, n))


def _run(grids, dt, steps, rtol, thetas, grid_id=None, **kw):
    import torch
    from paper_1605_04718_amd.api import Problem
    p = Problem(grids, dt, steps, rtol, max_batch=16, **kw)
    gid = None if grid_id is None else torch.tensor(grid_id, dtype=torch.int32, device="cuda")
    out = [t.cpu().numpy() for t in p.forward_solve(torch.tensor(thetas, device="cuda"),
                                                    grid_id=gid)]
    p.close()
    return out


@pytest.mark.parametrize("n,fp64", ALL)
def test_a_small_cap_that_plain_cg_meets(n, fp64):
    """The oracle's own iteration count as the cap, where it is below 16."""
    from paper_1605_04718_amd.api import Grid
    need_gpu()
    dt, rtol = 5e-7 * (64 / n) ** 2, 1e-10 if fp64 else 1e-7
    u0, v0 = _rough(n)
    theta = (0.1, 0.9, 200.0, 3.0)
    uo, vo, it, so = oracle.forward_solve(theta, u0, v0, dt, 1, rtol=rtol)
    cap = int(np.max(it)) + 1  # (one more: a residual may end a hair above the tolerance)
    assert so == 0 and 3 <= cap < 16
    u, v, st, got = _run(Grid(n=n, u0=u0, v0=v0), dt, 1, rtol, np.array([theta]), precision=fp64,
                         cg_maxit=cap)
    assert st[0] == 0 and got.max() <= cap, (cap, got)
    tol = (2.0 ** -50 if fp64 else 2.0 ** -23) + 4 * 1.2 * rtol
    assert rel_l2(u[0], uo) <= tol and rel_l2(v[0], vo) <= tol


def test_a_small_cap_in_a_mixed_fp64_batch():
    from paper_1605_04718_amd.api import Grid
    need_gpu()
    sizes = [64, 256, 32, 128]
    fields = [_rough(n) for n in sizes]
    grids = [Grid(n=n, u0=f[0], v0=f[1]) for n, f in zip(sizes, fields)]
    gid = [0, 1, 2, 3, 3, 2, 1, 0, 7]
    thetas = np.array([(0.1, 0.9, 200.0, 3.0)] * len(gid))
    u, _, st, it = _run(grids, 3e-8, 1, 1e-9, thetas, gid, precision=1, cg_maxit=15)
    assert np.all(st[:8] == 0) and st[8] == 16
    for k in range(8):
        n = sizes[gid[k]]
        uo, _, _, so = oracle.forward_solve(thetas[k], *fields[gid[k]], 3e-8, 1, rtol=1e-13)
        assert so == 0
        assert rel_l2(u.reshape(9, -1)[k, :n * n], uo.ravel()) <= 2.0 ** -50 + 4 * 1.2e-9
    _, _, st, it = _run(grids, TAU, 1, 1e-9, thetas, gid, precision=1, cg_maxit=3)
    assert np.all(st[:8] == 1) and st[8] == 16 and it[:8].max() == 3


@pytest.mark.parametrize("n,fp64", ALL)
def test_the_preconditioned_iteration_stops_at_its_cap(n, fp64):
    """A stiff system and a tolerance that need more than 16 iterations: the cap
    is met in the first solve (FP32, stiffer) or within the corrections (FP64)."""
    from paper_1605_04718_amd.api import Grid
    need_gpu()
    u0, v0 = _rough(n)
    stiff = np.array([3e6 if fp64 else 1e7])
    thetas = np.array([(0.1, 0.9, 200.0, stiff[0] / (8 * n * n * TAU))])
    for cap in (16, 17):
        _, _, st, it = _run(Grid(n=n, u0=u0, v0=v0), TAU, 1, 1e-12 if fp64 else 1e-9, thetas,
                            precision=fp64, cg_maxit=cap)
        assert st[0] == 1 and it[0, 1] == cap, (st, it)
    _, _, st, it = _run(Grid(n=n, u0=u0, v0=v0), TAU, 1, 1e-12 if fp64 else 1e-9, thetas,
                        precision=fp64)
    assert st[0] == 0 and it[0, 1] > 17, (st, it)
