"""The FP64 solve of 32x32 items (four wavefronts, arrays in registers) against
the FP64 oracle: rough fields, so that every neighbour and mirror ghost counts,
the first steps (start vectors of 0, 1 and 2 increments), growth, more items than
workgroups, the misfit, and fields so small that the squared residuals pass the
point below which the kernel divides in full."""
import numpy as np
import pytest

import oracle
from gpu_common import THETA_TRUE, TAU, need_gpu

pytestmark = pytest.mark.gpu

THETAS = np.array([THETA_TRUE, (0.3, 0.6, 55.0, 5.0), (0.15, 0.8, 240.0, 50.0)])


def _problem(u0, v0, steps, rtol, rate=0.0, max_batch=8, y=None, **kw):
    from paper_1605_04718_amd.api import FP64, Grid, Problem
    g = Grid(n=32, u0=u0, v0=v0, growth=int(rate != 0.0), growth_rate=rate, y=y,
             **({} if y is None else {"sigma": 0.05}))
    return Problem(g, TAU, steps, rtol, precision=FP64, max_batch=max_batch, **kw)


def _rough(scale=1.0):
    rng = np.random.default_rng(9)
    return scale * rng.uniform(0.5, 1.5, (32, 32)), scale * rng.uniform(0.5, 1.5, (32, 32))


def _check(u0, v0, thetas, got_u, got_v, steps, rate, tol, rtol=1e-13):
    for k, th in enumerate(thetas):
        uo, vo, _, st = oracle.forward_solve(th, u0, v0, TAU, steps, rtol=rtol,
                                             growth=int(rate != 0.0), rate=rate)
        assert st == 0
        for got, want in ((got_u[k], uo), (got_v[k], vo)):
            assert np.linalg.norm(got - want) <= tol * np.linalg.norm(want)


@pytest.mark.parametrize("steps,rate", [(1, 0.0), (2, 0.0), (3, 0.01), (15, 0.01)])
def test_rough_fields_match_the_oracle_on_every_tile(steps, rate):
    import torch
    need_gpu()
    u0, v0 = _rough()
    y = np.random.default_rng(3).uniform(0.5, 1.5, (32, 32))
    p = _problem(u0, v0, steps, 1e-11, rate, y=y)
    th = torch.tensor(THETAS, device="cuda")
    first = None
    for cpt in (4, 8, 16):
        p.set_tile(0, cpt)
        u, v, st, it = (t.cpu().numpy() for t in p.forward_solve(th))
        assert np.all(st == 0)
        first = first or (u, v, it)
        for a, b in zip(first, (u, v, it)):
            assert np.array_equal(a, b)
    ll = p.log_likelihood(th)[0].cpu().numpy()
    p.close()
    # as the other field tests: 1.2 rtol |x| a step, 4 for its growth
    _check(u0, v0, THETAS, u, v, steps, rate, 2.0 ** -50 + 4 * 1.2 * steps * 1e-11)
    want = ((y - u) ** 2).sum(axis=(1, 2)) / (2 * 0.05 ** 2)
    assert np.allclose(np.abs(ll), want, rtol=1e-13)


def test_more_items_than_workgroups():
    import torch
    need_gpu()
    u0, v0 = _rough()
    m = 256 * 3 * 2 + 5
    p = _problem(u0, v0, 3, 1e-11, max_batch=m)
    th = torch.tensor(np.tile(THETAS, (m // 3 + 1, 1))[:m], device="cuda")
    u, v, st, _ = (t.cpu().numpy() for t in p.forward_solve(th))
    p.close()
    assert np.all(st == 0)
    _check(u0, v0, THETAS, u, v, 3, 0.0, 2.0 ** -50 + 4 * 1.2 * 3 * 1e-11)
    for k in range(m):
        assert np.array_equal(u[k], u[k % 3]) and np.array_equal(v[k], v[k % 3])


@pytest.mark.parametrize("scale", [1e-142, 1e-146])
def test_tiny_fields(scale):
    import torch
    need_gpu()
    u0, v0 = _rough(scale)
    thetas = np.array([(0.0, 0.0, 55.0, 5.0), (0.0, 0.0, 240.0, 50.0)])
    p = _problem(u0, v0, 3, 1e-7)
    u, v, st, _ = (t.cpu().numpy() for t in p.forward_solve(torch.tensor(thetas, device="cuda")))
    p.close()
    assert np.all(st == 0)
    _check(u0, v0, thetas, u, v, 3, 0.0, 4 * 1.2 * 3 * 1e-7, rtol=1e-9)
