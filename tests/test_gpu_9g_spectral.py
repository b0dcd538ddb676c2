"""The spectrally preconditioned solve against the FP64 oracle: every grid size
and precision that takes it, the first steps (where the start vector uses 0, 1 and 2 increments),
both ends of the diffusion ratio (the preconditioner's work grows with d),
growing domain, more items than one workgroup, and the iteration cap."""
import numpy as np
import pytest

import oracle
from gpu_common import THETA_TRUE, TAU, need_gpu
from paper_1605_04718_amd import inputs

pytestmark = pytest.mark.gpu

THETAS = np.array([THETA_TRUE, (0.3, 0.6, 55.0, 5.0), (0.15, 0.8, 240.0, 50.0)])


def _problem(n, steps, rtol, **kw):
    from paper_1605_04718_amd.api import Grid, Problem
    u0, v0 = inputs.initial_fields(n, THETA_TRUE[0], THETA_TRUE[1])
    rate = kw.pop("rate", 0.0)
    g = Grid(n=n, u0=u0, v0=v0, growth=int(rate != 0.0), growth_rate=rate)
    return Problem(g, TAU, steps, rtol, max_batch=8, **kw), u0, v0


@pytest.mark.parametrize("n,fp64", [(32, 0), (64, 0), (128, 0), (256, 0), (64, 1), (128, 1),
                                    (256, 1)])
@pytest.mark.parametrize("steps,rate,rtol", [(0, 0.0, 1e-9), (1, 0.0, 1e-9), (2, 0.0, 1e-9),
                                             (3, 0.01, 1e-9), (12, 0.0, 1e-9), (12, 0.01, 1e-7)])
def test_fields_match_the_oracle(n, fp64, steps, rate, rtol):
    import torch
    need_gpu()
    p, u0, v0 = _problem(n, steps, rtol, rate=rate, precision=fp64)
    u, v, status, _ = p.forward_solve(torch.tensor(np.tile(THETAS, (2, 1)), device="cuda"))
    assert p.check_solves() == 0
    u, v, status = u.double().cpu().numpy(), v.double().cpu().numpy(), status.cpu().numpy()
    p.close()
    # a step's residual of at most rtol |b| with |b| <= (1/dt + gamma) |x| and
    # A >= 1/dt moves the field by at most 1.2 rtol |x|; 4 covers its growth
    # over a few steps, and the output is rounded to FP32 (2^-24) or FP64
    tol = (2.0 ** -50 if fp64 else 2.0 ** -24) + 4 * 1.2 * steps * rtol
    for k in range(6):
        uo, vo, _, st = oracle.forward_solve(THETAS[k % 3], u0, v0, TAU, steps, rtol=1e-13,
                                             growth=int(rate != 0.0), rate=rate)
        assert st == 0 and status[k] == 0
        for got, want in ((u[k], uo), (v[k], vo)):
            err = np.linalg.norm(got - want) / np.linalg.norm(want)
            assert err <= tol, (k, err, tol)
    assert np.array_equal(u[:3], u[3:]) and np.array_equal(v[:3], v[3:])


@pytest.mark.parametrize("n,fp64", [(32, 0), (64, 0), (128, 0), (256, 0), (64, 1), (128, 1),
                                    (256, 1)])
def test_iteration_cap_is_reported(n, fp64):
    import torch
    need_gpu()
    p, _, _ = _problem(n, 3, 1e-9, cg_maxit=2, precision=fp64)
    _, _, status, it = p.forward_solve(torch.tensor(THETAS, device="cuda"))
    assert np.all(status.cpu().numpy() == 1)   # two plain iterations do not reach 1e-9 at step 0
    assert np.all(it.cpu().numpy().max(axis=1) == 2)
    p.close()


@pytest.mark.parametrize("fp64", [0, 1])
def test_groups_take_several_items_in_turn(fp64):
    """More 256^2 items than groups: copies of three parameter vectors give
    the same bits in every group, and no group gives up a wait."""
    import torch
    from paper_1605_04718_amd.api import Grid, Problem
    need_gpu()
    u0, v0 = inputs.initial_fields(256, THETA_TRUE[0], THETA_TRUE[1])
    p = Problem(Grid(n=256, u0=u0, v0=v0), TAU, 4, 1e-9, max_batch=150, precision=fp64)
    u, v, status, it = p.forward_solve(torch.tensor(np.tile(THETAS, (50, 1)), device="cuda"))
    assert p.check_solves() == 0
    u, v, status, it = (t.cpu().numpy() for t in (u, v, status, it))
    assert np.all(status == 0)
    for t in (u, v, it):
        t = t.reshape((50, 3) + t.shape[1:])
        assert np.array_equal(t, np.broadcast_to(t[:1], t.shape))
    p.close()


def test_fp64_noalloc_at_256_keeps_a_tile_that_needs_no_group():
    import torch
    from paper_1605_04718_amd import _lib
    from paper_1605_04718_amd.api import Grid, Problem, _ptr
    need_gpu()
    u0, v0 = inputs.initial_fields(256, THETA_TRUE[0], THETA_TRUE[1])
    p = Problem(Grid(n=256, u0=u0, v0=v0, y=u0 + 0.01, sigma=0.05), TAU, 2, 1e-10, max_batch=3,
                precision=1)
    th = torch.tensor(THETAS, device="cuda")
    want, st, _ = p.log_likelihood(th)
    got, st2 = torch.empty_like(want), torch.empty_like(st)
    _lib.check(_lib.lib().log_likelihood_batch_noalloc(
        p.h, 3, _ptr(th), _ptr(got), _ptr(st2), None, None), "log_likelihood_batch_noalloc")
    torch.cuda.synchronize()
    assert not st.any() and not st2.any()
    # fields within 4 * 1.2 * 2 * 1e-10 of each other move a misfit of
    # differences of about 0.01 by less than 2e-7 of itself
    assert torch.allclose(got, want, rtol=1e-6, atol=0)
    p.close()
