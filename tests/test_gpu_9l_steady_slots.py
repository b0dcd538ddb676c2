"""Steady-state stopping of the FP64 solves that refine their increments (64 x
64, 128 x 128): the true residual of the last refinement and the step size are
two workgroup sums in a row.  Every copy of an item must take the same steps
and give the same bits, as must a second run, and the stopping step is the
oracle's."""
import numpy as np
import pytest

import oracle
from gpu_common import TAU, need_gpu, rel_l2
from paper_1605_04718_amd import inputs

pytestmark = pytest.mark.gpu

THETAS = np.array([(0.1, 0.9, 200.0, 10.0), (0.1, 0.9, 200.0, 1.0)])


@pytest.mark.parametrize("n,cap,tol,copies", [(64, 400, 0.02, 200), (128, 200, 0.02, 100)])
def test_every_copy_stops_at_the_oracles_step(n, cap, tol, copies):
    import torch
    from paper_1605_04718_amd.api import FP64, Grid, Problem
    need_gpu()
    u0, v0 = inputs.initial_fields(n, 0.1, 0.9)
    p = Problem([Grid(n=n, u0=u0, v0=v0)], TAU, cap, 1e-12, precision=FP64,
                max_batch=2 * copies, steady_tol=tol)
    th = torch.tensor(np.tile(THETAS, (copies, 1)), device="cuda")
    print(f"steady FP64 {n}^2: {2 * copies} items, twice", flush=True)
    runs = [p.forward_solve_steady(th) for _ in range(2)]
    torch.cuda.synchronize()
    u, v, st, it, steps = runs[0]
    for run in runs:
        for t in run:
            t = t.reshape((copies, 2) + t.shape[1:])
            assert torch.equal(t, t[:1].expand_as(t))
    for a, b in zip(*runs):
        assert torch.equal(a, b)
    for k, theta in enumerate(THETAS):
        uo, vo, so, _, sto = oracle.forward_solve_steady(theta, u0, v0, TAU, cap, tol, rtol=1e-12)
        assert sto == int(st[k]) == 0 and int(steps[k]) == so
        assert so > 3  # (the stop is not the first step's)
        # FP64 fields after a few hundred steps at rtol 1e-12, as the other
        # steady-state test
        assert rel_l2(u[k].cpu().numpy().reshape(n, n), uo) < 1e-9
        assert rel_l2(v[k].cpu().numpy().reshape(n, n), vo) < 1e-9
    p.close()


@pytest.mark.parametrize("precision", [0, 1])
def test_misfit_after_a_steady_stop_of_the_streamed_tile(precision):
    """The streamed 256 x 256 solve: the misfit's sum follows the step size's."""
    import torch
    from paper_1605_04718_amd.api import Grid, Problem
    need_gpu()
    n, cap, tol, copies = 256, 60, 0.1, 24
    u0, v0 = inputs.initial_fields(n, 0.1, 0.9)
    y, sigma = inputs.noisy_data(u0, 0.01)
    p = Problem([Grid(n=n, u0=u0, v0=v0, y=y, sigma=sigma)], TAU, cap, 1e-7, precision=precision,
                max_batch=copies, steady_tol=tol)
    p.set_tile(0, 128)
    th = torch.tensor(np.tile(THETAS[:1], (copies, 1)), device="cuda")
    print(f"streamed steady 256^2, precision {precision}", flush=True)
    phi, st, _ = p.log_likelihood(th)
    u, _, st2, _, steps = p.forward_solve_steady(th)
    torch.cuda.synchronize()
    p.close()
    assert not st.any() and not st2.any() and int(steps.max()) == int(steps.min()) < cap
    assert torch.equal(phi, phi[:1].expand_as(phi))
    want = ((y - u[0].double().cpu().numpy().reshape(n, n)) ** 2).sum() / (2 * sigma ** 2)
    # FP32: u is read back rounded to 2^-24 of |u| = 1, against residuals of
    # about 0.05 in each cell
    assert abs(float(phi[0]) - want) <= (1e-5 if precision == 0 else 1e-12) * want
