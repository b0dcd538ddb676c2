"""Stiff systems: 8 c dt (the ratio of the operator's largest eigenvalue to its
smallest, less one) from 1e4 to 3e7, by the diffusion ratio and by the time step,
where one application of the preconditioner spans that ratio in its FP16 stages."""
import numpy as np
import pytest

import oracle
from gpu_common import TAU, need_gpu, rel_l2

pytestmark = pytest.mark.gpu

STIFF = np.array([1e4, 1e5, 1e6, 1e7, 3e7])


def _solve(n, fp64, dt, gamma, steps, rtol, u0, v0, stiff, **kw):
    import torch
    from paper_1605_04718_amd.api import Grid, Problem
    d = stiff / (8 * n * n * dt)
    thetas = np.stack([np.full_like(d, 0.1), np.full_like(d, 0.9), np.full_like(d, gamma), d], 1)
    p = Problem(Grid(n=n, u0=u0, v0=v0), dt, steps, rtol, precision=fp64, max_batch=len(d), **kw)
    print(f"stiff {n}^2 fp64 {fp64} dt {dt}", flush=True)
    u, v, st, it = p.forward_solve(torch.tensor(thetas, device="cuda"))
    u, v, st, it = (t.cpu().numpy() for t in (u, v, st, it))
    p.close()
    return thetas, u, v, st, it


def _rough(n):
    rng = np.random.default_rng(9)
    return rng.uniform(0.5, 1.5, (n, n)), rng.uniform(0.5, 1.5, (n, n))


@pytest.mark.parametrize("n,fp64", [(32, 0), (64, 0), (128, 0), (256, 0), (64, 1), (128, 1),
                                    (256, 1)])
@pytest.mark.parametrize("dt,gamma", [(TAU, 200.0), (0.01, 5.0)])
def test_stiff_systems_converge(n, fp64, dt, gamma):
    need_gpu()
    steps, rtol = 2, 1e-9 if fp64 else 1e-7
    u0, v0 = _rough(n)
    thetas, u, v, st, _ = _solve(n, fp64, dt, gamma, steps, rtol, u0, v0, STIFF, cg_maxit=4000)
    assert np.all(st == 0), st
    for k, th in enumerate(thetas):
        if not fp64 and STIFF[k] > 1e4:
            continue  # (the FP32 operator's own rounding, 2^-24 8 c dt, shows there)
        uo, vo, _, so = oracle.forward_solve(th, u0, v0, dt, steps, rtol=1e-13)
        assert so == 0
        # as the other field tests, and the rounding of A d in FP32
        tol = 4 * 1.2 * steps * rtol + (2.0 ** -50 if fp64 else 2.0 ** -24 * (1 + STIFF[k]))
        for got, want in ((u[k], uo), (v[k], vo)):
            assert rel_l2(got, want) <= tol, (k, rel_l2(got, want), tol)
