"""Sums over a group of workgroups (256 x 256) carry all bits of FP64: the misfit
of an FP64 solve against the exactly rounded sum over its own fields, and the
plain-CG group (16 cells per thread), whose results must not depend on how many
exchanges its group made before."""
import math

import numpy as np
import pytest

from gpu_common import THETA_TRUE, TAU, need_gpu, theta_batch
from paper_1605_04718_amd import inputs

pytestmark = pytest.mark.gpu


def test_fp64_misfit_is_summed_in_fp64():
    import torch
    from paper_1605_04718_amd.api import FP64, Grid, Problem
    need_gpu()
    n, m, sigma = 256, 12, 0.25  # (a power of two: dividing by 2 sigma^2 is exact)
    u0, v0 = inputs.initial_fields(n, THETA_TRUE[0], THETA_TRUE[1])
    y = u0 + np.random.default_rng(4).normal(0.0, 0.05, (n, n))
    p = Problem([Grid(n=n, u0=u0, v0=v0, y=y, sigma=sigma)], TAU, 2, 1e-9, precision=FP64,
                max_batch=m)
    th = torch.tensor(theta_batch(m, seed=6), device="cuda")
    phi, st, _ = p.log_likelihood(th)
    u, _, st2, _ = p.forward_solve(th)
    phi, u = phi.cpu().numpy(), u.cpu().numpy()
    p.close()
    assert not st.any() and not st2.any()
    for k in range(m):
        e = (y - u[k].reshape(n, n)).ravel()
        # the squares exactly, by splitting at 26 bits
        hi = (e * 134217729.0) - (e * 134217729.0 - e)
        lo = e - hi
        want = math.fsum(np.concatenate([hi * hi, 2 * hi * lo, lo * lo])) / (2 * sigma ** 2)
        # positive terms: 32 fused additions per thread, then 6 + 4 + 4 levels
        assert abs(phi[k] - want) <= 46 * 2.0 ** -53 * want, (k, phi[k] / want - 1)


def test_plain_cg_group_gives_the_same_bits_to_every_copy():
    import torch
    from paper_1605_04718_amd.api import Grid, Problem
    need_gpu()
    n, copies = 256, 64
    u0, v0 = inputs.initial_fields(n, THETA_TRUE[0], THETA_TRUE[1])
    p = Problem([Grid(n=n, u0=u0, v0=v0, y=u0 + 0.01, sigma=0.05)], TAU, 3, 1e-7,
                max_batch=3 * copies)
    p.set_tile(0, 16)
    th = torch.tensor(np.tile(theta_batch(3, seed=7), (copies, 1)), device="cuda")
    phi, st, _ = p.log_likelihood(th)
    assert not st.any() and p.check_solves() == 0
    p.close()
    phi = phi.reshape(copies, 3)
    assert torch.equal(phi, phi[:1].expand_as(phi))
