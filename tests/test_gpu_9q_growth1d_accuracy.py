"""Rounding errors of the one-dimensional solve: its fields are no further from
a solve in extended precision than those of cyclic reduction over all rows in FP64,
and growth so fast that rho^2 overflows is solved (without diffusion)."""
import numpy as np
import pytest

import oracle.growth1d as og
from gpu_common import need_gpu
from paper_1605_04718_amd import inputs

pytestmark = pytest.mark.gpu

THETA = (0.1, 0.9, 1000.0, 10.0)


def _steps(beta, rho_t, tau, n_steps, real):
    beta = beta.astype(real)
    c = [beta[:, k] for k in range(3)]
    c.append(real(rho_t) - 1 - c[0] - c[1] - c[2])
    t_end = real(n_steps) * real(tau)
    for k in range(n_steps):
        s = real(k) * real(tau) / t_end
        rho = 1 + s * (c[0] + s * (c[1] + s * (c[2] + s * c[3])))
        drho = (c[0] + s * (2 * c[1] + s * (3 * c[2] + s * 4 * c[3]))) / t_end
        yield rho, drho


def _systems(x, rho, drho, tau, real):
    """Diagonal (without diffusion), right-hand side and diffusion of u and v;
    arrays [species, row, item]."""
    a, b, g, d = (real(t) for t in THETA)
    n = x.shape[1]
    u, v = x
    diag = 1 / real(tau) + drho / rho + g * np.stack([1 - u * v, u * u])
    k = real(n) * real(n) / (rho * rho)
    rhs = x / real(tau) + g * np.array([a, b], dtype=real)[:, None, None]
    return diag, rhs, np.stack([k, d * k])


def _thomas(diag, rhs, k):
    n = diag.shape[1]
    cp, x = np.empty_like(diag), np.empty_like(rhs)
    for i in range(n):
        main = diag[:, i] + k * ((i > 0) + (i < n - 1))
        if i:
            main = main - k * cp[:, i - 1]
        cp[:, i] = k / main
        x[:, i] = (rhs[:, i] + (k * x[:, i - 1] if i else 0)) / main
    for i in range(n - 2, -1, -1):
        x[:, i] += cp[:, i] * x[:, i + 1]
    return x


def _cyclic_reduction(diag, rhs, k):
    n = diag.shape[1]
    sides = np.full((1, n, 1), 2.0)
    sides[0, [0, -1]] = 1.0
    main, d = diag + k[:, None] * sides, rhs
    lo = np.broadcast_to(-k[:, None], main.shape).copy()
    up = lo.copy()
    lo[:, 0] = up[:, -1] = 0.0

    def shift(z, by, fill):
        out = np.full_like(z, fill)
        if by > 0:
            out[:, by:] = z[:, :-by]
        else:
            out[:, :by] = z[:, -by:]
        return out

    s = 1
    while s < n:
        fl, fu = lo / shift(main, s, 1.0), up / shift(main, -s, 1.0)
        main, d, lo, up = (main - fl * shift(up, s, 0.0) - fu * shift(lo, -s, 0.0),
                           d - fl * shift(d, s, 0.0) - fu * shift(d, -s, 0.0),
                           -fl * shift(lo, s, 0.0), -fu * shift(up, -s, 0.0))
        s *= 2
    return d / main


@pytest.mark.parametrize("n", [40, 128])
def test_no_further_off_than_cyclic_reduction(n):
    import torch
    from paper_1605_04718_amd.api import Growth1D
    need_gpu()
    items, n_steps, tau = 48, 1000, 1e-4
    u0, v0 = inputs.initial_fields_1d(n)
    rho_t = np.exp(0.001 * n_steps * tau)
    beta = inputs.box_draws(items, (-0.2, -0.2, -0.2), (0.4, 0.2, 0.2), seed=7)
    p = Growth1D(n, n_steps, tau, THETA, u0, v0, rho_T=rho_t, max_batch=items)
    u, v, st = p.forward(torch.tensor(beta, device="cuda"))
    p.close()
    assert not st.any()
    got = np.stack([u.cpu().numpy().T, v.cpu().numpy().T])
    ends = []
    for real, solve in ((np.longdouble, _thomas), (np.float64, _cyclic_reduction)):
        x = np.repeat(np.stack([u0, v0]).astype(real)[:, :, None], items, 2)
        for rho, drho in _steps(beta, rho_t, tau, n_steps, real):
            x = solve(*_systems(x, rho, drho, tau, real))
        ends.append(x)
    want, other = ends
    for s in range(2):
        err = [float(np.sqrt(np.mean((z[s] - want[s]) ** 2))) for z in (got, other)]
        assert err[0] <= 1.05 * err[1], (s, err)  # (rounding: 5 % for the sample)


def test_growth_whose_square_overflows():
    import torch
    from paper_1605_04718_amd.api import Growth1D
    need_gpu()
    n, n_steps, tau = 24, 5, 1.25e5  # rho = exp(125 k); rho^2 = exp(750), inf, at k = 3
    theta = (0.1, 0.9, 1e-7, 10.0)
    u0, v0 = inputs.initial_fields_1d(n)
    p = Growth1D(n, n_steps, tau, theta, u0, v0, law=Growth1D.EXP, max_batch=1)
    u, v, st = p.forward(m=1)
    p.close()
    assert int(st[0]) == 0
    uo, vo = og.forward(theta, u0, v0, tau, n_steps, og.rho_exp_pair)
    for a, b in ((u, uo), (v, vo)):
        assert np.allclose(a[0].cpu().numpy(), b, rtol=1e-12, atol=0)
