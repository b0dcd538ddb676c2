"""FP64 solves of 64 x 64 to 256 x 256 outside the range of their FP32 corrections:
fields of any size that FP64 plain CG takes, fields that leave the range on the
way, and systems stiffer than 8 c dt = 2^24, alone and beside ordinary items."""
import numpy as np
import pytest

import oracle
from gpu_common import THETA_TRUE, TAU, need_gpu, rel_l2
from paper_1605_04718_amd import inputs

pytestmark = pytest.mark.gpu

SIZES = [64, 128, 256]


def _rough(n):
    rng = np.random.default_rng(9)
    return rng.uniform(0.5, 1.5, (n, n)), rng.uniform(0.5, 1.5, (n, n))


def _problem(grids, dt, steps, rtol, max_batch=64, **kw):
    from paper_1605_04718_amd.api import FP64, Problem
    return Problem(grids, dt, steps, rtol, precision=FP64, max_batch=max_batch, **kw)


def _run(p, thetas, grid_id=None):
    import torch
    th = torch.tensor(np.asarray(thetas, dtype=np.float64), device="cuda")
    gid = None if grid_id is None else torch.tensor(grid_id, dtype=torch.int32, device="cuda")
    u, v, st, it = (t.cpu().numpy() for t in p.forward_solve(th, grid_id=gid))
    return u, v, st, it


def _tol(steps, rtol):
    # as the other field tests: 1.2 rtol |x| a step, 4 for its growth
    return 2.0 ** -50 + 4 * 1.2 * steps * rtol


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("scale", [1e-13, 1e-30, 1e-45, 1e-120, 1e13, 1e60, 1e120])
def test_fields_of_any_size(n, scale):
    """Without a reaction the solve is linear: scaled fields give the scaled result."""
    from paper_1605_04718_amd.api import Grid
    need_gpu()
    steps, rtol = 3, 1e-10
    u0, v0 = _rough(n)
    thetas = [(0.1, 0.9, 0.0, 10.0), (0.1, 0.9, 0.0, 50.0)]
    p = _problem(Grid(n=n, u0=u0 * scale, v0=v0 * scale), TAU, steps, rtol)
    print(f"fields {scale} {n}^2", flush=True)
    u, v, st, _ = _run(p, thetas)
    p.close()
    assert np.all(st == 0), st
    for k, th in enumerate(thetas):
        uo, vo, _, so = oracle.forward_solve(th, u0, v0, TAU, steps, rtol=1e-13)
        assert so == 0
        assert rel_l2(u[k] / scale, uo) <= _tol(steps, rtol)
        assert rel_l2(v[k] / scale, vo) <= _tol(steps, rtol)


@pytest.mark.parametrize("n", SIZES)
def test_fields_that_decay_out_of_range(n):
    """a = b = 0: u falls by a factor of about six a step."""
    from paper_1605_04718_amd.api import Grid
    need_gpu()
    steps, rtol, dt = 60, 1e-9, 0.01
    u0, v0 = _rough(n)
    theta = (0.0, 0.0, 500.0, 5.0)
    p = _problem(Grid(n=n, u0=u0, v0=0.01 * v0), dt, steps, rtol)
    u, v, st, _ = _run(p, [theta, theta])
    p.close()
    assert np.all(st == 0), st
    uo, vo, _, so = oracle.forward_solve(theta, u0, 0.01 * v0, dt, steps, rtol=1e-13)
    assert so == 0 and np.abs(uo).max() < 1e-30
    assert rel_l2(u[0], uo) <= _tol(steps, rtol) and rel_l2(v[0], vo) <= _tol(steps, rtol)


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("dt,gamma", [(TAU, 200.0), (0.1, 0.5)])
def test_systems_of_any_stiffness(n, dt, gamma):
    from paper_1605_04718_amd.api import Grid
    need_gpu()
    steps, rtol = 2, 1e-10
    u0, v0 = _rough(n)
    stiff = np.array([1e3, 1e7, 3e7, 1e9, 1e12])
    thetas = np.stack([np.full(5, 0.1), np.full(5, 0.9), np.full(5, gamma),
                       stiff / (8 * n * n * dt)], 1)
    p = _problem(Grid(n=n, u0=u0, v0=v0), dt, steps, rtol)
    print(f"stiffness {n}^2 dt {dt}", flush=True)
    u, v, st, _ = _run(p, thetas)
    p.close()
    assert np.all(st == 0), st
    for k, th in enumerate(thetas):
        uo, vo, _, so = oracle.forward_solve(th, u0, v0, dt, steps, rtol=1e-13)
        assert so == 0
        tol = _tol(steps, rtol) + 2.0 ** -53 * stiff[k]  # the rounding of A d in FP64
        assert rel_l2(u[k], uo) <= tol and rel_l2(v[k], vo) <= tol, (k, tol)


def test_mixed_batch_with_items_out_of_range():
    """Stiff items of every class among ordinary ones, which keep their bits."""
    from paper_1605_04718_amd.api import Grid
    need_gpu()
    steps, rtol = 2, 1e-9
    fields = {n: _rough(n) for n in (256, 32, 128, 64)}
    grids = [Grid(n=n, u0=f[0], v0=f[1]) for n, f in fields.items()]
    p = _problem(grids, TAU, steps, rtol)
    gid = np.tile(np.arange(4), 6).astype(np.int32)
    ordinary = np.tile(np.array([THETA_TRUE]), (24, 1))
    thetas = ordinary.copy()
    stiff = np.zeros(24, dtype=bool)
    stiff[[0, 5, 2, 11, 17, 16]] = True
    thetas[stiff, 3] = 1e8
    u0, v0, st0, _ = _run(p, ordinary, gid)
    u, v, st, _ = _run(p, thetas, gid)
    bad = gid.copy()
    bad[3] = 9
    _, _, st1, _ = _run(p, thetas, bad)
    p.close()
    assert np.all(st0 == 0) and np.all(st == 0)
    assert st1[3] == 16 and np.all(np.delete(st1, 3) == 0)
    for k, n in enumerate(np.array(list(fields))[gid]):
        # (a row holds the largest class; an item fills its start)
        a, b = u.reshape(24, -1)[k, :n * n], v.reshape(24, -1)[k, :n * n]
        if not stiff[k]:
            assert np.array_equal(a, u0.reshape(24, -1)[k, :n * n])
            assert np.array_equal(b, v0.reshape(24, -1)[k, :n * n])
            continue
        uo, vo, _, so = oracle.forward_solve(thetas[k], *fields[n], TAU, steps, rtol=1e-13)
        assert so == 0
        assert rel_l2(a, uo.ravel()) <= _tol(steps, rtol)
        assert rel_l2(b, vo.ravel()) <= _tol(steps, rtol)


def test_captured_chain_with_stiff_proposals():
    """Metropolis steps of an FP64 64 x 64 problem whose proposals reach d = 1e8:
    replays of the captured step against direct launches, bit for bit."""
    import torch
    from paper_1605_04718_amd.api import ChainState, Grid
    need_gpu()
    n = 64
    u0, v0 = inputs.initial_fields(n, THETA_TRUE[0], THETA_TRUE[1])
    uo, _, _, _ = oracle.forward_solve(THETA_TRUE, u0, v0, TAU, 2, rtol=1e-12)
    y, sigma = inputs.noisy_data(uo, 0.01)
    states = []
    for captured in (False, True):
        p = _problem([Grid(n=n, u0=u0, v0=v0, y=y, sigma=100 * sigma)], TAU, 2, 1e-9,
                     lo=(0.0, 0.0, np.log(50.0), np.log(5.0)),
                     hi=(1.0, 1.0, np.log(500.0), np.log(1e9)), step=(0.02, 0.02, 0.05, 5.0),
                     free_mask=0b1111, max_batch=16)
        phi = torch.tensor(np.tile([THETA_TRUE[0], THETA_TRUE[1], np.log(200.0), np.log(1e4)],
                                   (16, 1)), device="cuda")
        ch = ChainState.create(phi, torch.full((16,), np.inf, dtype=torch.float64, device="cuda"),
                               seed=3, trace_steps=8)
        torch.cuda.synchronize()
        with torch.cuda.stream(torch.cuda.Stream() if captured else torch.cuda.default_stream()):
            for _ in range(8):
                p.mcmc_step(ch, 1)
                torch.cuda.synchronize()
        assert (p.captured_graphs() > 0) == captured
        states.append([t.cpu().numpy() for t in (ch.trace, ch.loglik, ch.n_solves, ch.fail_bits)])
        p.close()
    for a, b in zip(*states):
        assert np.array_equal(a, b)
    trace, loglik, _, failed = states[0]
    assert np.exp(trace[:, :, 3]).max() > 1e7  # stiff states were reached
    assert np.isfinite(loglik).all() and not failed.any()


def _near_singular(n, nearness):
    """Fields and the gamma at which 1/dt + gamma (1 - u v) + N^2 L, less `nearness` of
    gamma, becomes singular; and that step's u by a direct solve."""
    import scipy.sparse as sp
    import scipy.sparse.linalg as sl
    x = (np.arange(n) + 0.5) / n
    w = np.cos(np.pi * x)[:, None] * np.cos(2 * np.pi * x)[None, :]
    u0, v0 = 1 + 0.3 * w, 3 + w.T
    e = np.ones(n)
    one = sp.diags([np.r_[1, 2 * np.ones(n - 2), 1], -e[:-1], -e[:-1]], [0, 1, -1])
    lap = sp.kron(one, sp.identity(n)) + sp.kron(sp.identity(n), one)
    m = (sp.identity(n * n) / TAU + n * n * lap).tocsc()
    q = sp.diags((u0 * v0 - 1).ravel())
    lu = sl.splu(m)
    op = sl.LinearOperator((n * n, n * n), matvec=lambda y: lu.solve(q @ y))
    gamma = 1 / sl.eigs(op, k=1, which="LR", tol=1e-15, v0=np.ones(n * n))[0][0].real
    gamma *= 1 - nearness
    u = sl.splu((m - gamma * q).tocsc()).solve(u0.ravel() / TAU + gamma * 0.1)
    return u0, v0, gamma, u.reshape(n, n)


@pytest.mark.parametrize("n", [64, 128])
@pytest.mark.parametrize("nearness", [1e-2, 1e-4, 1e-6, 1e-8])
@pytest.mark.parametrize("rtol", [1e-7, 1e-12])
def test_nearly_singular_systems(n, nearness, rtol):
    from paper_1605_04718_amd.api import Grid
    need_gpu()
    u0, v0, gamma, want = _near_singular(n, nearness)
    p = _problem(Grid(n=n, u0=u0, v0=v0), TAU, 1, rtol)
    print(f"singular within {nearness}: {n}^2 rtol {rtol}", flush=True)
    u, _, st, _ = _run(p, [(0.1, 0.9, gamma, 10.0)])
    p.close()
    assert st[0] == 0
    # the smallest eigenvalue is nearness / dt and the largest about 8 N^2: a
    # residual of rtol |b| (the rounding of either solve: 2^-53 (1 + 8 N^2 dt)
    # |x'| / dt) is an error of so much of x' over nearness; 10 for the norms
    eps = 2.0 ** -53 * (1 + 8 * n * n * TAU)
    tol = 10 * (rtol * np.linalg.norm(u0) / np.linalg.norm(want) + 2 * eps) / nearness
    assert rel_l2(u[0], want) <= tol, (rel_l2(u[0], want), tol)


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("rtol", [1e-14, 1e-15, 1e-17])
def test_tolerances_below_the_rounding(n, rtol):
    from paper_1605_04718_amd.api import Grid
    need_gpu()
    u0, v0 = _rough(n)
    thetas = [THETA_TRUE, (0.15, 0.8, 240.0, 50.0)]
    p = _problem(Grid(n=n, u0=u0, v0=v0), TAU, 3, rtol)
    u, v, st, _ = _run(p, thetas)
    p.close()
    assert np.all(st == 0), st
    for k, th in enumerate(thetas):
        uo, vo, _, so = oracle.forward_solve(th, u0, v0, TAU, 3, rtol=1e-14)
        assert so == 0
        # both to 2^-53 of x through an operator of 8 c dt (c = 50 N^2 at most)
        tol = 4 * 3 * 2.0 ** -53 * (1 + 8 * th[3] * n * n * TAU) + 4 * 1.2 * 3 * 1e-14
        assert rel_l2(u[k], uo) <= tol and rel_l2(v[k], vo) <= tol
