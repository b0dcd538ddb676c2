"""log_likelihood_batch_noalloc at 256 x 256 in FP64, where groups of workgroups
solve an item: the kernels of log_likelihood_batch on the library's scratch, so
the same bits, with fewer and more items than the scratch holds groups, on the
streamed tile, under a small iteration cap, with stiff items, and replayed from a
HIP graph."""
import numpy as np
import pytest

from gpu_common import THETA_TRUE, TAU, need_gpu, theta_batch
from paper_1605_04718_amd import inputs
from test_zz_no_alloc import noalloc

pytestmark = pytest.mark.gpu


def _problem(max_batch, **kw):
    from paper_1605_04718_amd.api import FP64, Grid, Problem
    u0, v0 = inputs.initial_fields(256, THETA_TRUE[0], THETA_TRUE[1])
    return Problem(Grid(n=256, u0=u0, v0=v0, y=u0 + 0.01, sigma=0.05), TAU, 3, 1e-10,
                   max_batch=max_batch, precision=FP64, **kw)


def _thetas(m, seed):
    import torch
    th = np.vstack([THETA_TRUE, theta_batch(m, seed=seed)[: m - 1]])
    th[m // 2, 3] = 1e8  # (left to plain CG)
    return torch.tensor(th, device="cuda")


@pytest.mark.parametrize("cpt,maxit,m", [(32, 0, 1), (32, 0, 7), (32, 0, 75), (128, 0, 3),
                                         (32, 12, 3)])
def test_same_bits_as_the_allocating_call(cpt, maxit, m):
    import torch
    need_gpu()
    p = _problem(m, cg_maxit=maxit)
    p.set_tile(0, cpt)
    for seed in (3, 4):
        th = _thetas(m, seed)
        print(f"noalloc 256^2 FP64 cpt {cpt}, cap {maxit}: {m} items", flush=True)
        got = noalloc(p, th)
        want = p.log_likelihood(th)
        torch.cuda.synchronize()
        for a, b in zip(got, (want[0], want[1], want[2])):
            assert torch.equal(a, b)
        assert maxit or not want[1].any()
    assert p.check_solves() == 0
    p.close()


def test_replayed_from_a_graph():
    import torch
    from paper_1605_04718_amd import _lib
    from paper_1605_04718_amd.api import _ptr
    need_gpu()
    p = _problem(9)
    th = _thetas(9, 5)
    phi = torch.zeros(9, dtype=torch.float64, device="cuda")
    st = torch.zeros(9, dtype=torch.int32, device="cuda")
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        _lib.check(_lib.lib().log_likelihood_batch_noalloc(
            p.h, 9, _ptr(th), _ptr(phi), _ptr(st), None, side.cuda_stream), "noalloc")
    for seed in (6, 7, 8):
        th.copy_(_thetas(9, seed))
        want, want_st, _ = p.log_likelihood(th)
        phi.fill_(-1.0)
        st.fill_(-7)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(phi, want) and torch.equal(st, want_st)
    p.close()
