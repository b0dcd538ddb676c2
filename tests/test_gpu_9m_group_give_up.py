"""Group waits that give up anywhere in an item (256 x 256, groups of four
workgroups), forced from the host by a bound of a few microseconds on a
kernel's own waits: an item is either reported as timed out, with a misfit of
+inf, or its fields and misfit are the same bits as with the default bound."""
import numpy as np
import pytest

from gpu_common import THETA_TRUE, TAU, need_gpu, theta_batch
from paper_1605_04718_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,cpt,steps", [(0, 32, 3), (1, 32, 2), (0, 16, 2), (0, 32, 0),
                                                 (1, 32, 0)])
def test_an_item_is_whole_or_reported(precision, cpt, steps):
    import torch
    from paper_1605_04718_amd._lib import ST_GROUP_TIMEOUT
    from paper_1605_04718_amd.api import Grid, Problem
    need_gpu()
    n, m = 256, 128
    u0, v0 = inputs.initial_fields(n, THETA_TRUE[0], THETA_TRUE[1])
    p = Problem([Grid(n=n, u0=u0, v0=v0, y=u0 + 0.01, sigma=0.05)], TAU, steps, 1e-5,
                precision=precision, max_batch=m)
    p.set_tile(0, cpt)
    th = torch.tensor(theta_batch(m, seed=5), device="cuda")
    want_u, want_v, st, _ = p.forward_solve(th)
    want_phi, st2, _ = p.log_likelihood(th)
    assert not st.any() and not st2.any() and p.check_solves() == 0
    seen = np.zeros(2, dtype=int)
    for wait in (1, 30, 60, 90, 120, 160, 200, 250, 300, 400, 600, 1000):
        p.set_coop_wait(wait_ticks=wait, stall_ticks=0)
        for _ in range(4):
            print(f"256^2 precision {precision} cpt {cpt}: wait {wait} ticks", flush=True)
            u, v, st, _ = p.forward_solve(th)
            phi, st2, _ = p.log_likelihood(th)
            torch.cuda.synchronize()
            p.group_timeouts()
            for s in (st, st2):
                assert bool(((s == 0) | (s == ST_GROUP_TIMEOUT)).all()), s.unique()
                seen += [int((s == 0).sum()), int((s != 0).sum())]
            ok, ok2 = st == 0, st2 == 0
            same = [torch.equal(u[ok], want_u[ok]), torch.equal(v[ok], want_v[ok]),
                    torch.equal(phi[ok2], want_phi[ok2])]
            assert all(same), (wait, same)
            assert bool(torch.isinf(phi[~ok2]).all())
    p.close()
    print("whole, reported:", seen)
    assert seen.min() > 0  # both outcomes were met
