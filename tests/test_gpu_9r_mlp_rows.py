"""Surrogate batches past a million rows, whose first layer takes more blocks of
16 rows than a grid's second dimension holds."""
import numpy as np
import pytest

from gpu_common import need_gpu

pytestmark = pytest.mark.gpu


def test_more_than_a_million_rows():
    import torch
    from paper_1605_04718_amd.api import Grid, Problem
    need_gpu()
    rows, n = 65536 * 16 + 100, 32
    rng = np.random.default_rng(2)
    y = rng.uniform(0.5, 1.5, (n, n))
    lo, hi = (0.0, 0.0, 3.0, 1.0), (1.0, 1.0, 6.0, 4.0)
    p = Problem(Grid(n=n, u0=y, v0=y, y=y, sigma=0.1), 2.5e-4, 1, 1e-7, lo=lo, hi=hi,
                max_batch=rows)
    p.surrogate_create(width=64, depth=1, out_side=8, seed=5)
    p.surrogate_set_scaling(torch.zeros(64, device="cuda"), torch.ones(64, device="cuda"), 0.1)
    phi = torch.tensor(rng.uniform(lo, hi, (rows, 4)), device="cuda")
    print(f"surrogate misfits of {rows} rows", flush=True)
    ll = p.surrogate_loglik(phi)
    torch.cuda.synchronize()
    for at in (0, rows // 2, rows - 64):
        few = p.surrogate_loglik(phi[at:at + 64].contiguous())
        # (another tile: the same sums of 64 BF16 products in another order)
        assert torch.allclose(ll[at:at + 64], few, rtol=1e-5, atol=0)
    p.close()
