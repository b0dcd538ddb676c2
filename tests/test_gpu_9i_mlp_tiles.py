"""The surrogate's products at the edges of their tiles: widths that are odd
multiples of 64 (K steps of 64), 128 and 256, one layer and several, batches
below, at and above the padding, and a batch large enough for the tall tiles."""
import numpy as np
import pytest
from scipy.special import erf

from oracle import mlp as omlp
from gpu_common import need_gpu, rel_l2
from paper_1605_04718_amd import inputs
from test_gpu_3_surrogate import HI, LO, host_params, small_problem

pytestmark = pytest.mark.gpu


def bf16(x):
    import torch
    return torch.tensor(np.asarray(x)).to(torch.bfloat16).double().numpy()


def reference(params, x, target):
    """Forward and backward in FP64 with the roundings that the network makes:
    BF16 weights, activations and output gradients of the layers after the
    first; FP32 (here FP64) first layer, sums and epilogues."""
    w = [W if i == 0 else bf16(W) for i, (W, _) in enumerate(params)]
    h, zs, hs = x, [], [x]
    for i, (_, b) in enumerate(params):
        z = h @ w[i].T + b
        zs.append(z)
        h = z if i == len(params) - 1 else bf16(0.5 * z * (1 + erf(z / np.sqrt(2))))
        hs.append(h)
    loss, dz = omlp.mse(h, target)
    grads = []
    for i in reversed(range(len(params))):
        d16 = bf16(dz) if i else dz
        grads.append((d16.T @ hs[i], dz.sum(0)))
        if i:
            z = zs[i - 1]
            dz = (d16 @ w[i]) * (0.5 * (1 + erf(z / np.sqrt(2)))
                                 + z * np.exp(-z * z / 2) / np.sqrt(2 * np.pi))
    return h, loss, grads[::-1]


# One rounding to BF16 is off by at most 2^-9 of the value.  Against a
# reference that rounds at the same places only values within FP32 rounding of
# a tie differ, so 2^-9 relative holds with room for every layer's flips; a
# gradient passes twice as many roundings.
FWD, GRAD = 2.0 ** -9, 2.0 ** -8


@pytest.mark.parametrize("width,depth,out_side,rows", [
    (64, 1, 8, 1), (64, 3, 16, 63), (192, 2, 8, 64), (128, 2, 16, 65), (256, 1, 32, 130),
    (320, 2, 8, 191), (512, 2, 32, 1100), (192, 3, 32, 2100)])
def test_products_at_the_edges_of_their_tiles(width, depth, out_side, rows):
    import torch
    need_gpu()
    p, _, _, y, _ = small_problem(width=width, depth=depth, out_side=out_side)
    rng = np.random.default_rng(width + rows)
    phi = inputs.box_draws(rows, LO, HI, seed=rows)
    dphi = torch.tensor(phi, device="cuda")
    target = rng.standard_normal((rows, out_side ** 2)).astype(np.float32)
    before = host_params(p)
    want, want_loss, want_grads = reference(before, omlp.scale_inputs(phi, LO, HI),
                                            target.astype(np.float64))

    out = p.surrogate_forward(dphi, raw=True).cpu().numpy()
    assert rel_l2(out, want) < FWD

    mean = rng.uniform(0.5, 1.5, out_side ** 2).astype(np.float32)
    sd = rng.uniform(0.1, 0.3, out_side ** 2).astype(np.float32)
    p.surrogate_set_scaling(torch.tensor(mean, device="cuda"), torch.tensor(sd, device="cuda"),
                            0.07)
    ll = p.surrogate_loglik(dphi).cpu().numpy()
    ybar = omlp.block_mean(y, out_side).ravel()
    want_ll = 0.5 * ((ybar - (mean + sd * out.astype(np.float64))) ** 2).sum(1) / 0.07 ** 2
    assert np.allclose(ll, want_ll, rtol=1e-5)  # FP32 epilogue on the same outputs

    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    p.surrogate_train_step(dphi, torch.tensor(target, device="cuda"), 1e-3, loss)
    torch.cuda.synchronize()
    assert loss.item() == pytest.approx(want_loss, rel=FWD)
    grads, after = host_params(p, dir=2), host_params(p)
    for (gW, gb), (wW, wb) in zip(grads, want_grads):
        assert rel_l2(gW, wW) < GRAD and rel_l2(gb, wb) < GRAD
    for (aW, ab), (wW, wb) in zip(after, omlp.adam_step(before, grads, {}, lr=1e-3)):
        # a first step moves every weight by at most the rate; FP32 arithmetic
        assert np.abs(aW - wW).max() < 2e-6 and np.abs(ab - wb).max() < 2e-6
    # the BF16 copies follow the weights
    out2 = p.surrogate_forward(dphi, raw=True).cpu().numpy()
    want2 = reference(after, omlp.scale_inputs(phi, LO, HI), target.astype(np.float64))[0]
    assert rel_l2(out2, want2) < FWD
    p.close()
