"""bfloat16 weight gradients whose k-tiles are copied into LDS: a minibatch against its two halves, whose reductions end elsewhere."""
import numpy as np
import pytest
import torch

from test_gpu_parity import ATARI, FOOT, _rollout, _split, dev, hts  # noqa: F811,F401

pytestmark = pytest.mark.gpu


# One sample and less than a k-tile of 64 (FC: 1, 3, 35), whole k-tiles (64), ragged ends of chunks and k-tiles; an odd number of
# 64-column halves of FC (3x44x52: 4; 2x36x36: 1).  The loss is a mean, so the rows' gradients of a half are exactly twice those in the
# whole; the sums are binary32 in another order, and a layer's input gradient that ends near a rounding edge of bfloat16 (2^-9) may fall
# on either side where the two sizes run different kernels.
@pytest.mark.parametrize("shape,A,half", [((2, 36, 36), 5, 1), ((3, 44, 52), 7, 3), ((3, 44, 52), 7, 64), (ATARI, 18, 35), (FOOT, 19, 65)])
def test_halves_add_up(hts, oracle, shape, A, half):  # noqa: F811
    B = 2 * half
    _, params, obs, actions, _, adv, ret = _rollout(oracle, shape, A, B, 970 + B, False)

    def grad(lo, hi):
        ctx = hts.Context(*shape, A, precision=1, max_learn_batch=hi - lo)
        g = torch.full((ctx.P,), float("nan"), device="cuda")
        ctx.hts_loss_and_grads(dev(obs[lo:hi]), dev(actions[lo:hi]), None, dev(adv[lo:hi]), dev(ret[lo:hi]), dev(params),
                               hts.HParams(algo=hts.ALGO_A2C), g)
        torch.cuda.synchronize()
        out = _split(g.cpu().numpy().astype(np.float64), shape, A)
        ctx.close()
        return out

    whole, a, b = grad(0, B), grad(0, half), grad(half, B)
    for name, w in whole.items():
        assert np.linalg.norm(w - (a[name] + b[name]) / 2) <= 2e-3 * np.linalg.norm(w), name
