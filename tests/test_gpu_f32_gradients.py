"""binary32 backward kernels: gradients at the edges of their tiles, and
over operands whose magnitudes spread over many binades, against the oracle's float64 gradient."""
import numpy as np
import pytest
import torch

import hts_synth as syn
from test_gpu_parity import ATARI, _rollout, _split, dev, hts, oracle_hp  # noqa: F401

pytestmark = pytest.mark.gpu


# 128 / 129 rows: last of the wave-per-segment, first of the tile kernels; 65 = one row more than a 64-row tile; 3x44x52 and
# 2x36x36 frames have feature counts that end inside a tile, and conv1 columns that end inside one beside the bias column.  A
# sum of n products of binary32 numbers in binary32 is off by about sqrt(n) 2^-24 of its size: n is at most B * P1 = 129 * 120
# (3x44x52) or 97 * 400 positions, so 1.2e-5.  Rows of `adv` scaled over 2^-20 .. 2^20 leave the gradient to a few rows.
@pytest.mark.parametrize("shape,A,B,spread", [((3, 44, 52), 7, 65, 0), ((3, 44, 52), 7, 96, 20), ((3, 44, 52), 7, 97, 20), ((3, 44, 52), 7, 129, 20),
                                              ((2, 36, 36), 5, 129, 0), (ATARI, 18, 97, 0)])
def test_f32_gradient(hts, oracle, shape, A, B, spread):  # noqa: F811
    Cc, H, W = shape
    net, params, obs, actions, old_logp, adv, ret = _rollout(oracle, shape, A, B, 300 + B, False)
    adv = (adv * 2.0 ** np.linspace(-spread, spread, B)).astype(np.float32)
    ctx = hts.Context(Cc, H, W, A, max_learn_batch=B)
    hp = hts.HParams(algo=hts.ALGO_A2C)
    grads = torch.full((ctx.P,), float("nan"), device="cuda")
    ctx.hts_loss_and_grads(dev(obs), dev(actions), None, dev(adv), dev(ret), dev(params), hp, grads)
    torch.cuda.synchronize()
    want, _ = oracle.loss_grads(net, params, obs, actions, old_logp, adv, ret, oracle_hp(oracle, hp), threads=oracle.host_threads())
    got = grads.cpu().numpy().astype(np.float64)
    for name, w in _split(want, shape, A).items():
        err = np.linalg.norm(_split(got, shape, A)[name] - w) / np.linalg.norm(w)
        assert err <= 1.2e-5, (name, err)
    ctx.close()
