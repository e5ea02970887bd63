"""conv1 of bf16 batches at the edges of its kernels: observations shared by 16, 3, 2 and 1 workgroups (each with the image
rows under its position tiles only; 4x84x84 frames take the kernels of conv1 and conv2 by now), first and last batch of each, against the kernels that serve other batch sizes, bit
for bit; the gradient of small bf16 minibatches, whose weight gradients take the large batches' kernels; and the knob that
sends them to the wave-per-segment ones."""
import numpy as np
import pytest
import torch

import hts_synth as syn
from test_gpu_parity import ATARI, FOOT, _act, _rollout, _split, dev, hts  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,A,sizes", [(FOOT, 19, (20, 21, 64, 85, 86, 127, 128, 129, 255)), (ATARI, 18, (63, 64, 85, 86, 128, 129, 255))])
def test_shared_observations_agree_bitwise(hts, shape, A, sizes, monkeypatch):  # noqa: F811
    n = max(sizes)
    params = dev(syn.init_params(21, *shape, A, bias_scale=0.05))
    obs = dev(syn.obs_football(23, 1, n)[0] if shape == FOOT else syn.obs_atari(23, 1, n)[0])
    monkeypatch.setenv("HTS_CONV1_SLAB_ROWS", "100000000")
    ctx = hts.Context(*shape, A, precision=1, max_act_batch=n)
    want = _act(ctx, obs, params, 5, 1, 0, A)
    ctx.close()
    monkeypatch.delenv("HTS_CONV1_SLAB_ROWS")
    ctx = hts.Context(*shape, A, precision=1, max_act_batch=n)
    for k in sizes:
        got = _act(ctx, obs[n - k:].contiguous(), params, 5, 1, n - k, A)
        assert all(np.array_equal(x[n - k:], y) for x, y in zip(want, got)), k
    ctx.close()


# Twice the rows, half the weight of each: a power of two, so every bfloat16 rounding of the backward pass is the same up to the
# exponent, and the gradient over 2 B rows is the mean of the gradients over its halves up to the order of binary32 sums of at
# most n = 128 * 400 terms (sqrt(n) 2^-24 = 1.4e-5).  32 and 64 rows take different conv1 kernels.
@pytest.mark.parametrize("shape,A,B", [(ATARI, 18, 32), (FOOT, 19, 32), (ATARI, 18, 64), ((3, 44, 52), 7, 64)])
def test_small_bf16_minibatch_gradient_is_the_mean_of_its_halves(hts, oracle, shape, A, B):  # noqa: F811
    _, params, obs, actions, old_logp, adv, ret = _rollout(oracle, shape, A, 2 * B, 700 + B, False)
    ctx = hts.Context(*shape, A, precision=1, max_learn_batch=2 * B)

    def gradient(lo, hi):
        g = torch.full((ctx.P,), float("nan"), device="cuda")
        rows = [dev(x[lo:hi]) for x in (obs, actions, adv, ret)]
        ctx.hts_loss_and_grads(rows[0], rows[1], None, rows[2], rows[3], dev(params), hts.HParams(algo=hts.ALGO_A2C), g)
        torch.cuda.synchronize()
        return _split(g.cpu().numpy().astype(np.float64), shape, A)

    whole, first, second = gradient(0, 2 * B), gradient(0, B), gradient(B, 2 * B)
    for name, w in whole.items():
        mean = 0.5 * (first[name] + second[name])
        assert np.linalg.norm(w - mean) <= 1.4e-5 * np.linalg.norm(mean), name
    ctx.close()


# HTS_SMALL_BATCH asks for the wave-per-segment kernels in every layer that has them.  Up to 32 rows that is the default; at 40 rows
# of bf16 conv1's weight gradient takes the image kernel by itself: the same products added in another order (binary32 sums of
# n = 40 * 400 terms, sqrt(n) 2^-24 = 7.6e-6), so some bits must differ, and every other tensor is the same bit for bit.
@pytest.mark.parametrize("B", [32, 40])
def test_small_batch_knob_covers_conv1(hts, oracle, B, monkeypatch):  # noqa: F811
    _, params, obs, actions, _, adv, ret = _rollout(oracle, ATARI, 18, B, 800 + B, False)
    grads = []
    for knob in (None, "128"):
        monkeypatch.delenv("HTS_SMALL_BATCH", raising=False) if knob is None else monkeypatch.setenv("HTS_SMALL_BATCH", knob)
        ctx = hts.Context(*ATARI, 18, precision=1, max_learn_batch=B)
        g = torch.full((ctx.P,), float("nan"), device="cuda")
        ctx.hts_loss_and_grads(dev(obs), dev(actions), None, dev(adv), dev(ret), dev(params), hts.HParams(algo=hts.ALGO_A2C), g)
        torch.cuda.synchronize()
        grads.append(_split(g.cpu().numpy(), ATARI, 18))
        ctx.close()
    default, forced = grads
    for name, w in default.items():
        same = np.array_equal(w, forced[name])
        assert same or (B == 40 and name in ("conv1.w", "conv1.b")), name
        assert np.linalg.norm(w.astype(np.float64) - forced[name]) <= 7.6e-6 * np.linalg.norm(w), name
    assert np.array_equal(default["conv1.w"], forced["conv1.w"]) == (B == 32)
