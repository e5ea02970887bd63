"""conv3 of large bf16 batches with weights in registers: rows of a batch that takes it against the same rows of a batch of another size, whose conv3 runs
on another kernel or in other groups, bit for bit (one sample a compute unit, two at a time, an odd last group, sizes around the cuts); the
learner's two copies of its output by the gradients, against those of the wave-per-segment forward kernels."""
import numpy as np
import pytest
import torch

import hts_synth as syn
from test_gpu_parity import ATARI, _act, dev, hts  # noqa: F401

pytestmark = pytest.mark.gpu
FOOTBALL = (16, 72, 96)


def _frames(shape, n, seed):
    return torch.randint(0, 256, (n, *shape), device="cuda", generator=torch.Generator(device="cuda").manual_seed(seed), dtype=torch.uint8)


@pytest.mark.parametrize("shape", [ATARI, FOOTBALL])
def test_actor_calls_agree_bitwise(hts, shape):  # noqa: F811
    n, A = 1551, 19
    params, obs = dev(syn.init_params(71, *shape, A, bias_scale=0.05)), _frames(shape, n, 72)
    ctx = hts.Context(*shape, A, precision=1, max_act_batch=n)
    want = [np.concatenate(x) for x in zip(*(_act(ctx, obs[i:i + 128].contiguous(), params, 5, 1, i, A) for i in range(0, n, 128)))]
    for k in (129, 255, 256, 257, 300, 511, 512, 513, 1535, 1536, 1551):
        got = _act(ctx, obs[n - k:].contiguous(), params, 5, 1, n - k, A)
        assert all(np.array_equal(x[n - k:], y) for x, y in zip(want, got)), k
    ctx.close()


# A sum of B terms in another order differs by no more than about B / 2 roundings of 2^-24 of its terms' size, here far below 1e-4 of a gradient; a mask or an
# activation of another row changes a gradient by its own size
@pytest.mark.parametrize("shape, B", [(ATARI, 131), (ATARI, 257), (FOOTBALL, 130), (FOOTBALL, 301)])
def test_gradients(hts, shape, B, monkeypatch):  # noqa: F811
    A = 6
    g = torch.Generator(device="cuda").manual_seed(B)
    params, obs = dev(syn.init_params(73, *shape, A, bias_scale=0.05)), _frames(shape, B, 74)
    actions = torch.randint(0, A, (B,), device="cuda", generator=g, dtype=torch.int32)
    adv, ret = torch.randn(B, device="cuda", generator=g), torch.randn(B, device="cuda", generator=g)
    grads = []
    for small in ("1000", None):
        monkeypatch.setenv("HTS_SMALL_BATCH", small) if small else monkeypatch.delenv("HTS_SMALL_BATCH")
        ctx = hts.Context(*shape, A, precision=1, max_learn_batch=B)
        out = torch.full((ctx.P,), float("nan"), device="cuda")
        ctx.hts_loss_and_grads(obs, actions, None, adv, ret, params, hts.HParams(algo=hts.ALGO_A2C), out)
        torch.cuda.synchronize()
        grads.append(out.double())
        ctx.close()
    assert bool(torch.isfinite(grads[1]).all())
    assert float((grads[1] - grads[0]).norm() / grads[0].norm()) < 1e-4
