"""conv1 and conv2, or all three conv layers, of bf16 actor calls of few frames in one kernel, a workgroup for some rows, against a launch for each
layer, bit for bit: sizes around the cuts between them and the other kernels, samples that do not fill the eight XCDs; parameters
that an update has just changed; frames at a multiple of 8 bytes but not of 16, and of 4."""
import numpy as np
import pytest
import torch

import hts_synth as syn
from test_gpu_parity import ATARI, _act, dev, hts  # noqa: F401

pytestmark = pytest.mark.gpu
FOOTBALL = (16, 72, 96)


def _frames(shape, n, seed):
    return torch.randint(0, 256, (n, *shape), device="cuda", generator=torch.Generator(device="cuda").manual_seed(seed), dtype=torch.uint8)


@pytest.mark.parametrize("shape, sizes", [(ATARI, (1, 7, 8, 9, 25, 32, 33, 47, 80, 81)), (FOOTBALL, (1, 5, 8, 9, 16, 17))])
def test_actor_calls_agree_bitwise(hts, shape, sizes, monkeypatch):  # noqa: F811
    n, A = max(sizes), 19
    params, obs = dev(syn.init_params(61, *shape, A, bias_scale=0.05)), _frames(shape, n, 62)
    monkeypatch.setenv("HTS_CONV12_ROWS_KERNEL", "0")
    separate = hts.Context(*shape, A, precision=1, max_act_batch=n)
    monkeypatch.delenv("HTS_CONV12_ROWS_KERNEL")
    ctx = hts.Context(*shape, A, precision=1, max_act_batch=n)
    for k in sizes:
        part = obs[n - k:].contiguous()
        want, got = _act(separate, part, params, 5, 1, 0, A), _act(ctx, part, params, 5, 1, 0, A)
        assert all(np.array_equal(x, y) for x, y in zip(want, got)), k
    separate.close()
    ctx.close()


@pytest.mark.parametrize("shape", [ATARI, FOOTBALL])
def test_frames_at_other_addresses(hts, shape):  # noqa: F811
    n, A = 9, 6
    params, obs = dev(syn.init_params(63, *shape, A, bias_scale=0.05)), _frames(shape, n, 64)
    ctx = hts.Context(*shape, A, precision=1, max_act_batch=n)
    want = _act(ctx, obs, params, 5, 1, 0, A)
    for shift in (8, 4):                                        # 4: the kernels of other frames
        room = torch.empty(obs.numel() + 16, dtype=torch.uint8, device="cuda")
        shifted = room[shift:shift + obs.numel()].view(obs.shape).copy_(obs)
        assert shifted.data_ptr() % 16 == shift
        assert all(np.array_equal(x, y) for x, y in zip(want, _act(ctx, shifted, params, 5, 1, 0, A))), shift
    ctx.close()


# the optimiser's kernel rewrites the copies of the network itself: an actor call behind an update reads what a fresh context would
@pytest.mark.parametrize("shape", [ATARI, FOOTBALL])
def test_weights_after_an_update(hts, shape):  # noqa: F811
    n, A = 9, 6
    params, obs = dev(syn.init_params(65, *shape, A, bias_scale=0.05)), _frames(shape, n, 66)
    g = torch.Generator(device="cuda").manual_seed(67)
    ctx = hts.Context(*shape, A, precision=1, max_act_batch=n, max_learn_batch=n)
    ctx.hts_track_params(True)
    before = _act(ctx, obs, params, 5, 1, 0, A)
    opt = hts.OptState(torch.zeros_like(params), torch.zeros_like(params), 0)
    ctx.hts_learner_step(obs, torch.randint(0, A, (n,), device="cuda", generator=g, dtype=torch.int32), torch.zeros(n, device="cuda"),
                         torch.randn(n, device="cuda", generator=g), torch.randn(n, device="cuda", generator=g), params, opt,
                         hts.HParams(algo=hts.ALGO_A2C, lr=1e-2))
    got = _act(ctx, obs, params, 5, 1, 0, A)
    fresh = hts.Context(*shape, A, precision=1, max_act_batch=n)
    want = _act(fresh, obs, params, 5, 1, 0, A)
    assert all(np.array_equal(x, y) for x, y in zip(want, got)) and not np.array_equal(before[3], got[3])
    ctx.close()
    fresh.close()
