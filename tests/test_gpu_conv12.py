"""conv1 and conv2 of bf16 batches of 4x84x84 frames in one kernel, against a launch each, bit for bit: one to five samples per workgroup, the
last ones on some workgroups only; frames gathered by index and conv1's output kept for the backward pass; compute-unit ranges, of more
samples than their units' workgroups hold row indices of; few frames at a multiple of 8 bytes but not of 16 (in the kernel of few rows: for this
one see test_gpu_launched_kernels.py); the learner's first rows."""
import numpy as np
import pytest
import torch

import hts_synth as syn
from launches import launches
from test_gpu_parity import ATARI, _act, dev, hts  # noqa: F401

pytestmark = pytest.mark.gpu
OFF, ON = "100000000", "1"


def _frames(n, seed):
    return torch.randint(0, 256, (n, *ATARI), device="cuda", generator=torch.Generator(device="cuda").manual_seed(seed), dtype=torch.uint8)


def test_actor_calls_agree_bitwise(hts, monkeypatch):  # noqa: F811
    n, A = 1030, 18
    params, obs = dev(syn.init_params(51, *ATARI, A, bias_scale=0.05)), _frames(n, 52)
    monkeypatch.setenv("HTS_CONV1_SLAB_ROWS", OFF)
    ctx = hts.Context(*ATARI, A, precision=1, max_act_batch=n)
    want = _act(ctx, obs, params, 5, 1, 0, A)
    ctx.close()
    for knob, sizes in ((ON, (1, 2, 255, 257, 512, 769, 1030)), (None, (47, 48))):
        monkeypatch.setenv("HTS_CONV1_SLAB_ROWS", knob) if knob else monkeypatch.delenv("HTS_CONV1_SLAB_ROWS")
        ctx = hts.Context(*ATARI, A, precision=1, max_act_batch=n)
        for k in sizes:
            got = _act(ctx, obs[n - k:].contiguous(), params, 5, 1, n - k, A)
            assert all(np.array_equal(x[n - k:], y) for x, y in zip(want, got)), k
        ctx.close()


def test_frames_at_a_multiple_of_eight_bytes(hts):  # noqa: F811
    n, A = 70, 6
    params, obs = dev(syn.init_params(53, *ATARI, A, bias_scale=0.05)), _frames(n, 54)
    ctx = hts.Context(*ATARI, A, precision=1, max_act_batch=n)
    want = _act(ctx, obs, params, 5, 1, 0, A)
    for shift in (8, 4):                                        # 4: the kernels of other frames
        room = torch.empty(obs.numel() + 16, dtype=torch.uint8, device="cuda")
        shifted = room[shift:shift + obs.numel()].view(obs.shape).copy_(obs)
        assert shifted.data_ptr() % 16 == shift
        assert all(np.array_equal(x, y) for x, y in zip(want, _act(ctx, shifted, params, 5, 1, 0, A))), shift
    ctx.close()


@pytest.mark.parametrize("B", [48, 300, 521])
def test_gradients_agree_bitwise(hts, B, monkeypatch):  # noqa: F811
    A, count = 18, 2 * B
    g = torch.Generator(device="cuda").manual_seed(B)
    params, obs = dev(syn.init_params(55, *ATARI, A, bias_scale=0.05)), _frames(count, 56)
    index = torch.randperm(count, device="cuda", generator=g)[:B].to(torch.int32)
    actions = torch.randint(0, A, (count,), device="cuda", generator=g, dtype=torch.int32)
    adv, ret = torch.randn(count, device="cuda", generator=g), torch.randn(count, device="cuda", generator=g)
    grads = []
    for knob in (OFF, ON):
        monkeypatch.setenv("HTS_CONV1_SLAB_ROWS", knob)
        ctx = hts.Context(*ATARI, A, precision=1, max_learn_batch=B)
        out = torch.full((ctx.P,), float("nan"), device="cuda")
        ctx.hts_loss_and_grads(obs, actions, None, adv, ret, params, hts.HParams(algo=hts.ALGO_A2C), out, index=index)
        torch.cuda.synchronize()
        grads.append(out)
        ctx.close()
    assert bool(torch.isfinite(grads[0]).all()) and torch.equal(*grads)


# 8 compute units and 600 rows would be 75 samples for each, more than a workgroup's 64: ten workgroups of 60
def test_few_compute_units(hts):  # noqa: F811
    n, A = 600, 18
    params, obs = dev(syn.init_params(57, *ATARI, A, bias_scale=0.05)), _frames(n, 58)
    ctx = hts.Context(*ATARI, A, precision=1, max_act_batch=n)
    want = _act(ctx, obs, params, 5, 1, 0, A)
    ctx.close()
    rng = hts.CuRangeStream(16, 8)
    ctx = hts.Context(*ATARI, A, precision=1, max_act_batch=n, stream=rng.stream)
    out = [torch.zeros(n, dtype=torch.int32, device="cuda"), torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda"), torch.zeros(n, A, device="cuda")]
    torch.cuda.synchronize()                      # what fills them runs on another stream
    ctx.hts_act(obs, params, 5, 1, 0, *out)
    torch.cuda.synchronize()
    ctx.close()
    rng.close()
    assert all(np.array_equal(x, y.cpu().numpy()) for x, y in zip(want, out))


# the learner's cut, by what an update launches: below it, one that was taken for the actor's made updates slower
@pytest.mark.parametrize("cus, cut", [(None, 64), (96, 48)])
def test_the_learners_cut(hts, cus, cut):  # noqa: F811
    rng = hts.CuRangeStream(0, cus) if cus else None
    stream, n, A = rng.stream if cus else torch.cuda.Stream(), 64, 18
    ctx = hts.Context(*ATARI, A, precision=1, max_learn_batch=n, stream=stream)
    params, obs, rows = dev(syn.init_params(59, *ATARI, A)), _frames(n, 60), torch.zeros(n, device="cuda")
    actions, out = torch.zeros(n, dtype=torch.int32, device="cuda"), torch.zeros(ctx.P, device="cuda")
    for B in (cut - 1, cut):
        call = lambda: ctx.hts_loss_and_grads(obs[:B], actions[:B], None, rows[:B], rows[:B], params, hts.HParams(algo=hts.ALGO_A2C), out)
        names = [x[0] for x in launches(call, stream)]
        assert [x for x in names if "conv1" in x] and any("conv12_kernel" in x for x in names) == (B == cut), (B, names)
    torch.cuda.synchronize()
    ctx.close()
    if rng:
        rng.close()
