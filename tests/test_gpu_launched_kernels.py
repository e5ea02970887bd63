"""Kernels that few of the package's shapes and sizes reach, each by a call that is seen to launch it (read from a captured graph), bit for bit against
another kernel of the same layers: conv1 and conv2 in one kernel on frames at a multiple of 8 bytes but not of 16 and with workgroups that hold as many
row indices as fit; conv2 with weights in registers, which 4x84x84 frames reach at a multiple of 4 bytes only, whole device and compute-unit ranges; the
stages of conv2's LDS-copy tiles; conv3 with weights in registers over many groups a workgroup, in the form that keeps both orders for the learner."""
import contextlib

import pytest
import torch

import hts_synth as syn
from launches import launches
from test_gpu_parity import ATARI, FOOT, dev, hts  # noqa: F401

pytestmark = pytest.mark.gpu
GREY3 = (3, 84, 84)              # the grids of 4x84x84 frames, conv1 and conv2 in kernels of their own
OFF = "100000000"


def _frames(shape, n, seed, shift=0):
    """u8 frames, the first of them `shift` bytes behind a multiple of 16."""
    size = n * shape[0] * shape[1] * shape[2]
    room = torch.empty(size + 16, dtype=torch.uint8, device="cuda")
    obs = room[shift:shift + size].view(n, *shape)
    obs.copy_(torch.randint(0, 256, (n, *shape), device="cuda", generator=torch.Generator(device="cuda").manual_seed(seed), dtype=torch.uint8))
    assert obs.data_ptr() % 16 == shift
    return obs


@contextlib.contextmanager
def _stream(hts, cus):  # noqa: F811
    """A stream, of `cus` compute units if given."""
    rng = hts.CuRangeStream(8, cus) if cus else None
    try:
        yield rng.stream if rng else torch.cuda.Stream()
    finally:
        torch.cuda.synchronize()
        if rng:
            rng.close()


def _act(ctx, obs, A):
    """Actor call: a function that enqueues it, and its outputs."""
    n = obs.shape[0]
    out = [torch.full((n,), -1, dtype=torch.int32, device="cuda"), torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda"), torch.zeros(n, A, device="cuda")]
    return lambda: ctx.hts_act(obs, None, 5, 1, 0, *out), out


def _gradient(hts, ctx, obs, A, seed, params, index, B):  # noqa: F811
    """The same for the loss and its gradient."""
    g, n = torch.Generator(device="cuda").manual_seed(seed), obs.shape[0]
    actions = torch.randint(0, A, (n,), device="cuda", generator=g, dtype=torch.int32)
    adv, ret = torch.randn(n, device="cuda", generator=g), torch.randn(n, device="cuda", generator=g)
    out, hp = torch.full((ctx.P,), float("nan"), device="cuda"), hts.HParams(algo=hts.ALGO_A2C)
    return lambda: ctx.hts_loss_and_grads(obs, actions, None, adv, ret, params, hp, out, index=index, B=B), [out]


def _run(call, out, stream, kernel):
    """The outputs of call(), which launches one `kernel`, and that launch: its name and workgroups."""
    found = [x[:2] for x in launches(call, stream) if kernel in x[0]]
    assert len(found) == 1, (kernel, found)
    torch.cuda.synchronize()
    call()
    torch.cuda.synchronize()
    return [x.clone() for x in out], found[0]


def _acts(hts, shape, obs, A, params, kernel, cus=None):  # noqa: F811
    with _stream(hts, cus) as stream:
        ctx = hts.Context(*shape, A, precision=1, max_act_batch=obs.shape[0], stream=stream)
        torch.cuda.synchronize()
        ctx.hts_sync_params(params)
        result = _run(*_act(ctx, obs, A), stream, kernel)
        ctx.close()
    return result


def _grads(hts, shape, obs, A, params, kernel, cus=None, index=None):  # noqa: F811
    B = obs.shape[0] if index is None else index.numel()
    with _stream(hts, cus) as stream:
        ctx = hts.Context(*shape, A, precision=1, max_learn_batch=B, stream=stream)
        result = _run(*_gradient(hts, ctx, obs, A, 7, params, index, B), stream, kernel)
        ctx.close()
    assert bool(torch.isfinite(result[0][0]).all())
    return result


def _same(got, want):
    return all(torch.equal(x, y) for x, y in zip(got, want))


# ---- conv1 and conv2 in one kernel ----
# 300 rows: one or two samples a workgroup; 521: two or three.  4 bytes: the kernels of other frames
@pytest.mark.parametrize("n", [300, 521])
def test_conv12_frames_at_a_multiple_of_eight_bytes(hts, n):  # noqa: F811
    A = 6
    params, obs, shifted, other = dev(syn.init_params(81, *ATARI, A, bias_scale=0.05)), _frames(ATARI, n, 82), _frames(ATARI, n, 82, 8), _frames(ATARI, n, 82, 4)
    want, _ = _acts(hts, ATARI, other, A, params, "conv1_image_kernel")
    for x in (obs, shifted):
        assert _same(_acts(hts, ATARI, x, A, params, "conv12_kernelILb0E")[0], want)


def test_conv12_learner_frames_at_a_multiple_of_eight_bytes(hts, monkeypatch):  # noqa: F811
    A, n, B = 6, 330, 301
    params = dev(syn.init_params(83, *ATARI, A, bias_scale=0.05))
    index = torch.randperm(n, device="cuda", generator=torch.Generator(device="cuda").manual_seed(84))[:B].to(torch.int32)
    for shift in (0, 8):
        obs = _frames(ATARI, n, 85, shift)
        got, _ = _grads(hts, ATARI, obs, A, params, "conv12_kernelILb1E", index=index)
        monkeypatch.setenv("HTS_CONV1_SLAB_ROWS", OFF)
        want, _ = _grads(hts, ATARI, obs, A, params, "conv1_image_kernel", index=index)
        monkeypatch.delenv("HTS_CONV1_SLAB_ROWS")
        assert _same(got, want), shift


# 8 compute units: 512 rows are 64 a workgroup, as many as it holds indices of; more rows take more workgroups, 640 ten of 64, 513 nine of 57
@pytest.mark.parametrize("n, workgroups", [(512, 8), (513, 9), (640, 10)])
def test_conv12_rows_of_a_workgroup(hts, n, workgroups):  # noqa: F811
    A = 6
    params, obs = dev(syn.init_params(86, *ATARI, A, bias_scale=0.05)), _frames(ATARI, n, 87)
    want, _ = _acts(hts, ATARI, obs, A, params, "conv12_kernel")
    got, at = _acts(hts, ATARI, obs, A, params, "conv12_kernel", 8)
    assert at[1] == workgroups and _same(got, want)


# around the sizes where actor calls go from the kernel of few rows to this one: whole device, 80 rows; without that kernel, 48
@pytest.mark.parametrize("knob, cut, below", [(None, 81, "conv12_rows_kernel"), ("0", 48, "Conv1Fwd")])
def test_conv12_first_actor_rows(hts, knob, cut, below, monkeypatch):  # noqa: F811
    A = 6
    params, obs = dev(syn.init_params(88, *ATARI, A, bias_scale=0.05)), _frames(ATARI, cut, 89)
    if knob:
        monkeypatch.setenv("HTS_CONV12_ROWS_KERNEL", knob)
    fewer, _ = _acts(hts, ATARI, obs[:-1], A, params, below)
    got, _ = _acts(hts, ATARI, obs, A, params, "conv12_kernelILb0E")
    assert _same([x[:-1] for x in got], fewer)


# ---- conv2 with weights in registers ----
@pytest.mark.parametrize("shape, shift, sizes", [(GREY3, 0, (2048, 2049, 2561)), (ATARI, 4, (2048, 2049)), (FOOT, 0, (3072, 3075))])
def test_conv2_in_registers(hts, shape, shift, sizes):  # noqa: F811
    A, n = 6, max(sizes)
    params, obs = dev(syn.init_params(91, *shape, A, bias_scale=0.05)), _frames(shape, n, 92, shift)
    less = min(sizes) - 1                                       # the first size that takes the LDS-copy kernel
    want, _ = _acts(hts, shape, obs[:less], A, params, "ConvFwd")
    for k in sizes:
        got, _ = _acts(hts, shape, obs[:k], A, params, "14regconv_kernel")
        assert _same([x[:less] for x in got], want), k


# As many workgroups as the stream has compute units: other shares of the batch, the same bits
@pytest.mark.parametrize("shape, n", [(GREY3, 2305), (FOOT, 3075)])
def test_conv2_in_registers_on_ranges(hts, shape, n):  # noqa: F811
    A = 6
    params, obs = dev(syn.init_params(93, *shape, A, bias_scale=0.05)), _frames(shape, n, 94)
    want, _ = _acts(hts, shape, obs, A, params, "14regconv_kernel")
    for cus in (192, 40):
        got, at = _acts(hts, shape, obs, A, params, "14regconv_kernel", cus)
        assert at[1] == cus and _same(got, want), cus


# ---- conv2 on LDS copies: 512 workgroups of 128x64 at 809 rows and three stages, 513 at 810 and two ----
def test_conv2_stages(hts):  # noqa: F811
    A = 6
    params, obs = dev(syn.init_params(95, *GREY3, A, bias_scale=0.05)), _frames(GREY3, 810, 96)
    fewer, three = _acts(hts, GREY3, obs[:-1], A, params, "ConvFwd")
    got, two = _acts(hts, GREY3, obs, A, params, "ConvFwd")
    assert "Li128ELi64ELi2ELi2ELi3E" in three[0] and "Li128ELi64ELi2ELi2ELi2E" in two[0]
    assert _same([x[:-1] for x in got], fewer)
    whole, _ = _acts(hts, GREY3, obs[:128].contiguous(), A, params, "ConvFwdIDF16bNS_9ConvLayerILi32E")
    assert _same([x[:128] for x in got], whole)


# ---- conv3 with weights in registers, learner: eight compute units, two samples a group, eight to nineteen groups a workgroup, the last one short ----
@pytest.mark.parametrize("shape, B", [(ATARI, 131), (ATARI, 301), (FOOT, 130), (FOOT, 257)])
def test_conv3_learner_groups(hts, shape, B):  # noqa: F811
    A = 6
    params, obs = dev(syn.init_params(97, *shape, A, bias_scale=0.05)), _frames(shape, B, 98)
    want, _ = _grads(hts, shape, obs, A, params, "conv3_regconv_kernel")
    got, at = _grads(hts, shape, obs, A, params, "conv3_regconv_kernel", 8)
    assert at[1] == 8 and _same(got, want)
