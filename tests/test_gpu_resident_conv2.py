"""conv2 of large bf16 batches, its weights in registers and its samples in LDS: on either side of its first sizes, with an odd sample
at the end and with unequal numbers of groups per workgroup, against the wave-per-segment kernels bit for bit.  (4x84x84 frames take conv1 and
conv2 in one kernel by now: their sizes here are that one's, and other frames of their grids are in test_gpu_launched_kernels.py.)"""
import numpy as np
import pytest
import torch

from test_gpu_parity import ATARI, FOOT, _act, dev, hts  # noqa: F401
import hts_synth as syn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,A,sizes", [(ATARI, 18, (2047, 2048, 2049, 2561)), (FOOT, 19, (3071, 3072, 3075))])
def test_rows_agree_bitwise(hts, shape, A, sizes, monkeypatch):  # noqa: F811
    n = max(sizes)
    params = dev(syn.init_params(41, *shape, A, bias_scale=0.05))
    g = torch.Generator(device="cuda").manual_seed(42)
    obs = torch.randint(0, 256, (n, *shape), device="cuda", generator=g, dtype=torch.uint8)
    monkeypatch.setenv("HTS_SMALL_BATCH", "1000000")
    ctx = hts.Context(*shape, A, precision=1, max_act_batch=n)
    want = _act(ctx, obs, params, 5, 1, 0, A)
    ctx.close()
    monkeypatch.delenv("HTS_SMALL_BATCH")
    ctx = hts.Context(*shape, A, precision=1, max_act_batch=n)
    for k in sizes:
        got = _act(ctx, obs[n - k:].contiguous(), params, 5, 1, n - k, A)
        assert all(np.array_equal(x[n - k:], y) for x, y in zip(want, got)), k
    ctx.close()


# As many workgroups as the stream has compute units: other shares of the batch, the same bits.
@pytest.mark.parametrize("cus", [192, 40])
def test_compute_unit_ranges_agree_bitwise(hts, cus):  # noqa: F811
    n, A = 2305, 18
    params = dev(syn.init_params(43, *ATARI, A, bias_scale=0.05))
    obs = torch.randint(0, 256, (n, *ATARI), device="cuda", generator=torch.Generator(device="cuda").manual_seed(44), dtype=torch.uint8)
    ctx = hts.Context(*ATARI, A, precision=1, max_act_batch=n)
    want = _act(ctx, obs, params, 5, 1, 0, A)
    ctx.close()
    rng = hts.CuRangeStream(8, cus)
    ctx = hts.Context(*ATARI, A, precision=1, max_act_batch=n, stream=rng.stream)
    out = [torch.zeros(n, dtype=torch.int32, device="cuda"), torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda"), torch.zeros(n, A, device="cuda")]
    torch.cuda.synchronize()                      # what fills them runs on another stream
    ctx.hts_act(obs, params, 5, 1, 0, *out)
    torch.cuda.synchronize()
    ctx.close()
    rng.close()
    assert all(np.array_equal(x, y.cpu().numpy()) for x, y in zip(want, out))
