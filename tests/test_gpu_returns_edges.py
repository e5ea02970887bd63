"""Returns and advantage normalisation at the edges of their kernels' ranges, against the oracle."""
import ctypes as C
import threading

import numpy as np
import pytest
import torch

import hts_synth as syn
from test_gpu_parity import dev, hts  # noqa: F401

pytestmark = pytest.mark.gpu


# four or sixteen wavefronts (4096 entries) / several workgroups (16384), remainders of a 4-entry vector, a pointer that is not 16-byte aligned.
# The kernels work in float64 and round once: half an ulp of binary32 (6e-8) relative, 3e-7 allowed for the float64 sums'
# effect on a value near zero.
@pytest.mark.parametrize("n,shift", [(1, 0), (5, 1), (4096, 0), (4097, 1), (16383, 0), (16384, 2), (16385, 0), (65537, 3), (528387, 0)])
def test_normalize_edges(hts, oracle, n, shift):  # noqa: F811
    ctx = hts.Context(4, 84, 84, 6, max_act_batch=1)
    a = (syn.normal_f32(n, syn.S_MISC, (n,)) * 3 + 100).astype(np.float32)
    buf = torch.full((n + 8,), 7.0, device="cuda")
    buf[shift:shift + n] = dev(a)
    ctx.hts_normalize_advantages(buf[shift:shift + n])
    torch.cuda.synchronize()
    got = buf.cpu().numpy()
    assert (got[:shift] == 7.0).all() and (got[shift + n:] == 7.0).all()
    np.testing.assert_allclose(got[shift:shift + n], oracle.normalize_adv(a), rtol=3e-7, atol=3e-7)
    ctx.close()


# One infinity or NaN makes the mean or the deviation infinite or NaN, and with it every result NaN: in the one-workgroup
# kernels (4 and 16 wavefronts) and in the several workgroups of larger arrays, wherever it stands (entry 0 is the point
# about which the latter sum).
@pytest.mark.parametrize("n", [5, 4096, 8192, 16384, 16385, 70000])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
def test_normalize_nonfinite(hts, n, value):  # noqa: F811
    ctx = hts.Context(4, 84, 84, 6, max_act_batch=1)
    for at in (0, n // 2, n - 1):
        a = syn.normal_f32(n, syn.S_MISC, (n,)).astype(np.float32)
        a[at] = value
        buf = dev(a)
        ctx.hts_normalize_advantages(buf)
        torch.cuda.synchronize()
        assert bool(torch.isnan(buf).all()), at
    ctx.close()


# Without a context the call goes to stream 0 and, beyond 16384 entries, its two launches pass their sums through one array of
# the library: calls of several threads with other sizes and means must come out as they do with a context, bit for bit.
def test_normalize_without_a_context_from_several_threads(hts):  # noqa: F811
    calls, sizes = 60, (4097, 16385, 70000, 300001)
    ctx = hts.Context(4, 84, 84, 6, max_act_batch=1, stream=torch.cuda.default_stream())
    lib = hts.binding.load_library()
    bufs, wants = [], []
    for i, n in enumerate(sizes):
        x = dev(syn.normal_f32(n, syn.S_MISC, (n,)) * (i + 1) + 10 * i)
        bufs.append([x.clone() for _ in range(calls)])
        ctx.hts_normalize_advantages(x)
        wants.append(x)
    torch.cuda.synchronize()
    codes, start = [], threading.Barrier(len(sizes))

    def work(mine, n):
        start.wait()
        for b in mine:
            codes.append(lib.hts_normalize_advantages(None, C.c_void_p(b.data_ptr()), n))

    threads = [threading.Thread(target=work, args=(b, n)) for b, n in zip(bufs, sizes)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert codes == [0] * (calls * len(sizes))
    for mine, want in zip(bufs, wants):
        assert all(torch.equal(b, want) for b in mine)
    ctx.close()


# Infinities and NaN spread backwards in time until the column's first step and never to another column, the same in the
# plain and the chunked kernels as in the oracle's sequential float64 recurrence (0 * inf at an episode's end is NaN there too).
@pytest.mark.parametrize("T,N", [(5, 40), (14, 40), (30, 40), (130, 40), (300, 40), (1100, 6), (70, 8200), (13, 131072)])
def test_gae_nonfinite(hts, oracle, T, N):  # noqa: F811
    ctx = hts.Context(4, 84, 84, 6, max_act_batch=1)
    r, v = syn.normal_f32(T + N, syn.S_REW, (T, N)), syn.normal_f32(T * 7 + N, syn.S_VAL, (T + 1, N))
    d = syn.dones_bernoulli(T + N, T, N, 0.02)
    r[T // 2, 0], r[T - 1, 1], v[T // 3, 2], v[T, 3], v[0, 4] = np.inf, -np.inf, np.nan, np.inf, np.nan
    r[T // 2, 5], r[T // 4, 5] = np.inf, -np.inf
    adv, ret = torch.zeros(T, N, device="cuda"), torch.zeros(T, N, device="cuda")
    ctx.hts_returns_gae(dev(r), dev(v), dev(d), 0.99, 0.95, adv, ret)
    torch.cuda.synchronize()
    with np.errstate(invalid="ignore"):
        a_ref, r_ref = oracle.gae(r, v, d, np.float32(0.99), np.float32(0.95))
    for got, want in ((adv, a_ref), (ret, r_ref)):
        np.testing.assert_allclose(got.cpu().numpy(), want.astype(np.float32), rtol=1e-6, atol=1e-6)
    ctx.close()


# plain / chunked kernels (11 steps; 131072 columns, 81920 for 33 to 96 steps), each column width (4, 16, 64; 64 up to 40 steps),
# spans that end exactly at, one step before and one step after a multiple of the span, a last workgroup with dead columns.
# The tolerance of the oracle's other returns tests: one binary32 rounding of a float64 recurrence.
@pytest.mark.parametrize("T,N", [(8, 3), (9, 1), (11, 100), (12, 1), (12, 70), (40, 65), (41, 65), (257, 5), (513, 512), (512, 513), (256, 17), (255, 16), (65, 8193),
                                 (64, 8192), (1025, 2), (9, 131071), (9, 131072), (12, 131071), (33, 81919), (33, 81920), (97, 81920)])
def test_gae_edges(hts, oracle, T, N):  # noqa: F811
    ctx = hts.Context(4, 84, 84, 6, max_act_batch=1)
    r, v = syn.normal_f32(T + N, syn.S_REW, (T, N)), syn.normal_f32(T * 7 + N, syn.S_VAL, (T + 1, N))
    d = syn.dones_bernoulli(T + N, T, N, 0.02)
    adv, ret = torch.zeros(T, N, device="cuda"), torch.zeros(T, N, device="cuda")
    ctx.hts_returns_gae(dev(r), dev(v), dev(d), 0.99, 0.95, adv, ret)
    torch.cuda.synchronize()
    a_ref, r_ref = oracle.gae(r, v, d, np.float32(0.99), np.float32(0.95))
    for got, want in ((adv, a_ref), (ret, r_ref)):
        err = np.abs(got.cpu().numpy().astype(np.float64) - want) / np.maximum(1.0, np.abs(want))
        assert float(err.max()) <= 1e-6
    ctx.close()


# The outputs may be written over the inputs (advantages over the rewards, returns over the first T rows of the values, or the
# other way round): plain kernel (T, N at either end of its range) and chunked kernels of each column width, with one span of
# time and with several, the last one partial.
@pytest.mark.parametrize("T,N", [(5, 33), (8, 40), (13, 131072), (13, 17), (30, 300), (130, 40), (300, 700), (700, 1030), (1100, 5), (2048, 6), (64, 8200), (135, 8200)])
def test_gae_in_place(hts, T, N):  # noqa: F811
    ctx = hts.Context(4, 84, 84, 6, max_act_batch=1)
    r, v = dev(syn.normal_f32(T + N, syn.S_REW, (T, N))), dev(syn.normal_f32(T * 7 + N, syn.S_VAL, (T + 1, N)))
    d = dev(syn.dones_bernoulli(T + N, T, N, 0.02))
    adv, ret = torch.zeros(T, N, device="cuda"), torch.zeros(T, N, device="cuda")
    ctx.hts_returns_gae(r, v, d, 0.99, 0.95, adv, ret)
    for swap in (False, True):
        r2, v2 = r.clone(), v.clone()
        outs = (v2[:T], r2) if swap else (r2, v2[:T])
        ctx.hts_returns_gae(r2, v2, d, 0.99, 0.95, *outs)
        torch.cuda.synchronize()
        assert torch.equal(outs[0], adv) and torch.equal(outs[1], ret) and torch.equal(v2[T], v[T]), swap
    ctx.close()
