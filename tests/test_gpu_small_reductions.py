"""Advantage normalisation where its one workgroup changes from eight wavefronts to sixteen; the gradient norm in the statistics."""
import numpy as np
import pytest
import torch

import hts_synth as syn
from test_gpu_parity import ATARI, _rollout, dev, hts  # noqa: F401

pytestmark = pytest.mark.gpu


# (bounds: float64 sums and one rounding, half an ulp of binary32 = 6e-8 relative; 3e-7 for the sums' effect near zero)
@pytest.mark.parametrize("n,shift", [(4097, 0), (8191, 0), (8192, 1), (8193, 0)])
def test_normalize_eight_wavefronts(hts, oracle, n, shift):  # noqa: F811
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


# The norm is that of the returned gradient: binary32 sums of squares, 32 a thread, then trees of 8 and at most 8 + 1 steps: 49 roundings
# of 2^-24, halved by the root.  With and without the statistics a step takes the same clip factor, hence the same bits.
@pytest.mark.parametrize("A", [6, 64])
def test_norm_in_the_statistics(hts, oracle, A):  # noqa: F811
    B = 20
    _, params, obs, actions, old_logp, adv, ret = _rollout(oracle, ATARI, A, B, 990 + A, False)
    ctx = hts.Context(*ATARI, A, max_learn_batch=B)
    hp = hts.HParams(algo=hts.ALGO_A2C, max_grad_norm=1e-3)
    g, stats = torch.zeros(ctx.P, device="cuda"), ctx.new_stats()
    ctx.hts_loss_and_grads(dev(obs), dev(actions), None, dev(adv), dev(ret), dev(params), hp, g, stats=stats)
    torch.cuda.synchronize()
    norm = np.linalg.norm(g.cpu().numpy().astype(np.float64))
    assert abs(ctx.read_stats(stats)["grad_norm"] - norm) <= 49 / 2 * 2.0 ** -24 * norm
    after = []
    for st in (None, ctx.new_stats()):
        p = dev(params)
        opt = hts.OptState(torch.zeros(ctx.P, device="cuda"), torch.zeros(ctx.P, device="cuda"), 0)
        ctx.hts_learner_step(dev(obs), dev(actions), None, dev(adv), dev(ret), p, opt, hp, stats=st)
        torch.cuda.synchronize()
        after.append(p.cpu().numpy())
    assert np.array_equal(*after) and not np.array_equal(after[0], params.astype(np.float32))
    ctx.close()
