"""Heads kernel at the batch sizes where its samples per workgroup change and with a last workgroup that is not full: an
actor call's logits, values and actions must equal, bit for bit, those of the same observations in other batches (every
batch size adds the same terms in the same order), and the learner's gradient must not depend on the workgroup either."""
import pytest
import torch

import hts_synth as syn
from test_gpu_parity import _act, dev, hts  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("A", [1, 16, 19, 24, 33, 64])
@pytest.mark.parametrize("N", [1025, 3075])
def test_heads_do_not_depend_on_the_batch(hts, A, N):  # noqa: F811
    shape = (2, 36, 36)
    params = dev(syn.init_params(9, *shape, A, bias_scale=0.05))
    obs = dev(syn.obs_uniform(10 + A, N, *shape))
    ctx = hts.Context(*shape, A, precision=1, max_act_batch=N)
    whole = _act(ctx, obs, params, 3, 1, 0, A)
    for lo, hi in ((0, 1), (1, 130), (700, 1024), (N - 1025, N)):
        part = _act(ctx, obs[lo:hi].contiguous(), params, 3, 1, lo, A)
        for w, p in zip(whole, part):
            assert (w[lo:hi] == p).all()
    ctx.close()


@pytest.mark.parametrize("A", [19, 20, 21])
@pytest.mark.parametrize("B", [513, 1024, 1025, 2049])
def test_heads_gradient_of_repeated_rows(hts, A, B):  # noqa: F811
    """B copies of one row: every row's share of the heads gradient is the same number, so pi.w's gradient is B times one
    row's, up to a binary32 chain over B equal terms (B 2^-24 at most) and the 1/B of the mean."""
    shape = (2, 36, 36)
    params = dev(syn.init_params(9, *shape, A, bias_scale=0.05))
    grads = []
    for n in (1, B):
        obs = dev(syn.obs_uniform(10, 1, *shape)).expand(n, -1, -1, -1).contiguous()
        ctx = hts.Context(*shape, A, precision=1, max_learn_batch=n)
        g = torch.zeros(ctx.P, device="cuda")
        ones = torch.ones(n, device="cuda")
        ctx.hts_loss_and_grads(obs, torch.zeros(n, dtype=torch.int32, device="cuda"), None, ones, ones, params, hts.HParams(), g)
        torch.cuda.synchronize()
        lo = ctx.P - (A + 1) * 513
        grads.append(g[lo:].double())
        ctx.close()
    assert float((grads[1] - grads[0]).norm() / grads[0].norm()) <= B * 2.0 ** -24
