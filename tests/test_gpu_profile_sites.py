"""The event timer: every launch site that has a name is timed in an iteration of its own work, in both precisions."""
import numpy as np
import pytest
import torch

from test_gpu_parity import _rollout, dev, hts  # noqa: F401

pytestmark = pytest.mark.gpu


# Rows on both sides of the wave-per-segment kernels' limit.  One launch at least of each site; as many of a shared launch under each of its names.
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("B", [40, 200])
def test_every_site_is_timed(hts, oracle, precision, B):  # noqa: F811
    shape, A = (2, 36, 36), 5
    _, params, obs, actions, old_logp, adv, ret = _rollout(oracle, shape, A, B, 300 + B, False)
    ctx = hts.Context(*shape, A, precision=precision, max_act_batch=B, max_learn_batch=B)
    obs_d, params_d, adv_d = dev(obs), dev(params), dev(adv)
    actions_d, logp, values = dev(actions), torch.zeros(B, device="cuda"), torch.zeros(B, device="cuda")
    opt, stats = hts.OptState(torch.zeros(ctx.P, device="cuda"), torch.zeros(ctx.P, device="cuda"), 0), ctx.new_stats()
    rew, vals, dones = torch.zeros(2, B, device="cuda"), torch.zeros(3, B, device="cuda"), torch.zeros(2, B, dtype=torch.uint8, device="cuda")
    out = torch.zeros(2, B, device="cuda"), torch.zeros(2, B, device="cuda")
    launches = {}
    for i, name in enumerate(ctx.profile_sites()):
        ctx.hts_profile_begin(i)
        ctx.hts_act(obs_d, params_d, 7, 0, 0, actions_d, logp, values)
        ctx.hts_returns_gae(rew, vals, dones, 0.99, 0.95, *out)
        ctx.hts_normalize_advantages(adv_d)
        ctx.hts_learner_step(obs_d, actions_d, logp, adv_d, dev(ret), params_d, opt, hts.HParams(algo=hts.ALGO_A2C), stats=stats)
        launches[name], ms = ctx.hts_profile_end()
        assert launches[name] >= 1 and np.isfinite(ms), name
    shared = ("wgrads", "heads_wgrad", "fc_wgrad") + (() if precision else ("conv1_wgrad", "conv2_wgrad", "conv3_wgrad"))
    assert [launches[n] for n in shared] == [1] * len(shared)
    ctx.close()
