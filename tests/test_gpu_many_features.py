"""bfloat16 gradients of a minibatch whose conv3 outputs take more than 4 GB."""
import numpy as np
import pytest
import torch

import hts_synth as syn
from test_gpu_parity import _split, hts  # noqa: F401

pytestmark = pytest.mark.gpu


# 43008 rows of 1x256x256 frames have 43008 * 50176 > 2^31 activations of two bytes in front of the FC layer.  They are 128 times the
# same 336 rows: every row's own gradient is exactly 1/128 of what it is among the 336 (a power of two: also after rounding to bfloat16),
# so the two gradients differ by the order of their binary32 sums only, of at most n = 43008 * 3969 / 256 terms (a chunk of conv1's
# positions): sqrt(n) 2^-24 = 4.9e-5.  Rows that read as zero are missed by far more: 208 of 43008 kept, fc.w is off by 0.99.
def test_more_than_4_gb_of_features(hts):  # noqa: F811
    shape, A, n, times = (1, 256, 256), 3, 336, 128
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("needs 100 GB of device memory")
    params = torch.from_numpy(syn.init_params(51, *shape, A)).cuda()
    g = torch.Generator(device="cuda").manual_seed(52)
    obs = torch.randint(0, 256, (n, *shape), device="cuda", generator=g, dtype=torch.uint8)
    actions = torch.randint(0, A, (n,), device="cuda", generator=g, dtype=torch.int32)
    adv, ret = torch.randn(n, device="cuda", generator=g), torch.randn(n, device="cuda", generator=g)
    grads = []
    for B in (n, n * times):
        ctx = hts.Context(*shape, A, precision=1, max_learn_batch=B)
        out = torch.full((ctx.P,), float("nan"), device="cuda")
        index = (torch.arange(B, device="cuda") % n).to(torch.int32)
        ctx.hts_loss_and_grads(obs, actions, None, adv, ret, params, hts.HParams(algo=hts.ALGO_A2C), out, index=index, B=B)
        torch.cuda.synchronize()
        grads.append(_split(out.cpu().numpy().astype(np.float64), shape, A))
        ctx.close()
    errs = {name: np.linalg.norm(grads[1][name] - w) / np.linalg.norm(w) for name, w in grads[0].items()}
    for name, e in errs.items():
        assert e <= 4.9e-5, (name, e)
