"""conv input gradients of the tile kernel, whose tiles are samples of one input position and leave out the taps that do not reach
it: against the wave-per-segment kernels, which multiply all of them in sample order."""
import numpy as np
import pytest
import torch

from test_gpu_parity import ATARI, FOOT, _rollout, _split, dev, hts  # noqa: F401

pytestmark = pytest.mark.gpu


# Tiles of 64 and 128 rows inside one position (256 samples), over two or three (131, 70) and over more than three, which multiply
# every tap (5, 20); 72x96 frames have a row of conv1 outputs that no conv2 window reaches.  The two sides add the same products in
# another order, binary32 sums of at most n = 256 * 400 terms: sqrt(n) 2^-24 = 1.9e-5.
@pytest.mark.parametrize("shape,A,B", [((3, 44, 52), 7, 5), ((3, 44, 52), 7, 20), ((3, 44, 52), 7, 70), (ATARI, 18, 131), (FOOT, 19, 70), ((2, 36, 36), 5, 256)])
@pytest.mark.parametrize("precision", [0, 1])
def test_input_gradients_agree(hts, oracle, shape, A, B, precision, monkeypatch):  # noqa: F811
    _, params, obs, actions, _, adv, ret = _rollout(oracle, shape, A, B, 950 + B, False)
    grads = []
    for knob in ("0", "1000000"):
        monkeypatch.setenv("HTS_SMALL_BATCH", knob)
        ctx = hts.Context(*shape, A, precision=precision, max_learn_batch=B)
        g = torch.full((ctx.P,), float("nan"), device="cuda")
        ctx.hts_loss_and_grads(dev(obs), dev(actions), None, dev(adv), dev(ret), dev(params), hts.HParams(algo=hts.ALGO_A2C), g)
        torch.cuda.synchronize()
        grads.append(_split(g.cpu().numpy().astype(np.float64), shape, A))
        ctx.close()
    # bfloat16 rounds each layer's gradient to 2^-9: a sum that ends near a rounding edge may fall on either side, here and there
    bound = 1.9e-5 if precision == 0 else 2e-3
    for name, w in grads[1].items():
        assert np.linalg.norm(grads[0][name] - w) <= bound * np.linalg.norm(w), name
