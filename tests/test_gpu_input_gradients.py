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


def _both_kinds(hts, monkeypatch, shape, A, B, precision, obs, actions, adv, ret, params):
    grads = []
    for knob in ("0", "1000000"):
        monkeypatch.setenv("HTS_SMALL_BATCH", knob)
        ctx = hts.Context(*shape, A, precision=precision, max_learn_batch=B)
        g = torch.full((ctx.P,), float("nan"), device="cuda")
        ctx.hts_loss_and_grads(dev(obs), dev(actions), None, dev(adv), dev(ret), dev(params), hts.HParams(algo=hts.ALGO_A2C), g)
        torch.cuda.synchronize()
        grads.append(_split(g.cpu().numpy().astype(np.float64), shape, A))
        ctx.close()
    return grads


# The order of the rows changes at these sizes (64x64: conv3 at 256 rows; 104x104: conv3 at 256 tiles; 128x128: conv2 of bfloat16 stays in sample order
# for its input's size), and they give 2, 4 and 8 runs of unequal samples.  Bounds as above, n = 1030 * 64 and 260 * 225 terms.
@pytest.mark.parametrize("shape,A,B", [((3, 44, 52), 7, 255), ((3, 44, 52), 7, 257), ((2, 64, 64), 6, 255), ((2, 64, 64), 6, 260), ((2, 36, 36), 5, 517),
                                       ((2, 36, 36), 5, 1030), ((1, 104, 104), 6, 140), ((1, 128, 128), 6, 130)])
@pytest.mark.parametrize("precision", [0, 1])
def test_row_orders_agree(hts, oracle, shape, A, B, precision, monkeypatch):  # noqa: F811
    _, params, obs, actions, _, adv, ret = _rollout(oracle, shape, A, B, 950 + B, False)
    got, want = _both_kinds(hts, monkeypatch, shape, A, B, precision, obs, actions, adv, ret, params)
    for name, w in want.items():
        assert np.linalg.norm(got[name] - w) <= (1.9e-5 if precision == 0 else 2e-3) * np.linalg.norm(w), name


# An infinite weight of conv3 that closes its channel's ReLU: 0 times infinity is NaN where its tap reaches a position.  A left-out tap gives
# none where it does not (the other kernels multiply a zero there); the gradients, sums over all positions, are NaN in the same entries.
@pytest.mark.parametrize("precision", [0, 1])
def test_infinite_weight(hts, oracle, precision, monkeypatch):  # noqa: F811
    shape, A, B = (3, 44, 52), 7, 260
    _, params, obs, actions, _, adv, ret = _rollout(oracle, shape, A, B, 971, False)
    params = np.array(params, np.float32)
    _split(params, shape, A)["conv3.w"][(5 * 64 + 3) * 9] = -np.inf           # output channel 5, input channel 3, tap (0, 0)
    got, want = _both_kinds(hts, monkeypatch, shape, A, B, precision, obs, actions, adv, ret, params)
    assert np.isnan(want["conv2.b"]).sum() == 1 and np.isfinite(want["fc.w"]).all()
    for name, w in want.items():
        assert np.array_equal(np.isfinite(got[name]), np.isfinite(w)), name
        ok = np.isfinite(w)
        assert np.linalg.norm((got[name] - w)[ok]) <= (1.9e-5 if precision == 0 else 2e-3) * np.linalg.norm(w[ok]), name
