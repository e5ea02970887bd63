"""conv2, FC and the FC input gradient of large bf16 batches, whose operand tiles are copied straight into LDS: batches that
end inside a tile, on either side of each change of tile or stages, against the wave-per-segment kernels bit for bit; and
gradients where the input gradient changes tiles and where a bias is summed beside the column tiles (binary32)."""
import numpy as np
import pytest
import torch

from test_gpu_parity import ATARI, FOOT, _act, _rollout, _split, dev, hts  # noqa: F401
import hts_synth as syn

pytestmark = pytest.mark.gpu


# workgroups of 64x64 FC tiles at these sizes (84x84): 168, 504, 560, 728, 728, 840, 896, 952; 4100 rows add the groups in the
# kernel; 809 and 810 rows stand on either side of conv2's change of stages, which 4x84x84 frames no longer reach
@pytest.mark.parametrize("shape,A,sizes", [(ATARI, 18, (129, 576, 577, 809, 810, 960, 961, 1030, 4100)), (FOOT, 19, (129, 203, 833, 1409)),
                                           ((3, 44, 52), 7, (129, 500, 2113))])
def test_large_batches_agree_bitwise(hts, shape, A, sizes, monkeypatch):  # noqa: F811
    n = max(sizes)
    params = dev(syn.init_params(31, *shape, A, bias_scale=0.05))
    g = torch.Generator(device="cuda").manual_seed(32)
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


# As for small minibatches (twice the rows, half the weight of each): binary32 sums of at most n = 700 * 400 terms in another
# order, sqrt(n) 2^-24 = 3.2e-5.  bf16: 350 rows take 64x64 tiles of three stages of the FC input gradient, 700 rows of two.  Three channels end
# conv1's weight gradient inside a column tile, whose bias column is binary32's to sum beside the tiles.
@pytest.mark.parametrize("shape,A,B,precision", [(ATARI, 18, 350, 1), ((3, 44, 52), 7, 150, 1), (ATARI, 18, 330, 0), ((3, 44, 52), 7, 150, 0)])
def test_gradient_is_the_mean_of_its_halves(hts, oracle, shape, A, B, precision):  # noqa: F811
    _, params, obs, actions, old_logp, adv, ret = _rollout(oracle, shape, A, 2 * B, 900 + B, False)
    ctx = hts.Context(*shape, A, precision=precision, max_learn_batch=2 * B)

    def gradient(lo, hi):
        g = torch.full((ctx.P,), float("nan"), device="cuda")
        rows = [dev(x[lo:hi]) for x in (obs, actions, adv, ret)]
        ctx.hts_loss_and_grads(rows[0], rows[1], None, rows[2], rows[3], dev(params), hts.HParams(algo=hts.ALGO_A2C), g)
        torch.cuda.synchronize()
        return _split(g.cpu().numpy().astype(np.float64), shape, A)

    whole, first, second = gradient(0, 2 * B), gradient(0, B), gradient(B, 2 * B)
    for name, w in whole.items():
        mean = 0.5 * (first[name] + second[name])
        assert np.linalg.norm(w - mean) <= 3.2e-5 * np.linalg.norm(mean), name
    ctx.close()


# The FC input gradient's tiles, whose rows leave through LDS, each with a batch that ends inside one: 64x64 of 3 stages (3 tiles of rows, 6 of
# columns), of 2 (539 tiles), 64x128 (833) and 128x128 (825 of 64x128, 425 of 128x128); 64x128 tiles that end inside the last of 49 halves.
# The wave-per-segment kernels add the same products in another order: bfloat16 rounds each layer's gradient to 2^-9, and a sum that ends near
# a rounding edge may fall on either side, here and there.
@pytest.mark.parametrize("shape,A,B", [((3, 44, 52), 7, 131), (ATARI, 18, 700), (ATARI, 18, 1030), (ATARI, 18, 2050)])
def test_fc_input_gradient_tiles(hts, shape, A, B, monkeypatch):  # noqa: F811
    g = torch.Generator(device="cuda").manual_seed(B)
    params = dev(syn.init_params(33, *shape, A, bias_scale=0.05))
    obs = torch.randint(0, 256, (B, *shape), device="cuda", generator=g, dtype=torch.uint8)
    actions = torch.randint(0, A, (B,), device="cuda", generator=g, dtype=torch.int32)
    adv, ret = torch.randn(B, device="cuda", generator=g), torch.randn(B, device="cuda", generator=g)
    grads = []
    for knob in ("0", "1000000"):
        monkeypatch.setenv("HTS_SMALL_BATCH", knob)
        ctx = hts.Context(*shape, A, precision=1, max_learn_batch=B)
        out = torch.full((ctx.P,), float("nan"), device="cuda")
        ctx.hts_loss_and_grads(obs, actions, None, adv, ret, params, hts.HParams(algo=hts.ALGO_A2C), out)
        torch.cuda.synchronize()
        grads.append(_split(out.cpu().numpy().astype(np.float64), shape, A))
        ctx.close()
    for name, w in grads[1].items():
        assert np.linalg.norm(grads[0][name] - w) <= 2e-3 * np.linalg.norm(w), name
