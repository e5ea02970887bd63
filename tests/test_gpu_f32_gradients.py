"""binary32 backward kernels: gradients at the edges of their tiles, and
over operands whose magnitudes spread over many binades, against the oracle's float64 gradient; the order of their sums,
bit for bit, against chains of fused multiply-adds on the host."""
import numpy as np
import pytest
import torch

import hts_synth as syn
from test_gpu_parity import ATARI, _rollout, _split, dev, hts, oracle_hp  # noqa: F401

pytestmark = pytest.mark.gpu


# 128 / 129 rows: last of the wave-per-segment, first of the tile kernels; 65 = one row more than a 64-row tile; 3x44x52 and
# 2x36x36 frames have feature counts that end inside a tile, and conv1 columns that end inside one beside the bias column.  A
# sum of n products of binary32 numbers in binary32 is off by about sqrt(n) 2^-24 of its size: n is at most B * P1 = 129 * 120
# (3x44x52) or 97 * 400 positions, so 1.2e-5.  Rows of `adv` scaled over 2^-20 .. 2^20 leave the gradient to a few rows.
@pytest.mark.parametrize("shape,A,B,spread", [((3, 44, 52), 7, 65, 0), ((3, 44, 52), 7, 96, 20), ((3, 44, 52), 7, 97, 20), ((3, 44, 52), 7, 129, 20),
                                              ((2, 36, 36), 5, 129, 0), (ATARI, 18, 97, 0)])
def test_f32_gradient(hts, oracle, shape, A, B, spread):  # noqa: F811
    Cc, H, W = shape
    net, params, obs, actions, old_logp, adv, ret = _rollout(oracle, shape, A, B, 300 + B, False)
    adv = (adv * 2.0 ** np.linspace(-spread, spread, B)).astype(np.float32)
    ctx = hts.Context(Cc, H, W, A, max_learn_batch=B)
    hp = hts.HParams(algo=hts.ALGO_A2C)
    grads = torch.full((ctx.P,), float("nan"), device="cuda")
    ctx.hts_loss_and_grads(dev(obs), dev(actions), None, dev(adv), dev(ret), dev(params), hp, grads)
    torch.cuda.synchronize()
    want, _ = oracle.loss_grads(net, params, obs, actions, old_logp, adv, ret, oracle_hp(oracle, hp), threads=oracle.host_threads())
    got = grads.cpu().numpy().astype(np.float64)
    for name, w in _split(want, shape, A).items():
        err = np.linalg.norm(_split(got, shape, A)[name] - w) / np.linalg.norm(w)
        assert err <= 1.2e-5, (name, err)
    ctx.close()


def _fma(a, b, c):
    """binary32 fma, correctly rounded: the exact product of two binary32 numbers and the sum rounded to odd fit float64."""
    p, c = np.asarray(a, np.float64) * np.asarray(b, np.float64), np.asarray(c, np.float64)
    s = p + c
    t = s - p
    e = (p - (s - t)) + (c - t)                                  # s + e is the exact sum
    to_odd = (e != 0.0) & ((s.view(np.int64) & 1) == 0)
    return np.where(to_odd, np.nextafter(s, np.copysign(np.inf, e)), s).astype(np.float32)


def test_f32_matrix_instruction_is_an_fma_chain(hts):  # noqa: F811
    """v_mfma_f32_32x32x2_f32 adds its products as a sequential chain of fused multiply-adds, lowest k first, so that a column
    summed by fma beside the tiles (a weight gradient's bias) has the bits that a tile of columns would give it."""
    M, N, K = 70, 33, 328
    a, b = syn.normal_f32(41, syn.S_MISC, (M, K)), syn.normal_f32(42, syn.S_MISC, (N, K))
    ctx = hts.Context(4, 84, 84, 6, max_act_batch=1)
    out = torch.full((M, N), float("nan"), device="cuda")
    ctx.hts_test_gemm(0, dev(a), dev(b), out)
    torch.cuda.synchronize()
    want = np.zeros((M, N), np.float32)
    for k in range(K):
        want = _fma(a[:, k, None], b[None, :, k], want)
    assert np.array_equal(out.cpu().numpy(), want)
    ctx.close()


def _chunked_column(dy, x):
    """What the tile kernels and the reduction make of a bias column: rows of dy in chunks of klen, each a chain of
    fma(dy, x, .), then eight ranges of chunks added in order, then the ranges; 64 chunks at most (256 for conv1)."""
    rows, maxz = len(dy), 256 if x == 255.0 else 64
    klen = max(256, -(-(-(-rows // maxz)) // 32) * 32)
    parts = []
    for k0 in range(0, rows, klen):
        s = np.zeros(dy.shape[1], np.float32)
        for row in dy[k0:k0 + klen]:
            s = _fma(row, np.float32(x), s)
        parts.append(s)
    assert rows % klen % 32                                      # the last k-tile is not full
    per = -(-len(parts) // 8)
    total = None
    for q in range(8):
        s = np.zeros(dy.shape[1], np.float32)
        for p in parts[q * per:(q + 1) * per]:
            s = s + p
        total = s if total is None else total + s
    return total


def test_f32_bias_gradients_are_fma_chains(hts):  # noqa: F811
    """conv biases of the tile kernels bit for bit.  A network whose activations are all 1 and whose weights are powers of two
    on one path per unit: every row's gradient at the value head is known, and what reaches the layers is that times a power of two."""
    shape, A, B = (3, 44, 52), 7, 131
    net = {n: np.zeros(s, np.float32) for n, s in syn.param_shapes(*shape, A)}
    H2, W2, H3, W3 = 4, 5, 2, 3                                  # 10x12 -> 4x5 -> 2x3 positions
    net["conv1.b"][:] = 1.0
    for c in range(32):
        net["conv2.w"][c, c, 0, 0] = 0.5
    net["conv2.b"][:32], net["conv2.b"][32:] = 0.5, 1.0
    for c in range(64):
        net["conv3.w"][c, c, 0, 0] = 0.5
    net["conv3.b"][:] = 0.5
    path = (2.0 ** -(np.arange(64 * H3 * W3) % 7)).astype(np.float32)
    net["fc.w"][0] = path
    net["v.w"].reshape(-1)[0] = 1.0
    value = np.float32(path.astype(np.float64).sum())
    ret = syn.normal_f32(43, syn.S_MISC, (B,))
    dv = (np.float32(0.5) * (np.float32(2.0) * (value - ret))) * (np.float32(1.0) / np.float32(B))
    dy3 = np.zeros((B, H2, W2, 64), np.float32)                  # on conv2's positions: the output positions are its first 2x3
    dy3[:, :H3, :W3] = dv[:, None, None, None] * path.reshape(64, H3, W3).transpose(1, 2, 0)
    dy2 = dy3 * np.float32(0.5)
    dy1 = np.zeros((B, 10, 12, 32), np.float32)
    dy1[:, 0:2 * H2:2, 0:2 * W2:2] = dy2[..., :32] * np.float32(0.5)
    want = {"conv3.b": _chunked_column(dy3[:, :H3, :W3].reshape(-1, 64), 1.0), "conv2.b": _chunked_column(dy2.reshape(-1, 64), 1.0),
            "conv1.b": _chunked_column(dy1.reshape(-1, 32), 255.0) * np.float32(1.0 / 255.0)}
    ctx = hts.Context(*shape, A, max_learn_batch=B)
    grads = torch.full((ctx.P,), float("nan"), device="cuda")
    params = np.concatenate([net[n].reshape(-1) for n, _ in syn.param_shapes(*shape, A)])
    ctx.hts_loss_and_grads(dev(syn.obs_uniform(44, B, *shape)), torch.zeros(B, dtype=torch.int32, device="cuda"), None,
                           torch.zeros(B, device="cuda"), dev(ret), dev(params), hts.HParams(algo=hts.ALGO_A2C, vf_coef=0.5, ent_coef=0.0), grads)
    torch.cuda.synchronize()
    got = _split(grads.cpu().numpy(), shape, A)
    for name, w in want.items():
        assert np.array_equal(got[name], w), (name, got[name][:4], w[:4])
    ctx.close()
