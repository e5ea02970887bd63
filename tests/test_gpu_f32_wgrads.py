"""binary32 weight gradients at the edges of their split: the heads' beyond 512 rows (groups of 16 segments of 32 rows, the last
one short) with more rows of heads than one tile holds, beside the conv and FC weight gradients of the same launch."""
import numpy as np
import pytest
import torch

from test_gpu_parity import ATARI, FOOT, _rollout, _split, dev, hts, oracle_hp  # noqa: F401

pytestmark = pytest.mark.gpu


# Sums of n <= 545 * 64 products (conv1 positions of 2x36x36 frames) in binary32: sqrt(n) 2^-24 = 1.1e-5 of their size.  Among the
# 1030 rows' activations some lie so near zero that a ReLU gate opens on one side only (one gate of one row: some 5e-5 of conv1.w's
# gradient); only the heads' own gradients, to which an activation near zero adds nothing, are compared there.
@pytest.mark.parametrize("A,B", [(5, 512), (33, 513), (64, 545), (18, 1030)])
def test_f32_gradient_of_many_rows(hts, oracle, A, B):  # noqa: F811
    shape = (2, 36, 36)
    net, params, obs, actions, old_logp, adv, ret = _rollout(oracle, shape, A, B, 500 + B, False)
    ctx = hts.Context(*shape, A, max_learn_batch=B)
    hp = hts.HParams(algo=hts.ALGO_A2C)
    index = torch.randperm(B, generator=torch.Generator().manual_seed(B)).to(torch.int32)
    grads = []
    for idx in (None, index.cuda()):
        g = torch.full((ctx.P,), float("nan"), device="cuda")
        ctx.hts_loss_and_grads(dev(obs), dev(actions), None, dev(adv), dev(ret), dev(params), hp, g, index=idx)
        torch.cuda.synchronize()
        grads.append(g.cpu().numpy().astype(np.float64))
    want, _ = oracle.loss_grads(net, params, obs, actions, old_logp, adv, ret, oracle_hp(oracle, hp), threads=oracle.host_threads())
    for got in grads:
        for name, w in _split(want, shape, A).items():
            if B == 1030 and name not in ("pi.w", "pi.b", "v.w", "v.b"):
                continue
            err = np.linalg.norm(_split(got, shape, A)[name] - w) / np.linalg.norm(w)
            assert err <= 1.1e-5, (name, err)
    ctx.close()


# The register kernels on the frames of the two workloads, chunks and last blocks ragged; an indexed minibatch, whose conv1 reads its frames through
# the index.  1e-4: binary32's bound for gradients (sums of 151 * 400 products are off by 1.5e-5 of their size, a gate of one row that opens on one
# side only by some 5e-5); a row or a column left out would be 1e-2 and more.
@pytest.mark.parametrize("shape,A,count,B", [(ATARI, 18, 160, 151), (FOOT, 19, 140, 133)])
def test_f32_gradient_of_workload_frames(hts, oracle, shape, A, count, B):  # noqa: F811
    net, params, obs, actions, old_logp, adv, ret = _rollout(oracle, shape, A, count, 700 + B, False)
    index = torch.randperm(count, generator=torch.Generator().manual_seed(B)).to(torch.int32)[:B]
    ctx = hts.Context(*shape, A, max_learn_batch=B)
    hp = hts.HParams(algo=hts.ALGO_A2C)
    g = torch.full((ctx.P,), float("nan"), device="cuda")
    ctx.hts_loss_and_grads(dev(obs), dev(actions), None, dev(adv), dev(ret), dev(params), hp, g, index=index.cuda())
    torch.cuda.synchronize()
    got = _split(g.cpu().numpy().astype(np.float64), shape, A)
    want, _ = oracle.loss_grads(net, params, obs, actions, old_logp, adv, ret, oracle_hp(oracle, hp), index=index.numpy(), threads=oracle.host_threads())
    for name, w in _split(want, shape, A).items():
        err = np.linalg.norm(got[name] - w) / np.linalg.norm(w)
        assert err <= 1e-4, (name, err)
    ctx.close()
