"""Returns and advantage normalisation at the edges of their kernels' ranges, against the oracle."""
import numpy as np
import pytest
import torch

import hts_synth as syn
from test_gpu_parity import dev, hts  # noqa: F401

pytestmark = pytest.mark.gpu


# one workgroup / several (16384 entries), remainders of a 4-entry vector, a pointer that is not 16-byte aligned.
# The kernels work in float64 and round once: half an ulp of binary32 (6e-8) relative, 3e-7 allowed for the float64 sums'
# effect on a value near zero.
@pytest.mark.parametrize("n,shift", [(1, 0), (5, 1), (16383, 0), (16384, 2), (16385, 0), (65537, 3), (528387, 0)])
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
