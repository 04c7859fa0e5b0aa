"""The summary's forms at the sizes where they change: a workgroup or a wave
to a partial, and the ragged ends of a workgroup's steps.

Tolerances as in test_gpu_forward.check: bf16 rounds phi(k) once (u = 2^-8,
4e-3 normwise for S and z with the FP32 sums), fp32 carries only FP32 sums
(1e-5 for S, 1e-6 for z)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2604_16590_amd as la
from gpu_util import TOL, as64, make_inputs, normwise, require_gpu, to_device

pytestmark = pytest.mark.gpu

# tokens: one step of four waves (bf16: 32 a wave, fp32: 16) less and more
# one; around the first second partial (4 d in bf16, 2 d in fp32); for the
# narrowest heads the last and first counts on either side of 2,048 tokens
# to a partial (64 partials)
SIZES = [(64, "bf16", n) for n in (31, 127, 128, 129, 256, 257, 8193)] + \
        [(64, "fp32", n) for n in (15, 63, 65, 128, 129, 8193)] + \
        [(128, "bf16", n) for n in (127, 129, 512, 513)] + \
        [(16, "bf16", 64 * 2048), (16, "bf16", 64 * 2048 + 1), (32, "fp32", 5 * 64 + 1)]


@pytest.mark.parametrize("d,dtype,N", SIZES)
def test_summary_forms(d, dtype, N):
    dev = require_gpu()
    B, H = (1, 1) if N > 100000 else (3, 3)  # nine items: not a multiple of eight
    q, k, v = make_inputs((B, H, N, d), dtype, seed=500 + N)
    tq, tk, tv = (to_device(x, dev) for x in (q, k, v))
    o, S, z = la.forward(tq, tk, tv, return_summary=True)
    torch.cuda.synchronize()
    o_ref, S_ref, z_ref = oracle.forward(q, k, v, want_summary=True)
    assert normwise(as64(o), o_ref) < TOL[dtype]
    assert normwise(S.cpu().numpy(), S_ref) < (4e-3 if dtype == "bf16" else 1e-5)
    assert normwise(z.cpu().numpy()[..., None], z_ref[..., None]) < (4e-3 if dtype == "bf16" else 1e-6)
    # the same bits alone as in a batch
    last = [x[B - 1:, H - 1:].contiguous() for x in (tq, tk, tv)]
    o1, S1, z1 = la.forward(*last, return_summary=True)
    torch.cuda.synchronize()
    assert torch.equal(o1, o[B - 1:, H - 1:]) and torch.equal(S1, S[B - 1:, H - 1:])
    assert torch.equal(z1, z[B - 1:, H - 1:])
    assert np.isfinite(as64(o)).all()
