"""Infinities at a head's last token, where the sequence ends inside a step:
the rows that pad the step add nothing, so the results are those of the
definition, not NaN.

The references follow from the definition: phi > 0, so an infinite upstream
gradient of one value feature makes that column of dS, and of dV for every
key, +infinity and leaves the other columns as they are.  Tolerances as in
test_gpu_backward."""
import numpy as np
import pytest
import torch

import oracle
import paper_2604_16590_amd as la
from gpu_util import TOL, as64, make_inputs, normwise, require_gpu, to_device

pytestmark = pytest.mark.gpu


# tokens: a tile of 16 cut, the second tile of a step missing, one step and
# one token, several workgroups with steps past the end; d = 16 is the
# two-pass form, fp32 has forms of its own
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("d", [16, 32, 64, 128])
@pytest.mark.parametrize("N", [5, 16, 33, 77, 1041])
def test_infinite_gradient_of_the_last_token(N, d, dtype):
    dev = require_gpu()
    feature = 5
    host = make_inputs((1, 2, N, d), dtype, seed=700 + N + d, streams=(0, 1, 2, 3))
    q, k, v, g = (to_device(x, dev) for x in host)
    ref = oracle.backward(*host)
    _, S, z = la.forward(q, k, v, return_summary=True)
    g[:, :, N - 1, feature] = float("inf")
    dq, _, dv = la.backward(q, k, v, S, z, g)
    torch.cuda.synchronize()
    other = [c for c in range(d) if c != feature]
    assert torch.isposinf(dv[..., feature]).all()
    assert normwise(as64(dv)[..., other], ref[2][..., other]) < TOL[dtype]
    assert normwise(as64(dq)[:, :, :N - 1], ref[0][:, :, :N - 1]) < TOL[dtype]
