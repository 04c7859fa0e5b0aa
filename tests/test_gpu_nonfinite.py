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


# the last token's 1 / den beyond fp32: every entry of dS takes the sign of
# that token's gradient times infinity, and dV with it (phi(k) > 0)
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("d", [16, 32, 64, 128])
@pytest.mark.parametrize("N", [17, 77])
def test_infinite_normaliser_of_the_last_token(N, d, dtype):
    dev = require_gpu()
    q, k, v, g = (to_device(x, dev) for x in make_inputs((1, 2, N, d), dtype, seed=800 + N + d, streams=(0, 1, 2, 3)))
    k = torch.full_like(k, -80.0)  # phi(k) ~ 2e-35
    q[:, :, N - 1] = -20.0         # its den ~ 2e-9 d N 2e-35 < 1 / FLT_MAX
    _, S, z = la.forward(q, k, v, return_summary=True)
    _, _, dv = la.backward(q, k, v, S, z, g)
    torch.cuda.synchronize()
    sign = torch.sign(g[:, :, N - 1:])
    assert (sign != 0).all()
    assert torch.equal(dv, (sign * float("inf")).expand_as(dv).to(dv.dtype))
