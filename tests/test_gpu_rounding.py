"""FP64 sums to bf16 operands: rounded once, not through fp32."""
import pytest
import torch

import paper_2604_16590_amd as la
from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


# beside a midpoint of two bf16 values by less than fp32 holds: above one whose
# lower neighbour is even, below one whose upper neighbour is
@pytest.mark.parametrize("value,rounded", [
    (1 + 2.0 ** -8 + 2.0 ** -40, 1 + 2.0 ** -7), (1 + 3 * 2.0 ** -8 - 2.0 ** -40, 1 + 2.0 ** -7),
    (-1 - 2.0 ** -8 - 2.0 ** -40, -1 - 2.0 ** -7), (1 + 2.0 ** -8, 1.0), (1 + 3 * 2.0 ** -8, 1 + 2.0 ** -6)])
def test_summary_operands_are_rounded_once(value, rounded):
    # d = 128 takes S as its bf16 hi part in the query backward: with phi = 1,
    # z and dO one-hot, dQ of the other features is that part
    dev = require_gpu()
    d, N = 128, 33
    q = torch.zeros((1, 1, N, d), dtype=torch.bfloat16, device=dev)
    g = torch.zeros_like(q)
    g[..., 7] = 1
    S = torch.full((1, 1, d, d), value, dtype=torch.float64, device=dev)
    z = torch.zeros((1, 1, d), dtype=torch.float64, device=dev)
    z[..., 5] = 1
    dq, _, _ = la.backward(q, q, q, S, z, g)
    torch.cuda.synchronize()
    other = [c for c in range(d) if c != 5]
    assert bool((dq[..., other].double() == rounded).all())
