"""How a head's sums over tokens are held: runs of at most 512 (d = 128: 1,024)
bf16 tokens in FP32, joined in FP64, a partial of four runs rounded once."""
import pytest
import torch

import paper_2604_16590_amd as la
from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,run", [(64, 512), (128, 1024)])
@pytest.mark.parametrize("heads", [1, 40])
def test_runs_are_joined_in_fp64(heads, d, run):
    # phi(0) = 1; the first run of the first partial sums to 2^24, the next
    # three to 1 each: 2^24 + 3 is held to half an ulp (of 2), where sums in
    # FP32 stay at 2^24
    dev = require_gpu()
    N = 16 * run
    k = torch.zeros((1, heads, N, d), dtype=torch.bfloat16, device=dev)
    v = torch.zeros_like(k)
    v[:, :, :run] = 2.0 ** 24 / run
    v[:, :, run:4 * run:run] = 1
    _, S, z = la.forward(k, k, v, return_summary=True)
    torch.cuda.synchronize()
    assert float((S - (2.0 ** 24 + 3)).abs().max()) <= 1
    assert bool((z == N).all())
