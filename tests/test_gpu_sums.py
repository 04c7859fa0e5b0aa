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


# the longest sequence of four waves to a partial at d = 128, and one more
@pytest.mark.parametrize("N", [64 * 2048, 64 * 2048 + 1])
def test_widest_heads_around_the_longest_teams(N):
    dev = require_gpu()
    gen = torch.Generator(device=dev).manual_seed(N)
    k, v = (torch.randn((1, 3, N, 128), generator=gen, device=dev).bfloat16() for _ in range(2))
    _, S, z = la.forward(k[:, :, :N], k, v, return_summary=True)
    _, S1, z1 = la.forward(k[:, 2:], k[:, 2:], v[:, 2:], return_summary=True)
    torch.cuda.synchronize()
    assert torch.equal(S[:, 2:], S1) and torch.equal(z[:, 2:], z1)
    f = torch.where(k > 0, k.float() + 1, torch.exp(k.float())).bfloat16().double()
    for h in range(3):  # bf16 products are exact in 64 bits
        ref = torch.matmul(f[0, h].t().contiguous(), v[0, h].double())
        assert float((S[0, h] - ref).norm() / ref.norm()) < 1e-4
