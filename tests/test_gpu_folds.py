"""Rules that choose a kernel's form by the number of heads: the same bits from
a call whose heads are many and from one head alone."""
import pytest
import torch

import paper_2604_16590_amd as la
from gpu_util import TOL, as64, normwise, require_gpu

pytestmark = pytest.mark.gpu


# workgroups of the apply at d = 128 from 129 heads on: one round of the chip
# (three, two a head, one), several, and fewer blocks than workgroups
@pytest.mark.parametrize("heads,N", [(129, 1100), (300, 700), (384, 2049), (511, 300), (700, 129)])
def test_apply_of_many_wide_heads(heads, N):
    dev = require_gpu()
    gen = torch.Generator(device=dev).manual_seed(heads)
    q = torch.randn((1, heads, N, 128), generator=gen, device=dev).bfloat16()
    S = torch.randn((1, heads, 128, 128), generator=gen, device=dev).double()
    z = torch.rand((1, heads, 128), generator=gen, device=dev).double() + 1
    o = la.apply(q, S, z)
    f = torch.where(q > 0, q.float() + 1, torch.exp(q.float())).bfloat16().double()
    ref = torch.matmul(f, S) / torch.matmul(f, z[..., None])
    torch.cuda.synchronize()
    assert normwise(as64(o), ref.cpu().numpy()) < TOL["bf16"]
    for h in (0, heads - 1):
        assert torch.equal(la.apply(q[:, h:h + 1], S[:, h:h + 1], z[:, h:h + 1]), o[:, h:h + 1])
