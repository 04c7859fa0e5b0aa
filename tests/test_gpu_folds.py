"""Rules that choose a kernel's form by the number of heads: the same bits from
a call whose heads are many and from one head alone."""
import pytest
import torch

import oracle
import paper_2604_16590_amd as la
from gpu_util import TOL, as64, normwise, require_gpu

pytestmark = pytest.mark.gpu


def combined(f):
    """f's results, and whether it launched the combine."""
    la.profile_enable(True)
    try:
        r = f()
        torch.cuda.synchronize()
        return r, "combine" in la.profile_read()
    finally:
        la.profile_enable(False)


# The partial sums of a head added up by the workgroups that read them, or by
# the combine before: calls that take different forms (the kernel timer tells
# which), and the oracle's results.
# Heads, tokens: 3 and 4 partials (d <= 32: up to 16), ragged.  At d <= 64 one
# head folds and many combine; at d = 128 one or two workgroups a head fold and the
# thirteen of a head alone combine (the key pass: from 512 heads)
@pytest.mark.parametrize("d,dtype,heads,N,passes", [
    (16, "bf16", 300, 319, 2), (16, "bf16", 300, 765, 2), (16, "bf16", 300, 1024, 2), (16, "fp32", 300, 319, 2),
    (32, "bf16", 300, 383, 2), (32, "bf16", 300, 512, 2), (32, "bf16", 300, 639, 2), (32, "bf16", 300, 2047, 2),
    (32, "fp32", 300, 319, 2), (32, "fp32", 300, 1024, 2),
    (64, "bf16", 300, 767, 2), (64, "bf16", 300, 1024, 2),
    (128, "bf16", 256, 1100, 1), (128, "bf16", 256, 1600, 1), (128, "bf16", 1000, 1100, 2), (128, "bf16", 600, 1599, 2)])
def test_partials_folded_or_combined(d, dtype, heads, N, passes):
    dev = require_gpu()
    gen = torch.Generator(device=dev).manual_seed(d + N)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    q, k, v, g = (torch.randn((1, heads, N, d), generator=gen, device=dev).to(dt) for _ in range(4))
    (o, S, z), many = combined(lambda: la.forward(q, k, v, return_summary=True))
    grads, many_b = combined(lambda: la.backward(q, k, v, S, z, g))
    o2 = la.apply(q, S, z)
    assert torch.equal(o, o2)
    for h in (0, heads // 2, heads - 1):
        x = [t[:, h:h + 1] for t in (q, k, v)]
        (o1, S1, z1), one = combined(lambda: la.forward(*x, return_summary=True))
        grads1, one_b = combined(lambda: la.backward(*x, S1, z1, g[:, h:h + 1]))
        assert many != one and (passes == 1 or many_b != one_b)
        for a, b in zip((o, S, z) + tuple(grads), (o1, S1, z1) + tuple(grads1)):
            assert torch.equal(a[:, h:h + 1], b)
    host = [t.float().cpu().numpy() for t in x + [g[:, h:h + 1]]]
    assert normwise(as64(o1), oracle.forward(*host[:3])) < TOL[dtype]
    for a, r in zip(grads1, oracle.backward(*host)):
        assert normwise(as64(a), r) < TOL[dtype]


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
