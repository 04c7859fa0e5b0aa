"""Workspaces of the least size that a pass accepts, where not even one head's
usual partials fit: fewer partials, the same accuracy, nothing written beyond
the workspace.  Tolerances as in test_gpu_forms."""
import ctypes

import pytest
import torch

import oracle
from gpu_util import TOL, as64, make_inputs, normwise, require_gpu, to_device
from paper_2604_16590_amd import _binding as BB

pytestmark = pytest.mark.gpu


def up(n):
    return -(-n // 256) * 256


@pytest.mark.parametrize("H,N,d,dtype", [
    (1, 4096, 128, "fp32"), (3, 4096, 128, "fp32"), (1, 4096, 64, "fp32"), (1, 777, 32, "fp32"), (1, 600, 16, "fp32"),
    (1, 1000, 64, "bf16"), (1, 2048, 128, "bf16"), (1, 513, 32, "bf16"), (1, 4096, 16, "bf16")])
def test_least_workspace_of_few_heads(H, N, d, dtype):
    dev = require_gpu()
    host = make_inputs((1, H, N, d), dtype, seed=N + d, streams=(0, 1, 2, 3))
    q, k, v, g = (to_device(x, dev) for x in host)
    o, dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(4))
    S = torch.full((1, H, d, d), float("nan"), dtype=torch.float64, device=dev)
    z = torch.full((1, H, d), float("nan"), dtype=torch.float64, device=dev)
    desc = BB.make_desc(q, o)
    st = BB._stream(q.device)
    partials = -(-N // (2048 if d == 128 else 512))
    images = BB.workspace_size(desc, 2)
    least = up(H * partials * (d * d + d) * 4) + up(H * d * d * 8) + up(H * d * 8) + images
    stash = 0 if dtype == "bf16" and d >= 32 else up(H * N * 8)

    def call(pass_, nbytes, ws):
        if pass_ == 0:
            return BB.lib().la_forward(ctypes.byref(desc), *[x.data_ptr() for x in (q, k, v, o, S, z, ws)], nbytes, st)
        return BB.lib().la_backward(ctypes.byref(desc), *[x.data_ptr() for x in (q, k, v, S, z, g, dq, dk, dv, ws)],
                                    nbytes, st)

    for pass_, nbytes in ((0, least), (1, least + stash + images)):
        ws = torch.zeros(nbytes + 4096, dtype=torch.uint8, device=dev)
        ws[nbytes:] = 0xA5
        if nbytes <= BB.workspace_size(desc, pass_):
            assert call(pass_, nbytes - 256, ws) == 3  # LA_ERR_OOM
        assert call(pass_, nbytes, ws) == 0
        torch.cuda.synchronize()
        assert bool((ws[nbytes:] == 0xA5).all())
    o_ref, S_ref, z_ref = oracle.forward(*host[:3], want_summary=True)
    assert normwise(as64(o), o_ref) < TOL[dtype]
    assert normwise(S.cpu().numpy(), S_ref) < (4e-3 if dtype == "bf16" else 1e-5)
    assert normwise(z.cpu().numpy()[..., None], z_ref[..., None]) < (4e-3 if dtype == "bf16" else 1e-6)
    for x, r in zip((dq, dk, dv), oracle.backward(*host)):
        assert normwise(as64(x), r) < TOL[dtype]


@pytest.mark.parametrize("H", [1, 8])
def test_served_member_of_the_least_size(H):
    # a budget with no room for the usual workspace: parts of the heads (the
    # same bits), or for one head fewer partials
    import paper_2604_16590_amd as la
    from paper_2604_16590_amd import serve
    dev = require_gpu()
    N, d = 4096, 128
    host = make_inputs((1, H, N, d), "fp32", seed=H)
    q, k, v = (to_device(x, dev) for x in host)
    o = torch.full_like(q, float("nan"))
    desc = BB.make_desc(q, o)
    keep = up(H * d * d * 8) + up(H * d * 8)
    least = up(H * 2 * (d * d + d) * 4) + keep + BB.workspace_size(desc, 2)
    assert least < BB.workspace_size(desc, 0)
    torch.cuda.synchronize()
    with serve.Server(keep + least, max_slots=1, n_streams=1) as srv:
        assert srv.wait(srv.submit(desc, q, k, v, o)).state == serve.DONE
    if H > 1:
        assert torch.equal(o, la.forward(q, k, v))
    assert normwise(as64(o), oracle.forward(*host)) < TOL["fp32"]
