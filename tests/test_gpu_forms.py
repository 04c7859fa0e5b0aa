"""The kernels' forms at the sizes and values where they change: a workgroup or a wave
to a partial, the ragged ends of a workgroup's steps, fp32 values that leave
the range of the bf16 split.

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
# narrowest heads the last and first counts of one wave to a partial of 2,048 tokens
# (64 partials); the longest sequence of four waves to a partial and one more
SIZES = [(128, "fp32", n) for n in (31, 33, 128, 129, 300)] + [(64, "bf16", n) for n in (31, 127, 128, 129, 256, 257, 8193)] + \
        [(64, "fp32", n) for n in (15, 63, 65, 128, 129, 8193)] + \
        [(128, "bf16", n) for n in (127, 129, 512, 513)] + \
        [(64, "bf16", 64 * 512), (64, "bf16", 64 * 512 + 1)] + \
        [(16, "bf16", 64 * 2048), (16, "bf16", 64 * 2048 + 1), (32, "fp32", 5 * 64 + 1)]


@pytest.mark.parametrize("d,dtype,N", SIZES)
def test_summary_forms(d, dtype, N):
    dev = require_gpu()
    B, H = (1, 1) if N > 30000 else (3, 3)  # nine items: not a multiple of eight
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


# a wave to a partial's run or to the whole partial, run after run: the same
# bits from one head, from many, and from views in which heads share cache
# lines; two runs of a partial and its last partial's one, whole and ragged
@pytest.mark.parametrize("d,heads,N", [
    (16, 8, 4097), (16, 8, 33001), (16, 4, 300000), (32, 130, 4097), (32, 40, 33001), (32, 36, 64 * 2048),
    (64, 16, 32769), (64, 16, 40001), (64, 14, 64 * 2048 + 65)])
def test_summary_runs(d, heads, N):
    dev = require_gpu()
    gen = torch.Generator(device=dev).manual_seed(N)
    q, k, v = (torch.randn((1, heads, N, d), generator=gen, device=dev).bfloat16() for _ in range(3))
    views = [x.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) for x in (q, k, v)]
    last = [x[:, heads - 1:] for x in (q, k, v)]
    o, S, z = la.forward(q, k, v, return_summary=True)
    ov, Sv, zv = la.forward(*views, return_summary=True)
    o1, S1, z1 = la.forward(*last, return_summary=True)
    torch.cuda.synchronize()
    assert torch.equal(S, Sv) and torch.equal(z, zv) and torch.equal(o, ov)
    assert torch.equal(S[:, heads - 1:], S1) and torch.equal(z[:, heads - 1:], z1) and torch.equal(o[:, heads - 1:], o1)
    host = [x.float().cpu().numpy() for x in last]
    o_ref, S_ref, z_ref = oracle.forward(*host, want_summary=True)
    assert normwise(as64(o1), o_ref) < TOL["bf16"]
    assert normwise(S1.cpu().numpy(), S_ref) < 4e-3
    assert normwise(z1.cpu().numpy()[..., None], z_ref[..., None]) < 4e-3


@pytest.mark.parametrize("N", [257, 4097, 20001, 200001])
def test_summary_runs_fp32(N):
    # d = 16, forward and the backward's reduction
    dev = require_gpu()
    host = make_inputs((1, 2, N, 16), "fp32", seed=N, streams=(0, 1, 2, 3))
    q, k, v, g = (to_device(x, dev) for x in host)
    o, S, z = la.forward(q, k, v, return_summary=True)
    got = la.backward(q, k, v, S, z, g)
    torch.cuda.synchronize()
    o_ref, S_ref, z_ref = oracle.forward(*host[:3], want_summary=True)
    assert normwise(as64(o), o_ref) < TOL["fp32"]
    assert normwise(S.cpu().numpy(), S_ref) < 1e-5 and normwise(z.cpu().numpy()[..., None], z_ref[..., None]) < 1e-6
    for x, r in zip(got, oracle.backward(*host)):
        assert normwise(as64(x), r) < TOL["fp32"]


@pytest.mark.parametrize("d", [16, 32, 64, 128])
@pytest.mark.parametrize("kind", ["tiny_v", "tiny_k", "huge_v", "inf_v", "nan_v", "inf_k", "nan_k", "zeros"])
def test_fp32_extremes(kind, d):
    # values outside the range in which fp32 splits into bf16 parts, and
    # non-finite ones: the summary is the fp32 one, with the same infinities
    # and NaNs as the definition gives
    dev = require_gpu()
    N = 700
    q, k, v = make_inputs((1, 2, N, d), "fp32", seed=77)
    if kind == "tiny_v":
        v *= np.float32(1e-33)
    elif kind == "tiny_k":
        k -= np.float32(76)  # phi ~ 1e-33
    elif kind == "huge_v":
        v[0, 0, 3::160] *= np.float32(1e34)
        v[0, 0, 5, 1] = np.finfo(np.float32).max  # rounds to infinity in bf16
    elif kind == "inf_v":
        v[0, 1, 333, 5] = np.inf
        v[0, 1, 600, 7] = -np.inf
    elif kind == "nan_v":
        v[0, 1, 333, 5] = np.nan
    elif kind == "inf_k":
        k[0, 0, 20, 4] = np.inf
        k[0, 1, 21] = -np.inf
    elif kind == "nan_k":
        k[0, 0, 20, 4] = np.nan
    else:
        v[:, :, 100:400] = 0
    tq, tk, tv = (to_device(x, dev) for x in (q, k, v))
    _, S, z = la.forward(tq, tk, tv, return_summary=True)
    torch.cuda.synchronize()
    K, V = k.astype(np.float64), v.astype(np.float64)
    with np.errstate(all="ignore"):
        # phi as the kernels define it: exp2 of the fp32 product x log2(e),
        # whose rounding is |x| log2(e) 2^-24 of phi (6e-6 at -76)
        f = np.exp2((k * np.float32(1.44269504)).astype(np.float64))
        f = np.where(K > 0, K + 1, f)
        S_ref = np.matmul(np.swapaxes(f, 2, 3), V)
        z_ref = f.sum(2)
        # the partial sums are fp32: beyond its largest value, infinite
        S_ref = np.where(np.abs(S_ref) > np.finfo(np.float32).max, np.copysign(np.inf, S_ref), S_ref)
    for got, ref, tol in ((S.cpu().numpy(), S_ref, 1e-5), (z.cpu().numpy()[..., None], z_ref[..., None], 1e-6)):
        ok = np.isfinite(ref)
        assert np.array_equal(np.isnan(got), np.isnan(ref))
        assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
        assert normwise(np.where(ok, got, 0), np.where(ok, ref, 0)) < tol


# tokens: one 16-token tile and its neighbours; a workgroup's block (d = 128:
# eight waves, 64: four; two tiles a wave in the apply) and its neighbours
@pytest.mark.parametrize("d,N", [(d, n) for d in (64, 128) for n in (1, 15, 17, 127, 129, 255, 257, 1100)])
@pytest.mark.parametrize("out", ["fp32", "bf16"])
def test_fp32_rows(d, N, out):
    # the fp32 row kernels against the oracle, with the gated apply, on
    # views of [B, N, H, d] storage
    dev = require_gpu()
    B, H = 2, 3
    od = torch.float32 if out == "fp32" else torch.bfloat16
    host = make_inputs((B, H, N, d), "fp32", seed=900 + N + d, streams=(0, 1, 2, 3))
    view = lambda dt: torch.empty((B, N, H, d), dtype=dt, device=dev).permute(0, 2, 1, 3)
    q, k, v, g = (view(torch.float32).copy_(to_device(x, dev)) for x in host)
    o, S, z = la.forward(q, k, v, out=view(od), return_summary=True)
    dq, dk, dv = la.backward(q, k, v, S, z, g, grad_dtype=od)
    other = view(od).copy_(to_device(make_inputs((B, H, N, d), "fp32", seed=901)[0], dev))
    sigma = torch.tensor([0.3, 4.0], dtype=torch.float64, device=dev)
    mixed = la.apply_gated(q, S, z, other, sigma, out=view(od))
    torch.cuda.synchronize()
    tol = TOL[out]
    ref = oracle.forward(*host[:3])
    assert normwise(as64(o), ref) < tol
    w = (0.5 / (0.5 + np.array([0.3, 4.0])))[:, None, None, None]
    assert normwise(as64(mixed), w * ref + (1 - w) * as64(other)) < tol
    grads = oracle.backward(*host)
    if N == 1:  # the gradients of q and k vanish
        grads, got = grads[2:], (dv,)
    else:
        got = (dq, dk, dv)
    for x, r in zip(got, grads):
        assert normwise(as64(x), r) < tol


@pytest.mark.parametrize("d", [64, 128])
def test_fp32_rows_outside_the_split_range(d):
    # scales below the split's range take the fp32 instructions: the
    # problem is linear in v and in the upstream gradient, so scaling
    # either by 2^-100 scales the results, to rounding
    dev = require_gpu()
    host = make_inputs((1, 2, 333, d), "fp32", seed=41, streams=(0, 1, 2, 3))
    q, k, v, g = (to_device(x, dev) for x in host)
    c = 2.0 ** -100
    o, S, z = la.forward(q, k, v, return_summary=True)
    grads = la.backward(q, k, v, S, z, g)
    o1, S1, z1 = la.forward(q, k, v * c, return_summary=True)
    grads_v = la.backward(q, k, v * c, S1, z1, g)
    grads_g = la.backward(q, k, v, S, z, g * c)
    # a few of a tile's tokens outside the range, the rest as they were
    q2 = q.clone()
    q2[:, :, 40:43] = -75.0  # phi ~ 2^-108
    o2 = la.forward(q2, k, v)
    torch.cuda.synchronize()
    assert normwise(as64(o1) / c, as64(o)) < 1e-5
    for i, name in enumerate(("dq", "dk", "dv")):
        assert normwise(as64(grads_g[i]) / c, as64(grads[i])) < 1e-5, name
    assert normwise(as64(grads_v[0]) / c, as64(grads[0])) < 1e-5
    assert normwise(as64(grads_v[2]), as64(grads[2])) < 1e-5
    keep = np.r_[0:40, 43:333]
    assert normwise(as64(o2)[:, :, keep], as64(o)[:, :, keep]) < 1e-5
    mean = as64(S).sum(2) / as64(z).sum(2)[..., None]  # equal weights
    assert normwise(as64(o2)[:, :, 41], mean) < 1e-5


# the fused query backward: one 32-token block of a wave and its neighbours,
# a partial's end, heads that share cache lines (views of [B, N, H, d])
@pytest.mark.parametrize("d,N", [(d, n) for d in (16, 32, 64, 128) for n in (31, 33, 127, 129, 513, 2049)])
@pytest.mark.parametrize("layout", ["bhnd", "bnhd"])
def test_backward_forms(layout, d, N):
    dev = require_gpu()
    B, H = 1, 5
    host = make_inputs((B, H, N, d), "bf16", seed=300 + N + d, streams=(0, 1, 2, 3))
    q, k, v, g = (to_device(x, dev) for x in host)
    if layout == "bnhd":
        q, k, v, g = (x.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) for x in (q, k, v, g))
    _, S, z = la.forward(q, k, v, return_summary=True)
    got = la.backward(q, k, v, S, z, g)
    torch.cuda.synchronize()
    for x, r in zip(got, oracle.backward(*host)):
        assert normwise(as64(x), r) < TOL["bf16"]
    # the last head alone: the same bits
    one = [x[:, H - 1:] for x in (q, k, v, S, z, g)]
    alone = la.backward(*one)
    torch.cuda.synchronize()
    for x, y in zip(got, alone):
        assert torch.equal(x[:, H - 1:], y)


# up to four partials (d <= 32: sixteen) are added up by the workgroups that
# need them (one head), or by a pass before where many workgroups would read
# them: the same bits
@pytest.mark.parametrize("d,heads,partials", [
    (d, h, p) for d, h in ((16, 1100), (32, 300), (64, 130), (128, 66)) for p in (1, 2, 3, 4)] + [
    (d, 300, p) for d in (16, 32) for p in (5, 7, 12, 16)])
def test_partials_added_up_by_their_readers(partials, d, heads):
    dev = require_gpu()
    N = 4 * d * partials
    gen = torch.Generator(device=dev).manual_seed(d + partials)
    q, k, v, g = (torch.randn((1, heads, N, d), generator=gen, device=dev).bfloat16() for _ in range(4))
    o, S, z = la.forward(q, k, v, return_summary=True)
    got = la.backward(q, k, v, S, z, g)
    last = [x[:, heads - 1:] for x in (q, k, v)]
    o1, S1, z1 = la.forward(*last, return_summary=True)
    got1 = la.backward(*last, S1, z1, g[:, heads - 1:])
    o2 = la.apply(last[0], S1, z1)
    torch.cuda.synchronize()
    for x, y in zip((o, S, z, o) + tuple(got), (o1, S1, z1, o2) + tuple(got1)):
        assert torch.equal(x[:, heads - 1:], y)
    host = [x.float().cpu().numpy() for x in last + [g[:, heads - 1:]]]
    assert normwise(as64(o1), oracle.forward(*host[:3])) < TOL["bf16"]
    for x, r in zip(got1, oracle.backward(*host)):
        assert normwise(as64(x), r) < TOL["bf16"]


# the tiled step where its kernels change: footprints of 512 positions and
# one more (offsets kept in LDS or not), cells longer than the window table,
# a cell's last 16-token tile, one position per cell row
@pytest.mark.parametrize("dims,core,halo,H,d", [
    ((3, 16, 64), (2, 16, 32), (1, 0, 0), 2, 32), ((3, 16, 66), (2, 16, 33), (1, 0, 0), 2, 32),
    ((1, 1, 3300), (1, 1, 3300), (0, 0, 40), 2, 16), ((1, 3, 3000), (1, 2, 1500), (0, 1, 700), 1, 32),
    ((5, 7, 3), (2, 3, 1), (1, 1, 0), 3, 64), ((9, 4, 17), (3, 4, 16), (1, 2, 8), 1, 64)])
def test_tiled_forms(dims, core, halo, H, d):
    from test_gpu_tiles import oracle_tiled
    dev = require_gpu()
    q, k, v = make_inputs((1, 1, dims[0] * dims[1] * dims[2], H * d), "bf16", seed=60)
    shape = tuple(dims) + (H, d)
    o = la.tiled_forward(*(to_device(x, dev).view(shape) for x in (q, k, v)), core, halo)
    torch.cuda.synchronize()
    flat = tuple(dims) + (H * d,)
    ref = oracle_tiled(*(x.reshape(flat) for x in (q, k, v)), dims, core, halo, H, d)
    assert normwise(as64(o).reshape(1, 1, -1), ref.reshape(1, 1, -1)) < TOL["bf16"]


# a workspace smaller than la_workspace_size: parts of the heads, one after the
# other, with the same bits and nothing written beyond it
@pytest.mark.parametrize("layout", ["bhnd", "bnhd"])
@pytest.mark.parametrize("d,dtype,N", [(128, "fp32", 3849), (16, "bf16", 963)])
@pytest.mark.parametrize("B,H,room", [(1, 3, (1, 1)), (1, 5, (1, 2)), (3, 2, (2, 2)), (3, 2, (1, 2))])
def test_small_workspace(B, H, room, d, dtype, N, layout):
    import ctypes
    from paper_2604_16590_amd import _binding as BB
    dev = require_gpu()
    host = make_inputs((B, H, N, d), dtype, seed=9, streams=(0, 1, 2, 3))
    q, k, v, g = (to_device(x, dev) for x in host)
    if layout == "bnhd":
        q, k, v, g = (x.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) for x in (q, k, v, g))
    sigma = torch.linspace(0.1, 2.0, B, dtype=torch.float64, device=dev)
    want = la.forward_gated(q, k, v, g, sigma, out=torch.empty_like(q), return_summary=True)
    grads = la.backward(q, k, v, want[1], want[2], g)
    desc = BB.make_desc(q, want[0])
    small = BB.AttnDesc(room[0], room[1], *[getattr(desc, f) for f, _ in BB.AttnDesc._fields_[2:]])
    got = [torch.full_like(x, float("nan")) for x in want]
    ggot = [torch.full_like(x, float("nan")) for x in grads]
    gdesc = BB.make_desc(q, grads[0])
    st = BB._stream(q.device)

    def call(pass_, nbytes, ws):
        if pass_ == 0:
            return BB.lib().la_forward_gated(
                ctypes.byref(desc), q.data_ptr(), k.data_ptr(), v.data_ptr(), g.data_ptr(), sigma.data_ptr(),
                0.5, got[0].data_ptr(), got[1].data_ptr(), got[2].data_ptr(), ws.data_ptr(), nbytes, st)
        return BB.lib().la_backward(
            ctypes.byref(gdesc), q.data_ptr(), k.data_ptr(), v.data_ptr(), want[1].data_ptr(), want[2].data_ptr(),
            g.data_ptr(), *[x.data_ptr() for x in ggot], ws.data_ptr(), nbytes, st)

    up = lambda n: -(-n // 256) * 256
    parts = -(-N // (2048 if d == 128 else 512))  # the least: a partial for so many tokens
    images = BB.workspace_size(desc, 2)
    least = up(B * H * parts * (d * d + d) * 4) + up(B * H * d * d * 8) + up(B * H * d * 8) + images
    stash = up(B * H * N * 8)
    for pass_, low in ((0, least), (1, least + stash + images)):
        nbytes = max(BB.workspace_size(small, pass_), low)
        assert nbytes < BB.workspace_size(desc, pass_)
        ws = torch.zeros(nbytes + 4096, dtype=torch.uint8, device=dev)
        ws[nbytes:] = 0xA5
        assert call(pass_, nbytes, ws) == 0
        torch.cuda.synchronize()
        assert bool((ws[nbytes:] == 0xA5).all())
        assert call(pass_, low - 256, ws) == 3  # LA_ERR_OOM
    for x, y in zip(tuple(want) + tuple(grads), got + ggot):
        assert torch.equal(x, y)
