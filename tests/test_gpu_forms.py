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
# narrowest heads the last and first counts on either side of 2,048 tokens
# to a partial (64 partials)
SIZES = [(128, "fp32", n) for n in (31, 33, 128, 129, 300)] + [(64, "bf16", n) for n in (31, 127, 128, 129, 256, 257, 8193)] + \
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
