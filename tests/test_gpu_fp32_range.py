"""fp32 inputs at the edges of the range in which they split into bf16 parts:
products beyond fp32, and columns, rows and tokens of very small values
beside ordinary ones, each to the fp32 path's own relative accuracy.

Small values lie in [2^-122, 2^-119]: normal in fp32, while a three-part bf16
split keeps them to 2^-134 at best, 2^-12 of the value.  Tolerance 1e-5 as
for all fp32 results, against the definition in 64 bits (phi as the kernels
define it: exp2 of the fp32 product x log2(e))."""
import numpy as np
import pytest
import torch

import paper_2604_16590_amd as la
from gpu_util import as64, make_inputs, normwise, require_gpu, to_device

pytestmark = pytest.mark.gpu

TINY = 2.0 ** -122
TOL = 1e-5
N = 300


def phi(x):
    f = np.exp2((x * np.float32(1.44269504)).astype(np.float64))
    return np.where(x > 0, x.astype(np.float64) + 1, f)


def tiny(rng, shape):
    """Random signs, magnitudes 1 to 4 TINY."""
    return (TINY * rng.uniform(1, 4, shape) * rng.choice([-1.0, 1.0], shape)).astype(np.float32)


def inputs(d):
    q, k, v, g = make_inputs((1, 2, N, d), "fp32", seed=90 + d, streams=(0, 1, 2, 3))
    return q, k, v, g, np.random.default_rng(d)


@pytest.mark.parametrize("d", [16, 32, 64, 128])
def test_products_beyond_fp32_are_infinite(d):
    dev = require_gpu()
    big = 1.005 * 2.0 ** 70  # its first bf16 part lies above it
    q, k, v, _, _ = inputs(d)
    k[:] = 2.0 ** 70
    v[:] = big
    tq, tk, tv = (to_device(x, dev) for x in (q, k, v))
    _, S, z = la.forward(tq, tk, tv, return_summary=True)
    torch.cuda.synchronize()
    assert torch.isposinf(S).all() and torch.isfinite(z).all()


@pytest.mark.parametrize("d", [16, 32, 64, 128])
def test_small_columns_of_the_summary(d):
    dev = require_gpu()
    q, k, v, _, rng = inputs(d)
    v[..., 3] = tiny(rng, v.shape[:3])
    k[..., 2] = rng.uniform(-85, -84, k.shape[:3])  # phi = 2^-122.6 .. 2^-121.2
    _, S, _ = la.forward(*(to_device(x, dev) for x in (q, k, v)), return_summary=True)
    torch.cuda.synchronize()
    S = S.cpu().numpy()
    ref = np.matmul(np.swapaxes(phi(k), 2, 3), v.astype(np.float64))
    c = np.arange(d) != 2
    assert normwise(S[:, :, c, 3], ref[:, :, c, 3]) < TOL
    e = np.arange(d) != 3
    assert normwise(S[:, :, 2, e], ref[:, :, 2, e]) < TOL
    assert normwise(S[:, :, c][..., e], ref[:, :, c][..., e]) < TOL


@pytest.mark.parametrize("d", [16, 32, 64, 128])
def test_small_tokens_and_columns_of_the_apply(d):
    dev = require_gpu()
    q, k, v, _, rng = inputs(d)
    q[:, :, 40:43] = rng.uniform(-85, -84, (1, 2, 3, d))
    S = rng.standard_normal((1, 2, d, d))
    S[..., 3] = tiny(rng, (1, 2, d))
    z = rng.uniform(1, 2, (1, 2, d))
    o = as64(la.apply(to_device(q, dev), *(torch.from_numpy(x).to(dev) for x in (S, z))))
    f = phi(q)
    ref = np.matmul(f, S) / np.matmul(f, z[..., None])
    e = np.arange(d) != 3
    for t in (slice(0, 40), slice(40, 43), slice(43, N)):
        assert normwise(o[:, :, t][..., e], ref[:, :, t][..., e]) < TOL
        if t.start != 40:  # (a small token's products with a small column are below fp32)
            assert normwise(o[:, :, t, 3], ref[:, :, t, 3]) < TOL


@pytest.mark.parametrize("d", [16, 32, 64, 128])
def test_small_rows_and_columns_of_the_backward(d):
    dev = require_gpu()
    q, k, v, g, rng = inputs(d)
    g[..., 3] = tiny(rng, g.shape[:3])
    S = rng.standard_normal((1, 2, d, d))
    S[:, :, 2] = tiny(rng, (1, 2, d))
    z = rng.uniform(1, 2, (1, 2, d)) / d
    z[..., 2] = 0  # so that row of dQ is that row of S G alone
    dq, _, dv = la.backward(*(to_device(x, dev) for x in (q, k, v)),
                            *(torch.from_numpy(x).to(dev) for x in (S, z)), to_device(g, dev))
    dq, dv = as64(dq), as64(dv)
    f, G = phi(q), g.astype(np.float64)
    Gd = G / np.matmul(f, z[..., None])
    dphi = np.minimum(f, 1)
    dq_ref = np.matmul(Gd, np.swapaxes(S, 2, 3))[..., 2] * dphi[..., 2]
    assert normwise(dq[..., 2], dq_ref) < TOL
    dv_ref = np.matmul(phi(k), np.matmul(np.swapaxes(f, 2, 3), Gd))
    e = np.arange(d) != 3
    assert normwise(dv[..., 3], dv_ref[..., 3]) < TOL
    assert normwise(dv[..., e], dv_ref[..., e]) < TOL
