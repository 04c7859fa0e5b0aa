"""Performance cases of the library: calls that a program makes through the
public entry points, over the sizes, types and layouts they take.

A case is a dict of plain values.  `prepare` makes a program's inputs on the
GPU, `run` is one pass, `work` the bytes and operations a pass cannot do
without, `exact` the result in 64 bits by plain torch.

op       forward        la.forward
         train          la.linear_attention and its gradients (autograd)
         apply          la.apply: new queries against a kept summary
         apply_gated    la.apply_gated: the same, blended with another branch
         forward_gated  la.forward_gated
         tiled          la.tiled_forward: tiles with halos over a field
         serve          one ensemble request through serve.Server
layout   bhnd           [B, H, N, d] contiguous
         bnhd           views of a fused projection's [B, N, H, d]
"""
import math

import torch

import paper_2604_16590_amd as la
from paper_2604_16590_amd import serve

DEVICE = "cuda:0"


def _attn(name, op, B, H, N, d, dtype="bf16", layout="bhnd"):
    return {"name": name, "op": op, "B": B, "H": H, "N": N, "d": d, "dtype": dtype,
            "layout": layout}


def _tiled(name, dims, core, halo, H, d):
    return {"name": name, "op": "tiled", "T": dims[0], "Y": dims[1], "X": dims[2],
            "ct": core[0], "cy": core[1], "cx": core[2],
            "ht": halo[0], "hy": halo[1], "hx": halo[2], "H": H, "d": d, "dtype": "bf16"}


def listed():
    return [
        # the small fp32 problem: one head, where launches and latency count
        _attn("forward_small_fp32", "forward", 1, 1, 4096, 64, "fp32"),
        # a short ragged sequence trained through autograd: the smallest step
        _attn("train_small", "train", 1, 2, 1000, 128),
        # eight frames of the 32 x 64 patch grid, four ensemble members
        _attn("forward_grid", "forward", 4, 16, 16384, 64),
        # the fwd+bwd shape of 64 x 64 x 64 tokens
        _attn("train_frames", "train", 2, 16, 262144, 64),
        # the long-context step, 256 x 64 x 128 tokens: the largest
        _attn("train_long_context", "train", 1, 8, 2097152, 128),
        # the long-context heads in single precision, a quarter of the tokens
        _attn("train_long_fp32", "train", 1, 8, 524288, 128, "fp32"),
        # single precision at the grid's head size, ragged
        _attn("train_ragged_fp32", "train", 2, 16, 20011, 64, "fp32"),
        # one diffusion step of temporal cross-attention against a kept
        # history, gated into the spatial branch, on projection views
        _attn("apply_gated_step", "apply_gated", 8, 16, 32768, 64, "bf16", "bnhd"),
        # narrow heads on projection views, ragged
        _attn("train_narrow", "train", 4, 8, 30001, 32, "bf16", "bnhd"),
        # an ensemble request of 64 members through the server
        _attn("serve_request", "serve", 64, 16, 8192, 64),
        # the tiled step over 16 frames of the patch grid, ragged tiles
        _tiled("tiled_frames", (15, 32, 61), (4, 8, 16), (1, 2, 4), 8, 32),
        # the tiled step over the long-context field
        _tiled("tiled_long_context", (256, 64, 128), (8, 16, 16), (2, 4, 4), 16, 64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more call: types and head sizes by use, the work spread over its
    logarithm, most token counts odd."""
    op = rng.choice(["forward", "forward", "train", "train", "train", "apply", "apply_gated",
                     "forward_gated", "tiled", "tiled", "serve"])
    if op == "tiled":
        core = [rng.randint(3, 9), rng.randint(6, 18), rng.randint(6, 18)]
        halo = [rng.randint(0, c // 2) for c in core]
        dims = [_log_int(rng, 4, 100), rng.randint(16, 64), rng.randint(16, 96)]
        return {k: v for k, v in _tiled("", dims, core, halo, rng.choice([2, 4, 8, 16]),
                                        rng.choice([32, 64, 64])).items() if k != "name"}
    d = rng.choice([16, 32, 64, 64, 64, 128, 128])
    dtype = "bf16" if op == "serve" else rng.choice(["bf16", "bf16", "bf16", "fp32"])
    H = rng.choice([1, 2, 4, 8, 16])
    B = rng.choice([4, 16, 64]) if op == "serve" else rng.choice([1, 1, 2, 4, 8])
    elements = _log_int(rng, 1 << 18, 1 << (27 if dtype == "fp32" else 28))
    N = max(16, elements // (B * H * d))
    N = N if rng.random() < 0.25 else N | 1
    layout = "bhnd" if op == "serve" else rng.choice(["bhnd", "bhnd", "bnhd"])
    return {k: v for k, v in _attn("", op, B, H, N, d, dtype, layout).items() if k != "name"}


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _inputs(case, seed):
    """The tensors of a case, from the seed: queries, keys and values as a
    normalised projection leaves them, upstream gradients N(0, 1)."""
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    dt = _dtype(case)

    def normal(shape, std=1.0, dtype=dt):
        x = torch.empty(shape, dtype=dtype, device=DEVICE)
        return x.normal_(0.0, std, generator=gen)

    if case["op"] == "tiled":
        shape = (case["T"], case["Y"], case["X"], case["H"], case["d"])
        return {n: normal(shape) for n in ("q", "k", "v")}
    B, H, N, d = (case[n] for n in ("B", "H", "N", "d"))

    def tokens(std, length=N):
        if case["layout"] == "bnhd":
            return normal((B, length, H, d), std).permute(0, 2, 1, 3)
        return normal((B, H, length, d), std)

    std = math.sqrt(0.5)
    x = {"q": tokens(std)}
    if case["op"] in ("apply", "apply_gated"):
        # the history whose summary the program keeps
        hist = min(N, 4096)
        k, v = tokens(std, hist).double(), tokens(std, hist).double()
        f = _phi(k)
        x["S"] = torch.matmul(f.transpose(2, 3).contiguous(), v.contiguous())
        x["z"] = f.sum(2)
    else:
        x["k"], x["v"] = tokens(std), tokens(std)
    if case["op"] == "train":
        x["g"] = tokens(1.0)
    if case["op"] in ("apply_gated", "forward_gated"):
        x["other"] = tokens(std)
        # noise levels of a sampler, log-uniform over 0.02 .. 80
        x["sigma"] = torch.empty(B, dtype=torch.float64, device=DEVICE).uniform_(
            math.log(0.02), math.log(80.0), generator=gen).exp_()
    return x


class _Service:
    """A server and the buffers of one request, closed when dropped."""

    def __init__(self, case, x):
        B, H, N, d = (case[n] for n in ("B", "H", "N", "d"))
        self.server = serve.Server(2 << 30, max_slots=4, n_streams=4, max_slices_per_request=2)
        self.desc = serve.desc_for(B, H, N, d)
        self.x = x
        self.o = torch.empty_like(x["q"])

    def __del__(self):
        self.server.close()


def prepare(case, seed):
    x = _inputs(case, seed)
    op = case["op"]
    if op == "train":
        for n in ("q", "k", "v"):
            x[n].requires_grad_(True)
    elif op == "serve":
        torch.cuda.synchronize()  # the server reads the inputs on its own streams
        x = {"service": _Service(case, x)}
    elif op != "tiled":
        # the caller's output buffer, in the layout of its tensors
        x["out"] = torch.empty_like(x["q"])
    x["case"] = case
    return x


def run(state):
    case = state["case"]
    op = case["op"]
    if op == "train":
        q, k, v = state["q"], state["k"], state["v"]
        o = la.linear_attention(q, k, v)
        dq, dk, dv = torch.autograd.grad(o, (q, k, v), state["g"])
        return {"o": o.detach(), "dq": dq, "dk": dk, "dv": dv}
    if op == "forward":
        return la.forward(state["q"], state["k"], state["v"], out=state["out"])
    if op == "apply":
        return la.apply(state["q"], state["S"], state["z"], out=state["out"])
    if op == "apply_gated":
        return la.apply_gated(state["q"], state["S"], state["z"], state["other"], state["sigma"],
                              out=state["out"])
    if op == "forward_gated":
        return la.forward_gated(state["q"], state["k"], state["v"], state["other"],
                                state["sigma"], out=state["out"])
    if op == "tiled":
        return la.tiled_forward(state["q"], state["k"], state["v"],
                                (case["ct"], case["cy"], case["cx"]),
                                (case["ht"], case["hy"], case["hx"]))
    s = state["service"]
    rid = s.server.submit(s.desc, s.x["q"], s.x["k"], s.x["v"], s.o)
    r = s.server.wait(rid)
    if r.state != serve.DONE:
        raise RuntimeError("request failed (%d)" % r.error)
    s.server.release(rid)
    return s.o


def work(case):
    """Each tensor read or written once; two operations a product: q.S and
    phi(k) v in the forward; S g, phi(q) g, phi(k) dS and v dS on the way
    back.  (The tiles' halos are left out.)"""
    es = 2 if case["dtype"] == "bf16" else 4
    H, d = case["H"], case["d"]
    if case["op"] == "tiled":
        e = case["T"] * case["Y"] * case["X"] * H * d
        return {"bytes": 4 * e * es, "flops": 4 * e * d}
    e = case["B"] * case["N"] * H * d
    tensors, products = {"forward": (4, 2), "serve": (4, 2), "train": (8, 6), "apply": (2, 1),
                         "apply_gated": (3, 1), "forward_gated": (5, 2)}[case["op"]]
    size = tensors * e * es
    if case["op"] in ("apply", "apply_gated"):
        size += case["B"] * H * (d * d + d) * 8
    return {"bytes": size, "flops": 2 * products * e * d}


def _phi(x):
    return torch.where(x > 0, x + 1, torch.exp(x))


def _dphi(x):
    return torch.where(x > 0, torch.ones_like(x), torch.exp(x))


def _exact_tiled(case, x):
    """Every tile's attention over its extended, border-clamped tokens, and
    the Hann-weighted average of the tiles covering each position."""
    dims = [case[n] for n in ("T", "Y", "X")]
    core = [case[n] for n in ("ct", "cy", "cx")]
    halo = [case[n] for n in ("ht", "hy", "hx")]
    H, d = case["H"], case["d"]
    flat = {n: t.view(-1, H, d) for n, t in x.items()}
    num = torch.zeros(dims[0] * dims[1] * dims[2], H, d, dtype=torch.float64, device=DEVICE)
    wsum = torch.zeros(num.shape[0], dtype=torch.float64, device=DEVICE)

    def axis(k, j):
        """Clamped coordinates of tile j's range, which lie inside, weights."""
        L = core[k] + 2 * halo[k]
        u = torch.arange(L, device=DEVICE)
        p = j * core[k] - halo[k] + u
        w = torch.sin(math.pi * (u.double() + 0.5) / L) ** 2
        inside = (p >= 0) & (p < dims[k])
        return p.clamp(0, dims[k] - 1), torch.where(inside, w, torch.zeros_like(w))

    counts = [-(-n // c) for n, c in zip(dims, core)]
    for a in range(counts[0]):
        pt, wt = axis(0, a)
        for b in range(counts[1]):
            py, wy = axis(1, b)
            for c in range(counts[2]):
                px, wx = axis(2, c)
                at = ((pt[:, None, None] * dims[1] + py[None, :, None]) * dims[2]
                      + px[None, None, :]).reshape(-1)
                w = (wt[:, None, None] * wy[None, :, None] * wx[None, None, :]).reshape(-1)
                q, k, v = (flat[n][at].double().permute(1, 0, 2).contiguous() for n in "qkv")
                fk, fq = _phi(k), _phi(q)
                S = torch.matmul(fk.transpose(1, 2).contiguous(), v)
                o = torch.matmul(fq, S) / torch.matmul(fq, fk.sum(1)[:, :, None])
                # positions outside the grid have weight 0, and a clamped
                # index repeats: index_add_ takes both
                num.index_add_(0, at, o.permute(1, 0, 2) * w[:, None, None])
                wsum.index_add_(0, at, w)
    return num.div_(wsum[:, None, None]).view(dims + [H, d])


def exact(case, seed):
    x = _inputs(case, seed)
    op = case["op"]
    if op == "tiled":
        return _exact_tiled(case, x)
    B, H = case["B"], case["H"]
    names = ("o", "dq", "dk", "dv") if op == "train" else ("o",)
    res = {n: torch.empty(x["q"].shape, dtype=torch.float64, device=DEVICE) for n in names}
    for b in range(B):
        for h in range(H):
            q = x["q"][b, h].double()
            fq = _phi(q)
            if "S" in x:
                S, z = x["S"][b, h], x["z"][b, h]
            else:
                k, v = x["k"][b, h].double(), x["v"][b, h].double()
                fk = _phi(k)
                S, z = fk.t().contiguous() @ v, fk.sum(0)
            den = (fq @ z)[:, None]
            o = (fq @ S) / den
            if op == "train":
                g = x["g"][b, h].double()
                dnum = g / den
                dden = -(g * o).sum(1, keepdim=True) / den
                res["dq"][b, h] = (dnum @ S.t().contiguous() + dden * z) * _dphi(q)
                dS, dz = fq.t().contiguous() @ dnum, (fq * dden).sum(0)
                res["dv"][b, h] = fk @ dS
                res["dk"][b, h] = (v @ dS.t().contiguous() + dz) * _dphi(k)
                del g, dnum, dden
            if "sigma" in x:
                w = 0.5 / (0.5 + x["sigma"][b])
                o = w * o + (1 - w) * x["other"][b, h].double()
            res["o"][b, h] = o
    return res if op == "train" else res["o"]
