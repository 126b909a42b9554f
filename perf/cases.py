"""Performance cases: what a program that uses this library has it do, through its Python entry points.

A case is a dict of plain values:

    path    "infer"  one forward call (out, lse): encoding, prefill, or a few new queries against
                     many keys when M is given (cross-attention, decode)
            "train"  one differentiable call and its backward (out and every gradient)
    bias    "factors"  low-rank factors phi_q, phi_k
            "alibi"    rank-2 ALiBi factors (infer) or trained head slopes (train)
            "distance" exact rank-9 squared-distance factors of 3-D points with trained weights
            "relpos"   smooth relative-position bias on a square grid, two columns a frequency
            "dense"    a materialised bias shared over the batch
            "cosmul"   the multiplicative bias cos(i - j) as rank-2 factors
    dtype   "bf16" or "f32" storage of q, k, v, out;  phi: storage of the factors
    B, H, N, M (keys; 0: as many as queries), C, R, causal, shared (factors shared over the batch)
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2505_12044_amd import api, autograd, workloads


def _case(path, bias, B, H, N, C, R, dtype="bf16", phi="bf16", causal=False, shared=True, M=0):
    return {"path": path, "bias": bias, "B": B, "H": H, "N": N, "M": M, "C": C, "R": R, "dtype": dtype, "phi": phi,
            "causal": causal, "shared": shared}


def listed():
    cases = {
        # the smallest call: a short full-precision forward, where the launch and one pass over the keys are everything
        "tiny_fp32_infer": _case("infer", "factors", 1, 2, 256, 64, 4, "f32", "f32", shared=False),
        # full-precision training of a small model, ragged length
        "fp32_train": _case("train", "factors", 2, 8, 1500, 64, 8, "f32", "f32"),
        # a decoder reads a batch of prompts
        "alibi_prefill": _case("infer", "alibi", 4, 16, 4096, 128, 2, phi="f32", causal=True),
        # the same decoder makes its next token for a batch of cached sequences
        "alibi_decode": _case("infer", "alibi", 8, 16, 1, 128, 2, phi="f32", M=4096),
        # the same decoder is trained, slopes included
        "alibi_train": _case("train", "alibi", 4, 16, 4096, 128, 2, phi="f32", causal=True),
        # a vision model's window attention is trained with factors in the place of its bias table
        "vision_train": _case("train", "relpos", 8, 12, 1024, 64, 32),
        # the same model with the materialised bias
        "dense_train": _case("train", "dense", 8, 12, 1024, 64, 0),
        # triangle attention over the rows of a pair representation: inference, then training
        "pairformer_infer": _case("infer", "factors", 384, 4, 384, 32, 16),
        "pairformer_train": _case("train", "factors", 384, 4, 384, 32, 16),
        # one long-sequence training step, the largest call
        "long_train": _case("train", "factors", 2, 8, 16384, 128, 8, shared=False),
        # attention over a point cloud with a distance bias (an odd number of points, 16 channels)
        "pde_train": _case("train", "distance", 1, 8, 32186, 16, 9, phi="f32"),
        # multiplicative bias
        "mul_train": _case("train", "cosmul", 4, 16, 4096, 64, 2, phi="f32", causal=False),
    }
    return [dict(c, name=n) for n, c in cases.items()]


# ---- sizes ---------------------------------------------------------------------------------------
def _log(rng, lo, hi):
    """A whole number between lo and hi, spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _pairs(c):
    n, m = c["N"], c["M"] or c["N"]
    return c["B"] * c["H"] * (n * (n + 1) // 2 if c["causal"] else n * m)


def _flops(c):
    C, R = c["C"], c["R"]
    if c["bias"] == "cosmul":               # scores of C R channels, values of C
        fwd, bwd = 2 * (C * R + C), 2 * (3 * C * R + 2 * C)
    else:
        fwd, bwd = 2 * (2 * C + R), 2 * (5 * C + 3 * R)
    return float(_pairs(c)) * (fwd if c["path"] == "infer" else fwd + bwd)


def draw(rng):
    kind = rng.choice(("infer", "infer", "decode", "train", "train", "cross_train", "alibi_train", "dense_train",
                       "mul_train", "f32_infer", "f32_train"))
    H = rng.choice((1, 2, 4, 8, 12, 16))
    B = _log(rng, 1, 64)
    C = rng.choice((16, 32, 64, 128))
    phi = rng.choice(("bf16", "f32"))
    R = rng.choice((2, 3, 5, 9)) if phi == "f32" else rng.choice((4, 8, 16, 32, 50, 64))
    causal = rng.random() < 0.4
    shared = rng.random() < 0.6
    if kind == "infer":
        if rng.random() < 0.3:
            c = _case("infer", "alibi", B, H, _log(rng, 64, 16384), rng.choice((64, 128)), 2, phi="f32", causal=True)
        else:
            c = _case("infer", "factors", B, H, _log(rng, 64, 16384), C, R, phi=phi, causal=causal, shared=shared)
    elif kind == "decode":                   # one to a few new queries, up to 16384 keys
        c = _case("infer", "alibi", _log(rng, 1, 32), H, rng.choice((1, 1, 1, 2, 4, 8)), rng.choice((64, 128)), 2, phi="f32",
                  M=_log(rng, 256, 16384))
    elif kind == "train":
        bias = rng.choice(("factors", "factors", "relpos", "distance"))
        N = _log(rng, 64, 8192)
        if bias == "relpos":
            side = _log(rng, 8, 48)
            c = _case("train", "relpos", B, H, side * side, rng.choice((32, 64)), rng.choice((8, 16, 32)))
        elif bias == "distance":
            c = _case("train", "distance", 1, H, _log(rng, 500, 32186), rng.choice((16, 32)), 9, phi="f32")
        else:
            c = _case("train", "factors", B, H, N, C, R, phi=phi, causal=causal, shared=shared)
    elif kind == "cross_train":
        N, M = _log(rng, 32, 4096), _log(rng, 64, 8192)
        c = _case("train", "factors", B, H, N, C, R, phi=phi, shared=shared, M=M + (M == N))
    elif kind == "alibi_train":
        c = _case("train", "alibi", B, H, _log(rng, 64, 8192), rng.choice((64, 128)), 2, phi="f32", causal=True)
    elif kind == "dense_train":              # the bf16 backward takes lengths in steps of eight
        c = _case("train", "dense", _log(rng, 1, 8), H, 8 * _log(rng, 8, 256), rng.choice((32, 64, 128)), 0, causal=causal)
    elif kind == "mul_train":
        c = _case("train", "cosmul", B, H, _log(rng, 64, 4096), rng.choice((16, 32, 64)), 2, phi="f32", causal=causal)
    else:                                    # full precision: small models and checks
        c = _case("infer" if kind == "f32_infer" else "train", "factors", _log(rng, 1, 8), H, _log(rng, 64, 2048), C,
                  rng.choice((2, 4, 8, 16, 32)), "f32", "f32", causal=causal, shared=shared)
    # no drawn case costs more than the largest listed one: the batch shrinks first, then the heads, then the length
    limit = 3e10 if c["dtype"] == "f32" else (5e11 if c["bias"] == "distance" or c["C"] == 16 else 2e12)
    while _flops(c) > limit:
        if c["B"] > 1:
            c["B"] = (c["B"] + 1) // 2
        elif c["H"] > 1:
            c["H"] = (c["H"] + 1) // 2
        else:
            c["N"] = c["N"] // 2 // 8 * 8
    return c


# ---- inputs --------------------------------------------------------------------------------------
_DT = {"bf16": torch.bfloat16, "f32": torch.float32}


def _factors(c, seed, g):
    """phi_q, phi_k of the case's bias, float32 on the GPU, [1 or B, H, N or M, R]."""
    B, H, N, R = c["B"], c["H"], c["N"], c["R"]
    M = c["M"] or N
    dev = g.device
    Bp = 1 if c["shared"] else B
    if c["bias"] == "alibi":
        m = torch.tensor(workloads.alibi_slopes_f32(H), device=dev).view(1, H, 1)
        pq = (torch.arange(N, device=dev, dtype=torch.float32) + (M - N)).view(1, 1, N)      # the queries are the last positions
        pk = torch.arange(M, device=dev, dtype=torch.float32).view(1, 1, M).expand(1, H, M)
        return torch.stack((-m * pq, m.expand(1, H, N)), -1).contiguous(), torch.stack((torch.ones_like(pk), pk), -1).contiguous()
    if c["bias"] == "distance":
        rng = np.random.default_rng(seed)
        pq, pk = workloads.distance_factors(rng.random((N, 3)), 0.5 + rng.random((H, N)), 4.0)
        return torch.from_numpy(pq).to(dev), torch.from_numpy(pk).to(dev)
    if c["bias"] == "cosmul":
        t = torch.arange(N, device=dev, dtype=torch.float64) + torch.randint(0, 1000, (1,), generator=g, device=dev)
        x = torch.stack((t.cos(), t.sin()), -1).float().view(1, 1, N, 2).expand(1, H, N, 2).contiguous()
        return x, x.clone()
    if c["bias"] == "relpos":
        # sum_f a_f cos(w_f . (x_i - x_j) + p_f) with low frequencies: a smooth table over the offsets, bias std about 1
        side, F = int(round(math.sqrt(N))), R // 2
        t = torch.arange(N, device=dev)
        xy = torch.stack((t // side, t % side), -1).float()
        w = torch.randn((H, 2, F), generator=g, device=dev) * (2.0 * math.pi / side)
        p = 2.0 * math.pi * torch.rand((H, 1, F), generator=g, device=dev)
        a = math.sqrt(math.sqrt(2.0 / F))
        arg = torch.einsum("nd,hdf->hnf", xy, w)
        pq = a * torch.cat(((arg + p).cos(), (arg + p).sin()), -1)
        pk = a * torch.cat((arg.cos(), arg.sin()), -1)
        return pq[None].contiguous(), pk[None].contiguous()
    sc = float(R) ** -0.25                     # bias of standard deviation 1
    return (sc * torch.randn((Bp, H, N, R), generator=g, device=dev),
            sc * torch.randn((Bp, H, M, R), generator=g, device=dev))


def prepare(case, seed):
    c = case
    g = torch.Generator(device="cuda").manual_seed(seed)
    B, H, N, C = c["B"], c["H"], c["N"], c["C"]
    M = c["M"] or N
    train = c["path"] == "train"

    def normal(*shape):
        return torch.randn(shape, generator=g, device=g.device, dtype=torch.float32).to(_DT[c["dtype"]])

    s = {"case": c, "q": normal(B, H, N, C), "k": normal(B, H, M, C), "v": normal(B, H, M, C)}
    if train:
        s["dout"] = normal(B, H, N, C)
    if c["bias"] == "dense":
        s["bias"] = normal(1, H, N, N)
        leaves = ["q", "k", "v", "bias"]
    elif c["bias"] == "alibi" and train:
        s["slopes"] = torch.tensor(workloads.alibi_slopes_f32(H), device=g.device)
        leaves = ["q", "k", "v", "slopes"]
    else:
        pq, pk = _factors(c, seed, g)
        s["phi_q"], s["phi_k"] = pq.to(_DT[c["phi"]]), pk.to(_DT[c["phi"]])
        leaves = ["q", "k", "v", "phi_q", "phi_k"]
    if train:
        s["leaves"] = [s[n].requires_grad_() for n in leaves]
    return s


# ---- one pass ------------------------------------------------------------------------------------
def run(state):
    s = state
    c = s["case"]
    if c["path"] == "infer":
        if c["M"]:
            return api.fb_lowrank_xattn_fwd(s["q"], s["k"], s["v"], s["phi_q"], s["phi_k"])
        return api.fb_lowrank_attn_fwd(s["q"], s["k"], s["v"], s["phi_q"], s["phi_k"], causal=c["causal"])
    if c["bias"] == "dense":
        out = autograd.dense_bias_attention(s["q"], s["k"], s["v"], s["bias"], causal=c["causal"])
    elif c["bias"] == "alibi":
        out = autograd.alibi_attention(s["q"], s["k"], s["v"], s["slopes"], causal=c["causal"])
    elif c["bias"] == "cosmul":
        out = autograd.multiplicative_bias_attention(s["q"], s["k"], s["v"], s["phi_q"], s["phi_k"], causal=c["causal"])
    else:
        out = autograd.lowrank_bias_attention(s["q"], s["k"], s["v"], s["phi_q"], s["phi_k"], causal=c["causal"])
    return (out.detach(),) + torch.autograd.grad(out, s["leaves"], s["dout"])


# ---- what a pass cannot do without -----------------------------------------------------------------
def work(case):
    c = case
    B, H, N, C, R = c["B"], c["H"], c["N"], c["C"], c["R"]
    M = c["M"] or N
    e, pe = (4 if c["dtype"] == "f32" else 2), (4 if c["phi"] == "f32" else 2)
    rows_q, rows_k = B * H * N, B * H * M
    Bp = 1 if c["shared"] else B
    if c["bias"] == "dense":
        bias = H * N * N * e
    elif c["bias"] == "alibi" and c["path"] == "train":
        bias = H * 4
    else:
        bias = Bp * H * (N + M) * R * pe
    reads = (rows_q + 2 * rows_k) * C * e + bias             # q, k, v, bias
    writes = rows_q * C * e                                  # out
    if c["path"] == "infer":
        writes += rows_q * 4                                 # lse
    else:
        reads += rows_q * C * e                              # dout
        writes += (rows_q + 2 * rows_k) * C * e + bias       # gradients
    return {"bytes": float(reads + writes), "flops": _flops(c)}


def tolerance(case):
    """About four times the distance to the same path in 64 bits (measured over the listed and forty drawn cases):
    f32 up to 1.1e-6; bf16 up to 4.1e-3 with single values up to 0.19 off; the slope gradients 5.2e-3 (a sum over all
    queries that mostly cancels); the query-side distance factors' gradient 1.4e-2 (its columns multiply coordinates
    whose common part cancels)."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    if case["bias"] == "distance":
        return {"rel": 3e-2, "max": 0.7}
    if case["bias"] == "alibi" and case["path"] == "train":
        return {"rel": 2e-2, "max": 0.5}
    return {"rel": 1.2e-2, "max": 0.5}
