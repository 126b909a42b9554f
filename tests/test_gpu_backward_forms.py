"""The bf16 backward at the edges of its kernel forms: streamed lengths of one to six 32-row blocks around the
ring depth and around the 128-row tiles, both forms of the dkv kernel (up to 128 operand columns, and above),
every head dimension, causal and with separate key lengths, factors shared over the batch and per batch element.
Against the float64 oracle with the gradient bound of the other parity tests: 5e-2 flat, times max |phi| of the
other side for the factor gradients."""
import numpy as np
import pytest
import torch

from oracle import fb_oracle as O
from paper_2505_12044_amd import api, workloads as W
from tests._gpu_util import check_grad, dev, host

pytestmark = pytest.mark.gpu

#          C, R, phi      operand columns
WIDTHS = [(16, 0, "bf16"), (16, 2, "f32"), (16, 9, "f32"), (16, 24, "bf16"),
          (32, 4, "bf16"), (32, 6, "f32"), (32, 10, "f32"), (32, 64, "bf16"),
          (64, 0, "bf16"), (64, 16, "bf16"), (64, 5, "f32"), (64, 64, "bf16"),
          (128, 0, "bf16"), (128, 2, "f32"), (128, 9, "f32")]
#          N, M (0: as many as queries), causal, B
LENGTHS = [(1, 0, True, 2), (33, 0, False, 1), (97, 0, True, 2), (128, 0, False, 2), (161, 0, True, 1),
           (5, 190, False, 2), (129, 32, False, 1), (257, 0, True, 2)]
CASES = [(N, M, causal, B, C, R, phi, (i + j) % 2 == 0)
         for i, (C, R, phi) in enumerate(WIDTHS) for j, (N, M, causal, B) in enumerate(LENGTHS)]


@pytest.mark.parametrize("N,M,causal,B,C,R,phi,shared", CASES)
def test_backward_form(N, M, causal, B, C, R, phi, shared):
    _check_form(N, M, causal, B, C, R, phi, shared, 0.0)


# A scale of the caller's, which the forms carry in the query rows, with log2 e beside it, on the factor columns or in the
# exponent: one that rounds the query, and one that is a power of two.  Both at most the default, so the bounds hold as they do there.
@pytest.mark.parametrize("N,M,causal,B", [(97, 0, True, 2), (161, 0, False, 2), (6, 190, False, 2)])
@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("C,R,phi,scale", [(16, 9, "f32", 0.19), (16, 5, "bf16", 0.125), (32, 4, "f32", 0.15), (32, 10, "f32", 0.15), (32, 6, "f32", 0.125),
                                           (32, 16, "bf16", 0.15), (64, 9, "f32", 0.11), (64, 16, "bf16", 0.11), (64, 64, "bf16", 0.0625),
                                           (128, 8, "f32", 0.07), (128, 8, "bf16", 0.0625), (128, 8, "bf16", 0.07)])
def test_backward_form_with_a_scale(N, M, causal, B, C, R, phi, shared, scale):
    _check_form(N, M, causal, B, C, R, phi, shared, scale)


def _check_form(N, M, causal, B, C, R, phi, shared, scale):
    H, L = 2, M or N
    rng = np.random.default_rng(N * 7919 + L * 31 + C + R)
    rd = lambda *s: W.round_bf16(rng.standard_normal(s).astype(np.float32))
    q, k, v, dout = rd(B, H, N, C), rd(B, H, L, C), rd(B, H, L, C), rd(B, H, N, C)
    Bp, sc = 1 if shared else B, max(R, 1) ** -0.25
    pq = (sc * rng.standard_normal((Bp, H, N, R))).astype(np.float32)
    pk = (sc * rng.standard_normal((Bp, H, L, R))).astype(np.float32)
    if phi == "bf16":
        pq, pk = W.round_bf16(pq), W.round_bf16(pk)
    d = [dev(q, "bf16"), dev(k, "bf16"), dev(v, "bf16")] + ([dev(pq, phi), dev(pk, phi)] if R else [None, None])
    if M:
        out, lse = api.fb_lowrank_xattn_fwd(*d, scale=scale)
        grads = api.fb_lowrank_xattn_bwd(*d, out, lse, dev(dout, "bf16"), scale=scale)
    else:
        out, lse = api.fb_lowrank_attn_fwd(*d, causal=causal, scale=scale)
        grads = api.fb_lowrank_attn_bwd(*d, out, lse, dev(dout, "bf16"), causal=causal, scale=scale)
    torch.cuda.synchronize()
    label = f"bwd form N{N} M{L} C{C} R{R} {phi} causal={causal} shared={shared} scale={scale}"
    for b in range(B):
        for h in range(H):
            fq, fk = pq[0 if shared else b, h], pk[0 if shared else b, h]
            ref = O.attention_lowrank_grads(q[b, h], k[b, h], v[b, h], fq, fk, dout[b, h], causal=causal, scale=scale or None)
            for name, g, r in zip(("dq", "dk", "dv", "dphi_q", "dphi_k"), grads, ref):
                if g is not None:
                    other = pk if name == "dphi_q" else pq
                    gain = max(1.0, float(np.abs(other).max())) if name.startswith("dphi") else 1.0
                    check_grad(f"{label} (b,h)=({b},{h})", name, host(g[b, h]), r, gain=gain)
