"""The fp32 kernels at the edges of their 32-row tiles and of the rule that splits a tile's streamed side
over several waves (few tiles: up to 8 waves in the forward, 4 in the backward; 2048 tiles: one wave), against
the float64 oracle at the fp32 bounds (1e-4, gradients scaled by the largest entry)."""
import numpy as np
import pytest
import torch

from oracle import fb_oracle as O
from paper_2505_12044_amd import api
from tests._gpu_util import host, report

pytestmark = pytest.mark.gpu

NAMES = ("dq", "dk", "dv", "dphi_q", "dphi_k")


def _run(B, H, N, M, C, R, causal, shared, heads):
    rng = np.random.default_rng(7 * N + 3 * M + C + R)
    f32 = lambda *s: rng.standard_normal(s).astype(np.float32)
    q, dout, k, v = f32(B, H, N, C), f32(B, H, N, C), f32(B, H, M, C), f32(B, H, M, C)
    Bp = 1 if shared else B
    pq = (0.5 * f32(Bp, H, N, R)) if R else None
    pk = (0.5 * f32(Bp, H, M, R)) if R else None
    t = lambda x: None if x is None else torch.from_numpy(x).cuda()
    d = [t(q), t(k), t(v), t(pq), t(pk)]
    if N == M:
        out, lse = api.fb_lowrank_attn_fwd(*d, causal=causal)
        grads = api.fb_lowrank_attn_bwd(*d, out, lse, t(dout), causal=causal)
    else:
        out, lse = api.fb_lowrank_xattn_fwd(*d)
        grads = api.fb_lowrank_xattn_bwd(*d, out, lse, t(dout))
    torch.cuda.synchronize()
    for b, h in heads:
        fq = pq[min(b, Bp - 1), h] if R else np.zeros((N, 0))
        fk = pk[min(b, Bp - 1), h] if R else np.zeros((M, 0))
        label = f"f32 B{B} H{H} N{N} M{M} C{C} R{R} causal={causal} (b,h)=({b},{h})"
        print(label, flush=True)
        ro, rl = O.attention_lowrank(q[b, h], k[b, h], v[b, h], fq, fk, causal=causal)
        for name, got, ref in (("out", out[b, h], ro), ("lse", lse[b, h], rl)):
            e, _, _ = report(label, name, host(got), ref)
            assert e <= 1e-4, (label, name, e)
        ref = O.attention_lowrank_grads(q[b, h], k[b, h], v[b, h], fq, fk, dout[b, h], causal=causal)
        for name, g, r in zip(NAMES, grads, ref):
            if g is None:
                continue
            e, _, big = report(label, name, host(g[b, h]), r)
            assert e <= 1e-4 * max(1.0, big), (label, name, e, big)


@pytest.mark.parametrize("N,M", [(1, 1), (31, 31), (32, 32), (33, 33), (1, 97), (65, 31), (64, 257)])
@pytest.mark.parametrize("C,R", [(16, 3), (32, 8), (64, 17), (128, 0), (128, 64)])
def test_f32_tile_edges(N, M, C, R):
    _run(1, 2, N, M, C, R, False, True, [(0, 1)])


@pytest.mark.parametrize("N", [33, 127, 200])
@pytest.mark.parametrize("C,R", [(16, 16), (64, 4), (128, 33)])
def test_f32_causal_edges(N, C, R):
    _run(2, 1, N, N, C, R, True, False, [(1, 0)])


# launches of 1024 and of 2048 tiles and more: two waves per tile, one wave per tile
@pytest.mark.parametrize("B,H,N,M,C,R,causal", [(16, 32, 64, 64, 64, 8, True), (32, 32, 65, 65, 32, 5, True),
                                                (64, 32, 33, 70, 16, 9, False), (33, 32, 64, 40, 128, 16, False)])
def test_f32_many_tiles(B, H, N, M, C, R, causal):
    _run(B, H, N, M, C, R, causal, True, [(0, 0), (B - 1, H - 1)])
