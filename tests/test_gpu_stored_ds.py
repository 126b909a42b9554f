"""The bf16 backward at 128 channels that stores dS between its two main kernels: every factor form, causal, separate key
lengths, partial tiles, trained slopes, one launch over all heads and several over parts of them.  It agrees to the bit
with the recomputing form (the workspace without room for dS), and with the float64 oracle at the bounds of the other tests."""
import numpy as np
import pytest
import torch

from oracle import fb_oracle as O
from paper_2505_12044_amd import api, workloads as W
from tests._gpu_util import check_grad, dev, host

pytestmark = pytest.mark.gpu
C = 128


def _inputs(B, H, N, M, R, phi, shared):
    rng = np.random.default_rng(N * 13 + M + R)
    rd = lambda *s: W.round_bf16(rng.standard_normal(s).astype(np.float32))
    q, k, v, dout = rd(B, H, N, C), rd(B, H, M, C), rd(B, H, M, C), rd(B, H, N, C)
    Bp, sc = 1 if shared else B, max(R, 1) ** -0.25
    pq = (sc * rng.standard_normal((Bp, H, N, R))).astype(np.float32)
    pk = (sc * rng.standard_normal((Bp, H, M, R))).astype(np.float32)
    if phi == "bf16":
        pq, pk = W.round_bf16(pq), W.round_bf16(pk)
    return q, k, v, dout, pq, pk


def _workspace(least, room):
    """`least` bytes and room for dS behind the next multiple of 256, in a pattern that no dS holds throughout."""
    return torch.full((least + (room + 256 if room else 0),), 0xA5, dtype=torch.uint8, device="cuda")


def _written(ws, least, heads, N, M):
    """Whether a call left dS of the first `heads` heads behind the formula's size: part of every head, nothing past the last."""
    per, off = ((N + 127) // 128 * 128) * ((M + 127) // 128 * 128) * 2, (least + 255) // 256 * 256
    assert not bool((ws[off + heads * per:] != 0xA5).any())
    if heads == 0:
        return False
    head = (ws[off:off + heads * per].view(heads, per) != 0xA5).any(1)
    assert bool(head.all()) == bool(head.any())
    return bool(head.all())


def _least(B, H, N, M, R):      # the workspace formula of the header
    return (B * H * N * 8 + 15) // 16 * 16 + B * H * (N + M) * (C + (64 if R else 0)) * 2


@pytest.mark.parametrize("N,M,causal", [(1647, 0, False), (2207, 0, True), (2176, 0, True), (700, 1600, False), (3300, 1105, False)])
@pytest.mark.parametrize("R,phi", [(0, "bf16"), (8, "bf16"), (20, "bf16"), (64, "bf16"), (3, "f32"), (10, "f32")])
def test_stored_and_recomputed(N, M, causal, R, phi):
    B, H, L = (4 if causal or N < 1000 else 2), 8, M or N
    shared = R % 3 != 0
    q, k, v, dout, pq, pk = _inputs(B, H, N, L, R, phi, shared)
    d = [dev(q, "bf16"), dev(k, "bf16"), dev(v, "bf16")] + ([dev(pq, phi), dev(pk, phi)] if R else [None, None])
    got = []
    least = _least(B, H, N, L, R)
    room = api.load_library().fb_attn_bwd_call_workspace_bytes(B, H, N, L, C, R, int(causal), api.FB_BF16) - least
    assert room > 0
    for n in (room - 256, 0):
        ws = _workspace(least, n)
        if M:
            out, lse = api.fb_lowrank_xattn_fwd(*d)
            got.append(api.fb_lowrank_xattn_bwd(*d, out, lse, dev(dout, "bf16"), workspace=ws))
        else:
            out, lse = api.fb_lowrank_attn_fwd(*d, causal=causal)
            got.append(api.fb_lowrank_attn_bwd(*d, out, lse, dev(dout, "bf16"), causal=causal, workspace=ws))
        torch.cuda.synchronize()
        assert _written(ws, least, B * H if n else 0, N, L) == (n > 0)
    for x, y in zip(*got):
        assert (x is None and y is None) or torch.equal(x, y)
    b, h = B - 1, H - 1
    fq, fk = pq[0 if shared else b, h], pk[0 if shared else b, h]
    ref = O.attention_lowrank_grads(q[b, h], k[b, h], v[b, h], fq, fk, dout[b, h], causal=causal)
    for name, g, r in zip(("dq", "dk", "dv", "dphi_q", "dphi_k"), got[0], ref):
        if g is not None:
            other = pk if name == "dphi_q" else pq
            gain = max(1.0, float(np.abs(other).max())) if name.startswith("dphi") else 1.0
            check_grad(f"stored N{N} M{L} R{R} {phi} causal={causal}", name, host(g[b, h]), r, gain=gain)


@pytest.mark.parametrize("N,B,H,heads,chunk", [(1024, 8, 8, 32, 32), (1100, 8, 8, 32, 28)])
def test_parts_of_the_heads(N, B, H, heads, chunk):
    """Room for the dS of half the heads: two launches of each kernel, or three of the 28 heads that fill one round of the
    key side's workgroups; the same gradients."""
    torch.manual_seed(3)
    t = lambda *s: torch.randn(*s, device="cuda").to(torch.bfloat16)
    q, k, v, do, pq, pk = t(B, H, N, C), t(B, H, N, C), t(B, H, N, C), t(B, H, N, C), t(1, H, N, 8), t(1, H, N, 8)
    out, lse = api.fb_lowrank_attn_fwd(q, k, v, pq, pk)
    one = ((N + 127) // 128 * 128) ** 2 * 2
    got = []
    for room, n in ((B * H, B * H), (heads, chunk), (0, 0)):
        ws = _workspace(_least(B, H, N, N, 8), room * one)
        got.append(api.fb_lowrank_attn_bwd(q, k, v, pq, pk, out, lse, do, workspace=ws))
        torch.cuda.synchronize()
        assert _written(ws, _least(B, H, N, N, 8), n, N, N) == (n > 0)
    for other in got[1:]:
        assert all(torch.equal(x, y) for x, y in zip(got[0], other))


def test_slope_gradient():
    torch.manual_seed(4)
    B, H, N = 4, 8, 2200
    t = lambda *s: torch.randn(*s, device="cuda").to(torch.bfloat16)
    q, k, v, do = t(B, H, N, C), t(B, H, N, C), t(B, H, N, C), t(B, H, N, C)
    slopes = torch.tensor(W.alibi_slopes_f32(H), device="cuda")
    out, lse = api.fb_alibi_attn_fwd(q, k, v, slopes, causal=True)
    got = []
    least = _least(B, H, N, N, 2)
    room = api.load_library().fb_attn_bwd_call_workspace_bytes(B, H, N, N, C, 2, 1, api.FB_BF16) - least
    for n in (room - 256, 0):
        rows, ws = torch.empty(B, H, N, device="cuda"), _workspace(least, n)
        got.append((rows,) + tuple(api.fb_alibi_attn_bwd(q, k, v, slopes, out, lse, do, causal=True, workspace=ws, dslope_rows=rows)))
        torch.cuda.synchronize()
        assert _written(ws, least, B * H if n else 0, N, N) == (n > 0)
    assert all(torch.equal(x, y) for x, y in zip(*got))


@pytest.mark.parametrize("N,causal", [(1700, False), (2500, True)])
def test_multiplicative_bias(N, causal):
    """R = 1 at 128 channels: the additive backward with float gradients, its workspace behind the prepared rows."""
    torch.manual_seed(8)
    B, H = 1, 16
    t = lambda *s: torch.randn(*s, device="cuda").to(torch.bfloat16)
    q, k, v, do, pq, pk = t(B, H, N, C), t(B, H, N, C), t(B, H, N, C), t(B, H, N, C), t(1, H, N, 1), t(1, H, N, 1)
    out, lse = api.fb_lowrank_mulbias_attn_fwd(q, k, v, pq, pk, causal=causal)
    inner = _least(B, H, N, N, 0)
    room = api.load_library().fb_attn_bwd_call_workspace_bytes(B, H, N, N, C, 0, int(causal), api.FB_BF16) - inner
    assert room > 0
    least, got = 2 * B * H * N * C * 6 + inner, []
    for n in (room - 256, 0):
        ws = _workspace(least, n)
        got.append(api.fb_lowrank_mulbias_attn_bwd(q, k, v, pq, pk, out, lse, do, causal=causal, workspace=ws))
        torch.cuda.synchronize()
        # (the inner workspace starts where the gradients end: a multiple of 256 bytes in both sizes here)
        assert (2 * B * H * N * C * 6) % 256 == 0 and _written(ws, least, B * H if n else 0, N, N) == (n > 0)
    for x, y in zip(*got):
        assert torch.equal(x, y)


def test_runs_where_there_is_no_memory_for_ds():
    """A process that may take no more than the least workspace: the same gradients, without dS in memory."""
    torch.manual_seed(6)
    B, H, N = 2, 8, 2200
    t = lambda *s: torch.randn(*s, device="cuda").to(torch.bfloat16)
    q, k, v, do, pq, pk = t(B, H, N, C), t(B, H, N, C), t(B, H, N, C), t(B, H, N, C), t(1, H, N, 8), t(1, H, N, 8)
    out, lse = api.fb_lowrank_attn_fwd(q, k, v, pq, pk)
    ref = api.fb_lowrank_attn_bwd(q, k, v, pq, pk, out, lse, do)
    grads = tuple(torch.empty_like(x) for x in ref)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    try:
        torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + _least(B, H, N, N, 8) + (48 << 20)) / total)
        got = api.fb_lowrank_attn_bwd(q, k, v, pq, pk, out, lse, do, grads=grads)
        torch.cuda.synchronize()
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    for x, y in zip(got, ref):
        assert torch.equal(x, y)
