"""The fp32 backward that stores dS between its two sides: partial tiles on both sides, causal, separate key lengths,
factor widths with every kind of last column tile, one launch over all heads and several over parts of them, and the
workspace just too small for it (the recomputing form).  Against the float64 oracle at the fp32 bounds, and the two
forms against each other."""
import numpy as np
import pytest
import torch

from oracle import fb_oracle as O
from paper_2505_12044_amd import api
from tests._gpu_util import host, report

pytestmark = pytest.mark.gpu

NAMES = ("dq", "dk", "dv", "dphi_q", "dphi_k")


def _up(n):
    return (n + 31) // 32 * 32


def _run(B, H, N, M, C, R, causal, shared, heads, ws_heads=None):
    rng = np.random.default_rng(7 * N + 3 * M + C + R)
    f32 = lambda *s: rng.standard_normal(s).astype(np.float32)
    q, dout, k, v = f32(B, H, N, C), f32(B, H, N, C), f32(B, H, M, C), f32(B, H, M, C)
    Bp = 1 if shared else B
    pq = (0.5 * f32(Bp, H, N, R)) if R else None
    pk = (0.5 * f32(Bp, H, M, R)) if R else None
    t = lambda x: None if x is None else torch.from_numpy(x).cuda()
    d = [t(q), t(k), t(v), t(pq), t(pk)]
    kw = {}
    if ws_heads is not None:      # room for dS of ws_heads heads behind D, and the least the call takes
        least = api.fb_lowrank_attn_bwd_workspace_bytes(B, H, N, C, R)
        room = (B * H * N * 4 + 255) // 256 * 256 + ws_heads * _up(N) * _up(M) * 4
        kw["workspace"] = torch.empty(max(least, room), dtype=torch.uint8, device="cuda")
    if N == M:
        out, lse = api.fb_lowrank_attn_fwd(*d, causal=causal)
        grads = api.fb_lowrank_attn_bwd(*d, out, lse, t(dout), causal=causal, **kw)
    else:
        out, lse = api.fb_lowrank_xattn_fwd(*d)
        grads = api.fb_lowrank_xattn_bwd(*d, out, lse, t(dout), **kw)
    torch.cuda.synchronize()
    for b, h in heads:
        fq = pq[min(b, Bp - 1), h] if R else np.zeros((N, 0))
        fk = pk[min(b, Bp - 1), h] if R else np.zeros((M, 0))
        label = f"f32 stored B{B} H{H} N{N} M{M} C{C} R{R} causal={causal} room={ws_heads} (b,h)=({b},{h})"
        print(label, flush=True)
        ref = O.attention_lowrank_grads(q[b, h], k[b, h], v[b, h], fq, fk, dout[b, h], causal=causal)
        for name, g, r in zip(NAMES, grads, ref):
            if g is None:
                continue
            e, _, big = report(label, name, host(g[b, h]), r)
            assert e <= 1e-4 * max(1.0, big), (label, name, e, big)
    return grads


@pytest.mark.parametrize("N,M,causal", [(601, 601, False), (601, 601, True), (640, 640, True), (523, 801, False), (1000, 385, False)])
@pytest.mark.parametrize("C,R", [(32, 0), (32, 5), (32, 33), (64, 8), (64, 64), (128, 3)])
def test_stored_ds(N, M, causal, C, R):
    _run(4, 8, N, M, C, R, causal, N % 2 == 0, [(0, 0), (3, 7)])


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("C,R", [(32, 8), (64, 3)])
def test_parts_and_recomputed(causal, C, R):
    """60 heads of 601 rows: dS of all, of 35 (two launches of 30) and of none."""
    got = [_run(15, 4, 601, 601, C, R, causal, True, [(0, 0), (7, 2), (14, 3)], ws_heads=n) for n in (60, 35, 0)]
    # a launch's split of a tile over waves follows from its tile count, so the sums' order differs: a few ulp of fp32
    for other in got[1:]:
        for x, y in zip(got[0], other):
            assert float((x - y).norm() / y.norm()) < 1e-5


def test_an_oversized_workspace_is_fine():
    _run(2, 8, 700, 700, 64, 4, False, True, [(1, 7)], ws_heads=40)


@pytest.mark.parametrize("N,M,causal", [(601, 601, False), (601, 601, True), (640, 577, False), (330, 900, False)])
@pytest.mark.parametrize("C,R,scale", [(32, 8, 0.0), (64, 3, 0.0), (64, 8, 0.3), (128, 16, 0.0), (128, 0, 0.25)])
def test_same_bits_with_any_workspace(N, M, causal, C, R, scale):
    """60 heads: dS of all of them, of 35 (two launches of 30) and of none, and on the static scratch (which takes a few
    heads at a time, or none): the scores, D and the order of the sums are the same, so are the gradients."""
    torch.manual_seed(N + C)
    B, H = 15, 4
    t = lambda *s: torch.randn(*s, device="cuda")
    q, k, v, do = t(B, H, N, C), t(B, H, M, C), t(B, H, M, C), t(B, H, N, C)
    pq, pk = (t(1, H, N, R), t(1, H, M, R)) if R else (None, None)
    kw = {"scale": scale}
    if N == M:
        kw["causal"] = causal
        fwd, bwd = api.fb_lowrank_attn_fwd, api.fb_lowrank_attn_bwd
    else:
        fwd, bwd = api.fb_lowrank_xattn_fwd, api.fb_lowrank_xattn_bwd
    out, lse = fwd(q, k, v, pq, pk, **kw)
    least = api.load_library().fb_attn_bwd_call_workspace_bytes(B, H, N, M, C, R, -1, api.FB_F32)
    d = (B * H * N * 4 + 255) // 256 * 256
    got = [bwd(q, k, v, pq, pk, out, lse, do, **kw)]
    for heads in (60, 35, 0):
        room = d + heads * _up(N) * _up(M) * 4
        # (none: the sizes are such that the least workspace leaves no room for it)
        ws = torch.full((max(least, room),), 0xA5, dtype=torch.uint8, device="cuda")
        got.append(bwd(q, k, v, pq, pk, out, lse, do, workspace=ws, **kw))
        per = _up(N) * _up(M) * 4      # dS of the heads of one launch, nothing behind it; D alone where none fits
        fills = 30 * min(_up(N), _up(M)) // 32 >= (4096 if causal and C <= 64 else 512)      # two launches have to fill the chip
        n = {60: 60, 35: 30 if fills else 0, 0: 0}[heads]
        assert bool((ws[d:d + n * per].view(n, per) != 0xA5).any(1).all()) if n else not bool((ws[d:] != 0xA5).any())
        assert not bool((ws[d + n * per:] != 0xA5).any())
    if N == M:
        grads = tuple(None if x is None else torch.empty_like(x) for x in got[0])
        got.append(api.fb_lowrank_attn_bwd_noalloc(q, k, v, pq, pk, out, lse, do, grads, **kw))
    torch.cuda.synchronize()
    for n, other in enumerate(got[1:]):
        for name, x, y in zip(NAMES, got[0], other):
            if x is not None:
                assert torch.equal(x, y), (name, n, float((x - y).abs().max()))


@pytest.mark.parametrize("heads,N,causal", [(20000, 1, False), (9000, 5, True), (3000, 33, False)])
def test_very_many_short_heads(heads, N, causal):
    """One partial tile (or two) a head, thousands of heads to a launch: against float64, every head."""
    torch.manual_seed(N)
    C, R = 32, 3
    t = lambda *s: torch.randn(*s, device="cuda")
    q, k, v, do, pq, pk = t(heads, 1, N, C), t(heads, 1, N, C), t(heads, 1, N, C), t(heads, 1, N, C), t(heads, 1, N, R), t(heads, 1, N, R)
    out, lse = api.fb_lowrank_attn_fwd(q, k, v, pq, pk, causal=causal)
    got = api.fb_lowrank_attn_bwd(q, k, v, pq, pk, out, lse, do, causal=causal)
    leaves = [x.double().requires_grad_() for x in (q, k, v, pq, pk)]
    s = leaves[0] @ leaves[1].transpose(-1, -2) * C ** -0.5 + leaves[3] @ leaves[4].transpose(-1, -2)
    if causal:
        s = s.masked_fill(torch.ones(N, N, device="cuda").triu(1).bool(), float("-inf"))
    ref = torch.autograd.grad(s.softmax(-1) @ leaves[2], leaves, do.double())
    for name, x, y in zip(NAMES, got, ref):
        big = max(1.0, float(y.abs().max()))
        assert float((x.double() - y).abs().max()) <= 1e-4 * big, name
