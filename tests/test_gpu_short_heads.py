"""The kernels for heads whose keys fit one workgroup (head dimensions 16 and 32, up to 384 keys): one to twelve 32-key
tiles, odd and even numbers of query blocks, partial last tiles, fewer queries than keys, factor widths of one and two
16-column groups with every remainder the kernels take, several heads to a workgroup, and the lengths just outside.
Against the float64 oracle at the bounds of the other parity tests."""
import numpy as np
import pytest
import torch

from oracle import fb_oracle as O
from paper_2505_12044_amd import api, workloads as W
from tests._gpu_util import check_fwd, check_grad, dev, host

pytestmark = pytest.mark.gpu


def _run(B, H, N, M, C, R, phi, causal, shared, heads, offset=0.0):
    rng = np.random.default_rng(N * 7919 + M * 31 + C + R)
    rd = lambda *s: W.round_bf16(rng.standard_normal(s).astype(np.float32))
    q, k, v, dout = rd(B, H, N, C), rd(B, H, M, C), rd(B, H, M, C), rd(B, H, N, C)
    Bp, sc = 1 if shared else B, max(R, 1) ** -0.25
    pq = (sc * rng.standard_normal((Bp, H, N, R))).astype(np.float32)
    pk = (sc * rng.standard_normal((Bp, H, M, R))).astype(np.float32)
    if offset:      # the bias grows along the keys, so the reference maximum of the first block is outgrown
        pq[..., 0], pk[..., 0] = 1.0, np.linspace(0.0, offset, M, dtype=np.float32)
    if phi == "bf16":
        pq, pk = W.round_bf16(pq), W.round_bf16(pk)
    d = [dev(q, "bf16"), dev(k, "bf16"), dev(v, "bf16")] + ([dev(pq, phi), dev(pk, phi)] if R else [None, None])
    if N == M:
        out, lse = api.fb_lowrank_attn_fwd(*d, causal=causal)
        grads = api.fb_lowrank_attn_bwd(*d, out, lse, dev(dout, "bf16"), causal=causal)
    else:
        out, lse = api.fb_lowrank_xattn_fwd(*d)
        grads = api.fb_lowrank_xattn_bwd(*d, out, lse, dev(dout, "bf16"))
    torch.cuda.synchronize()
    label = f"short B{B} H{H} N{N} M{M} C{C} R{R} {phi} causal={causal} shared={shared}"
    for b, h in heads:
        fq, fk = pq[0 if shared else b, h], pk[0 if shared else b, h]
        ro, rl = O.attention_lowrank(q[b, h], k[b, h], v[b, h], fq, fk, causal=causal)
        check_fwd(f"{label} ({b},{h})", "out", host(out[b, h]), ro)
        check_fwd(f"{label} ({b},{h})", "lse", host(lse[b, h]), rl)
        ref = O.attention_lowrank_grads(q[b, h], k[b, h], v[b, h], fq, fk, dout[b, h], causal=causal)
        for name, g, r in zip(("dq", "dk", "dv", "dphi_q", "dphi_k"), grads, ref):
            if g is not None:
                other = pk if name == "dphi_q" else pq
                gain = max(1.0, float(np.abs(other).max())) if name.startswith("dphi") else 1.0
                # a few keys or queries sum many rows: bound by the size of the result as in the other sweeps
                check_grad(f"{label} ({b},{h})", name, host(g[b, h]), r, data_scaled=True, gain=gain)


@pytest.mark.parametrize("N", [1, 31, 32, 33, 64, 65, 97, 128, 129, 161, 192, 225, 321, 353, 383, 384, 385])
@pytest.mark.parametrize("C,R", [(16, 8), (16, 28), (32, 4), (32, 16), (32, 24)])
@pytest.mark.parametrize("causal", [False, True])
def test_lengths(N, C, R, causal):
    _run(2, 3, N, N, C, R, "bf16", causal, N % 2 == 0, [(0, 0), (1, 2)])


@pytest.mark.parametrize("N,M", [(1, 384), (33, 383), (32, 65), (64, 70), (100, 320), (200, 230)])
@pytest.mark.parametrize("C,R", [(16, 12), (32, 16), (32, 32)])
def test_fewer_queries_than_keys(N, M, C, R):
    _run(3, 2, N, M, C, R, "bf16", False, True, [(0, 1), (2, 0)])


@pytest.mark.parametrize("C,R,phi", [(16, 0, "bf16"), (32, 0, "bf16"), (16, 3, "f32"), (32, 5, "f32"), (32, 10, "bf16"), (16, 18, "bf16")])
@pytest.mark.parametrize("N", [40, 180, 290, 384])
@pytest.mark.parametrize("causal", [False, True])
def test_other_factors(C, R, phi, N, causal):
    _run(1, 2, N, N, C, R, phi, causal, True, [(0, 1)])


# several heads to a workgroup: 256 CUs hold 256 workgroups of seven to twelve waves, 512 of six (full rounds, and rounds
# that the dispatch leaves to the kernels of longer heads)
@pytest.mark.parametrize("B,H,N", [(130, 4, 300), (300, 2, 384), (60, 20, 40), (75, 8, 225), (128, 4, 300), (64, 8, 384), (96, 8, 225), (50, 10, 180)])
@pytest.mark.parametrize("C,R,causal,shared", [(32, 16, False, True), (16, 16, True, False)])
def test_many_heads(B, H, N, C, R, causal, shared):
    _run(B, H, N, N, C, R, "bf16", causal, shared, [(0, 0), (B // 2, H - 1), (B - 1, H - 1), (B - 1, 0)])


@pytest.mark.parametrize("C", [16, 32])
@pytest.mark.parametrize("N", [96, 300])
def test_outgrown_reference(C, N):
    """The bias rises by 30 along the keys: the rescaling path of every later block."""
    _run(64, 4, N, N, C, 8, "bf16", False, True, [(0, 0), (63, 3)], offset=30.0)


@pytest.mark.parametrize("N", [20, 32, 64, 95, 129, 161, 192, 225, 256, 300, 384])
@pytest.mark.parametrize("C,R,offset", [(16, 0, 0), (16, 12, 0), (32, 4, 0), (32, 16, 0), (32, 32, 0), (16, 12, 30), (32, 16, 30)])
def test_rounds_as_the_ring_kernel_does(N, C, R, offset):
    """Full attention: the reference maximum comes from the same block and the sums follow in the same order as in the
    kernel that longer heads take, so the output is the same to the bit (offset: also where the bias along the keys
    outgrows the reference); a rescaled row sum may be contracted differently."""
    torch.manual_seed(N + C + R)
    t = lambda *s: torch.randn(*s, device="cuda").to(torch.bfloat16)
    B, H = 64, 4          # a head for every workgroup
    q, k, v, pq, pk = t(B, H, N, C), t(B, H, N, C), t(B, H, N, C), t(1, H, N, R), t(1, H, N, R)
    if offset:
        pq[..., 0], pk[..., 0] = 1.0, torch.linspace(0.0, offset, N, device="cuda").to(torch.bfloat16)
    if R == 0:
        pq = pk = None
    got = api.fb_lowrank_attn_fwd(q, k, v, pq, pk)
    try:
        api.fb_tune_set("fwd_qb", 1)
        ref = api.fb_lowrank_attn_fwd(q, k, v, pq, pk)
    finally:
        api.fb_tune_set("fwd_qb", 0)
    torch.cuda.synchronize()
    assert torch.equal(got[0], ref[0])
    assert float((got[1] - ref[1]).abs().max()) <= 2 ** -21 * max(1.0, float(ref[1].abs().max()))


@pytest.mark.parametrize("M", [20, 64, 95, 160, 200, 225, 300, 384])
@pytest.mark.parametrize("C,R", [(16, 8), (16, 28), (32, 4), (32, 16), (32, 32)])
@pytest.mark.parametrize("level", [0.0, 2.0 ** 14])
def test_recomputes_the_scores_of_the_two_kernel_backward(M, C, R, level):
    """More query blocks than key blocks take the two kernels of longer heads.  Rows with a zero upstream gradient add
    nothing to the key side, so its gradients have to be those of the call without them, to the bit: the same scores, P,
    dP and dS.  level: a common part of all scores of a row (-lse is then of that size too)."""
    torch.manual_seed(M + C + R)
    t = lambda *s: torch.randn(*s, device="cuda").to(torch.bfloat16)
    B, H, N, more = 50, 4, M, (M + 31) // 32 * 32 + 32
    q, k, v, do, pq, pk = t(B, H, more, C), t(B, H, M, C), t(B, H, M, C), t(B, H, more, C), t(1, H, more, R), t(1, H, M, R)
    do[:, :, N:] = 0.0
    if level:
        pq[..., 0], pk[..., 0] = level, 1.0
    out, lse = api.fb_lowrank_xattn_fwd(q, k, v, pq, pk)
    ref = api.fb_lowrank_xattn_bwd(q, k, v, pq, pk, out, lse, do)
    cut = lambda x: x[:, :, :N].contiguous()
    got = api.fb_lowrank_attn_bwd(cut(q), k, v, cut(pq), pk, cut(out), cut(lse), cut(do))
    torch.cuda.synchronize()
    for name, x, y in zip(("dk", "dv", "dphi_k"), (got[1], got[2], got[4]), (ref[1], ref[2], ref[4])):
        assert torch.isfinite(x.float()).all() and torch.equal(x, y), name
    for name, x, y in zip(("dq", "dphi_q"), (got[0], got[3]), (cut(ref[0]), cut(ref[3]))):      # the same dS, summed in another order
        assert float((x.float() - y.float()).norm() / y.float().norm()) <= 1e-3, name


@pytest.mark.parametrize("N,kept", [(64, 20), (200, 150), (200, 33), (384, 32)])
@pytest.mark.parametrize("C", [16, 32])
@pytest.mark.parametrize("causal", [False, True])
def test_key_padding(N, kept, C, causal):
    """A factor column that masks the keys from `kept` on: whole blocks of a row hold nothing but the mask, the diagonal one
    (which gives a causal row its reference maximum) and the last among them."""
    rng = np.random.default_rng(N + kept + C)
    rd = lambda *s: W.round_bf16(rng.standard_normal(s).astype(np.float32))
    B, H, R = 64, 4, 8
    q, k, v, dout = rd(B, H, N, C), rd(B, H, N, C), rd(B, H, N, C), rd(B, H, N, C)
    pq, pk = 0.5 * rd(1, H, N, R), 0.5 * rd(1, H, N, R)
    pq[..., 0], pk[..., 0] = 1.0, np.where(np.arange(N) < kept, 0.0, -2.0 ** 14)
    d = [dev(x, "bf16") for x in (q, k, v, pq, pk)]
    out, lse = api.fb_lowrank_attn_fwd(*d, causal=causal)
    grads = api.fb_lowrank_attn_bwd(*d, out, lse, dev(dout, "bf16"), causal=causal)
    torch.cuda.synchronize()
    for b, h in ((0, 0), (63, 3)):
        label = f"padding N{N} kept {kept} C{C} causal={causal} ({b},{h})"
        ro, rl = O.attention_lowrank(q[b, h], k[b, h], v[b, h], pq[0, h], pk[0, h], causal=causal)
        check_fwd(label, "out", host(out[b, h]), ro)
        check_fwd(label, "lse", host(lse[b, h]), rl)
        ref = O.attention_lowrank_grads(q[b, h], k[b, h], v[b, h], pq[0, h], pk[0, h], dout[b, h], causal=causal)
        for name, g, r in zip(("dq", "dk", "dv", "dphi_k"), (*grads[:3], grads[4]), (*ref[:3], ref[4])):
            check_grad(label, name, host(g[b, h]), r, data_scaled=True, gain=max(1.0, float(np.abs(pq).max())))


@pytest.mark.parametrize("B", [90, 128])       # two heads to some workgroups (the longer kernels' call), to all
def test_same_result_on_every_run(B):
    torch.manual_seed(5)
    t = lambda *s: torch.randn(*s, device="cuda").to(torch.bfloat16)
    q, k, v, do, pq, pk = t(B, 4, 333, 32), t(B, 4, 333, 32), t(B, 4, 333, 32), t(B, 4, 333, 32), t(1, 4, 333, 16), t(1, 4, 333, 16)
    first = None
    for _ in range(4):
        out, lse = api.fb_lowrank_attn_fwd(q, k, v, pq, pk)
        got = (out, lse) + tuple(api.fb_lowrank_attn_bwd(q, k, v, pq, pk, out, lse, do))
        torch.cuda.synchronize()
        if first is None:
            first = got
        assert all(torch.equal(a, b) for a, b in zip(first, got))
