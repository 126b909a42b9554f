"""The few-query forward (decode) at its edges: query counts of and between its instantiations, key counts around one
step of a wave and of a workgroup, with and without the split over the grid, each factor form, against the float64
oracle at the forward's bounds, and against the tile kernel it stands beside."""
import numpy as np
import pytest
import torch

from oracle import fb_oracle as O
from paper_2505_12044_amd import api, workloads as W
from tests._gpu_util import dev, host

pytestmark = pytest.mark.gpu


def _case(B, H, N, M, C, R, phi, shared, seed):
    rng = np.random.default_rng(seed)
    mk = lambda *s: W.round_bf16(rng.standard_normal(s).astype(np.float32))
    q, k, v = mk(B, H, N, C), mk(B, H, M, C), mk(B, H, M, C)
    pq = pk = None
    if R:
        Bp = 1 if shared else B
        pq, pk = mk(Bp, H, N, R), mk(Bp, H, M, R)
        if phi == "f32":
            pq, pk = (x + 1e-3 * rng.standard_normal(x.shape).astype(np.float32) for x in (pq, pk))
    return q, k, v, pq, pk


def _check(B, H, N, M, C, R, phi, shared=True):
    q, k, v, pq, pk = _case(B, H, N, M, C, R, phi, shared, seed=N * 1000 + M + C + R)
    d = [dev(q, "bf16"), dev(k, "bf16"), dev(v, "bf16")] + [None if x is None else dev(x, phi) for x in (pq, pk)]
    out, lse = api.fb_lowrank_xattn_fwd(*d)
    try:
        api.fb_tune_set("fwd_qb", 1)
        out_t, lse_t = api.fb_lowrank_xattn_fwd(*d)
    finally:
        api.fb_tune_set("fwd_qb", 0)
    torch.cuda.synchronize()
    for b in range(B):
        for h in range(H):
            fq = pq[min(b, pq.shape[0] - 1), h] if R else np.zeros((N, 0))
            fk = pk[min(b, pk.shape[0] - 1), h] if R else np.zeros((M, 0))
            ro, rl = O.attention_lowrank(q[b, h], k[b, h], v[b, h], fq, fk)
            for o, l in ((out, lse), (out_t, lse_t)):
                assert np.abs(host(o[b, h]) - ro).max() <= 2e-2 and np.abs(host(l[b, h]) - rl).max() <= 2e-2


@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 7, 8])
@pytest.mark.parametrize("C,R,phi", [(128, 2, "f32"), (64, 0, "f32"), (32, 9, "f32"), (16, 5, "bf16"), (128, 16, "bf16"), (64, 8, "bf16")])
def test_few_queries(N, C, R, phi):
    for M in (N + 1, 129, 1111):
        _check(2, 2, N, M, C, R, phi, shared=N % 2 == 0)


@pytest.mark.parametrize("N,M", [(1, 31), (1, 32), (1, 33), (1, 127), (1, 128), (1, 129), (2, 257), (4, 63), (4, 65), (8, 16), (8, 17)])
def test_few_queries_key_edges(N, M):
    _check(1, 2, N, M, 128, 2, "f32")


def test_few_queries_one_workgroup_per_head():
    # 600 heads: no split; without a workspace: no split either
    _check(75, 8, 1, 300, 16, 2, "f32")
    q, k, v, pq, pk = _case(2, 3, 1, 5000, 64, 2, "f32", True, seed=5)
    d = [dev(q, "bf16"), dev(k, "bf16"), dev(v, "bf16"), dev(pq, "f32"), dev(pk, "f32")]
    a, la = api.fb_lowrank_xattn_fwd(*d)
    b, lb = torch.empty_like(a), torch.empty_like(la)
    st = api.load_library().fb_lowrank_xattn_fwd(*(t.data_ptr() for t in d), b.data_ptr(), lb.data_ptr(), 2, 3, 1, 5000, 64, 2,
                                                 api.FB_BF16, api.FB_F32, 1, 0.0, torch.cuda.current_stream().cuda_stream or None)
    assert st == 0
    torch.cuda.synchronize()
    # the same fp32 sums in another grouping, rounded to bf16
    assert float((a.float() - b.float()).abs().max()) <= 2.0 ** -7 * float(a.float().abs().max())
    assert float((la - lb).abs().max()) <= 1e-5


def test_few_queries_decoder_positions():
    # ALiBi at the end of a long cache: the factors are absolute positions, the bias near the diagonal is small
    B, H, M, C = 1, 4, 16384, 64
    rng = np.random.default_rng(3)
    mk = lambda *s: W.round_bf16(rng.standard_normal(s).astype(np.float32))
    q, k, v = mk(B, H, 1, C), mk(B, H, M, C), mk(B, H, M, C)
    m = W.alibi_slopes_f32(H)
    pq = np.zeros((1, H, 1, 2), np.float32); pk = np.zeros((1, H, M, 2), np.float32)
    for h in range(H):
        pq[0, h, 0] = (-m[h] * np.float32(M - 1), m[h])
        pk[0, h, :, 0] = 1.0
        pk[0, h, :, 1] = np.arange(M, dtype=np.float32)
    out, lse = api.fb_lowrank_xattn_fwd(dev(q, "bf16"), dev(k, "bf16"), dev(v, "bf16"), dev(pq, "f32"), dev(pk, "f32"))
    torch.cuda.synchronize()
    ro, rl = O.batched_attention_lowrank(q, k, v, pq, pk)
    assert np.abs(host(out) - ro).max() <= 2e-2 and np.abs(host(lse) - rl).max() <= 2e-3


def test_few_queries_scratch_on_a_raw_stream_handle():
    # the split's workspace is the binding's own: memory that the current stream takes right behind the call must not be it
    q, k, v, pq, pk = _case(2, 4, 2, 20000, 64, 2, "f32", True, seed=9)
    d = [dev(q, "bf16"), dev(k, "bf16"), dev(v, "bf16"), dev(pq, "f32"), dev(pk, "f32")]
    nbytes = api.load_library().fb_lowrank_xattn_fwd_workspace_bytes(2, 4, 2, 20000, 64, 2, api.FB_BF16)
    assert nbytes > 0
    out, lse = api.fb_lowrank_xattn_fwd(*d)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    o2, l2 = api.fb_lowrank_xattn_fwd(*d, stream=side.cuda_stream)
    torch.empty(nbytes, dtype=torch.uint8, device="cuda").fill_(255)
    torch.cuda.synchronize()
    assert torch.equal(out, o2) and torch.equal(lse, l2)


# Every channel count and factor form with its keys split over the grid, the last step ragged
@pytest.mark.parametrize("N", [1, 2, 3, 5, 8])
@pytest.mark.parametrize("C,R,phi,M", [(128, 2, "f32", 1111), (64, 0, "f32", 2111), (32, 9, "f32", 4200), (32, 16, "bf16", 4200),
                                       (16, 5, "bf16", 8300), (16, 2, "f32", 8300)])
def test_few_queries_split(N, C, R, phi, M):
    assert api.fb_lowrank_xattn_fwd_workspace_bytes(2, 2, N, M, C, R) > 0
    _check(2, 2, N, M, C, R, phi, shared=N % 2 == 0)


# Calls that the tile kernel does faster: many queries and factors without scratch for the splits, short sequences
@pytest.mark.parametrize("B,H,N,M,C,R,phi,scratch", [(1, 2, 8, 10000, 128, 16, "bf16", False), (1, 8, 8, 5000, 64, 8, "bf16", False),
                                                     (1, 2, 8, 64, 16, 16, "bf16", True), (2, 4, 4, 300, 32, 8, "bf16", True)])
def test_calls_that_stay_on_the_tile_kernel(B, H, N, M, C, R, phi, scratch):
    q, k, v, pq, pk = _case(B, H, N, M, C, R, phi, True, seed=M)
    d = [dev(q, "bf16"), dev(k, "bf16"), dev(v, "bf16"), dev(pq, phi), dev(pk, phi)]
    ws = torch.empty(1 << 24, dtype=torch.uint8, device="cuda")
    res = []
    for qb in (0, 1):
        out, lse = torch.empty_like(d[0]), torch.empty((B, H, N), device="cuda")
        api.fb_tune_set("fwd_qb", qb)
        st = api.load_library().fb_lowrank_xattn_fwd_ws(*(t.data_ptr() for t in d), out.data_ptr(), lse.data_ptr(), B, H, N, M, C, R,
                                                        api.FB_BF16, api.FB_F32 if phi == "f32" else api.FB_BF16, 1, 0.0,
                                                        ws.data_ptr() if scratch else None, ws.numel() if scratch else 0,
                                                        torch.cuda.current_stream().cuda_stream or None)
        api.fb_tune_set("fwd_qb", 0)
        assert st == 0
        res.append((out, lse))
    torch.cuda.synchronize()
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])


def test_few_queries_caller_buffers():
    # out and lse given: no allocation, as every other forward; with the caller's workspace the result of the binding's own
    B, H, N, M, C, R = 2, 3, 1, 5000, 64, 2
    d = [dev(x, t) for x, t in zip(_case(B, H, N, M, C, R, "f32", True, seed=11), ("bf16", "bf16", "bf16", "f32", "f32"))]
    need = api.fb_lowrank_xattn_fwd_workspace_bytes(B, H, N, M, C, R)
    assert need > 0
    ref, ref_lse = api.fb_lowrank_xattn_fwd(*d)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    for workspace in (None, ws, ws[:need - 16]):
        out, lse = torch.empty_like(ref), torch.empty_like(ref_lse)
        torch.cuda.synchronize()
        before = torch.cuda.memory_stats()["allocation.all.allocated"]
        api.fb_lowrank_xattn_fwd(*d, out=out, lse=lse, workspace=workspace)
        assert torch.cuda.memory_stats()["allocation.all.allocated"] == before
        torch.cuda.synchronize()
        if workspace is ws:
            assert torch.equal(out, ref) and torch.equal(lse, ref_lse)
        # without the split the same fp32 sums in another grouping, rounded to bf16
        assert float((out.float() - ref.float()).abs().max()) <= 2.0 ** -7 * float(ref.float().abs().max())
        assert float((lse - ref_lse).abs().max()) <= 1e-5
