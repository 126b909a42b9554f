"""fp32 kernels on biases of extreme size: whole rows and whole columns at the type's lowest value (padding queries and
keys), and factor products below -1e30.  A row whose scores are all the same lowest value is the mean of v, as the
float64 oracle has it; with zero upstream gradient there, the other rows' gradients are the oracle's (fp32 bounds:
1e-4, gradients scaled by the largest entry)."""
import numpy as np
import pytest
import torch

from oracle import fb_oracle as O
from paper_2505_12044_amd import api
from tests._gpu_util import host

pytestmark = pytest.mark.gpu

LOWEST = np.finfo(np.float32).min


def _t(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def _close(name, got, ref):
    assert np.isfinite(got).all(), name
    bound = 1e-4 * max(1.0, float(np.abs(ref).max()))
    assert np.abs(got - ref).max() <= bound, (name, float(np.abs(got - ref).max()), bound)


def _close_fwd(out, lse, ro, rl, low):
    _close("out", out, ro)
    _close("lse", lse[~low], rl[~low])
    assert np.allclose(lse[low], rl[low], rtol=2.0 ** -22, atol=0.0)


# tiles shared by eight (backward: four) waves, by two, and one wave each
@pytest.mark.parametrize("B,H,N", [(1, 1, 200), (16, 32, 70), (32, 32, 65)])
@pytest.mark.parametrize("C,causal", [(16, False), (64, True), (128, False)])
def test_dense_lowest_rows_and_keys(B, H, N, C, causal):
    rng = np.random.default_rng(B + N + C)
    f32 = lambda *s: rng.standard_normal(s).astype(np.float32)
    q, k, v, dout = f32(B, H, N, C), f32(B, H, N, C), f32(B, H, N, C), f32(B, H, N, C)
    bias = f32(1, H, N, N)
    low = np.zeros(N, bool)
    low[N - 30:] = True
    low[5] = True
    bias[..., low, :] = LOWEST
    bias[..., :, N - 30:] = LOWEST
    dout[:, :, low] = 0.0
    d = [_t(q), _t(k), _t(v), _t(bias)]
    out, lse = api.fb_dense_bias_attn_fwd(*d, causal=causal)
    grads = api.fb_dense_bias_attn_bwd(*d, out, lse, _t(dout), causal=causal)
    torch.cuda.synchronize()
    for b, h in {(0, 0), (B - 1, H - 1)}:
        ro, rl = O.attention_with_bias(q[b, h], k[b, h], v[b, h], bias[0, h], causal=causal)
        _close_fwd(host(out[b, h]), host(lse[b, h]), ro, rl, low)
        ref = O.attention_with_bias_grads(q[b, h], k[b, h], v[b, h], bias[0, h], dout[b, h], causal=causal)
        for name, g, r in zip(("dq", "dk", "dv", "dbias"), grads, ref):
            _close(name, host(g[b, h]), r)


@pytest.mark.parametrize("B,H,N,M", [(1, 2, 150, 150), (1, 1, 33, 500), (32, 32, 65, 65)])
def test_factor_products_below_the_smallest_score(B, H, N, M):
    rng = np.random.default_rng(N + M)
    f32 = lambda *s: rng.standard_normal(s).astype(np.float32)
    C, R = 64, 3
    q, dout, k, v = f32(B, H, N, C), f32(B, H, N, C), f32(B, H, M, C), f32(B, H, M, C)
    pq, pk = f32(1, H, N, R), f32(1, H, M, R)
    low = np.arange(N) % 3 == 1
    pq[..., R - 1] = np.where(low, np.float32(-1e16), np.float32(0))      # products -1e32 on those rows, 0 elsewhere
    pk[..., R - 1] = np.float32(1e16)
    dout[:, :, low] = 0.0
    d = [_t(q), _t(k), _t(v), _t(pq), _t(pk)]
    if N == M:
        out, lse = api.fb_lowrank_attn_fwd(*d)
        grads = api.fb_lowrank_attn_bwd(*d, out, lse, _t(dout))
    else:
        out, lse = api.fb_lowrank_xattn_fwd(*d)
        grads = api.fb_lowrank_xattn_bwd(*d, out, lse, _t(dout))
    torch.cuda.synchronize()
    for b, h in {(0, 0), (B - 1, H - 1)}:
        ro, rl = O.attention_lowrank(q[b, h], k[b, h], v[b, h], pq[0, h], pk[0, h])
        _close_fwd(host(out[b, h]), host(lse[b, h]), ro, rl, low)
        dq, dk, dv, dpq, dpk = O.attention_lowrank_grads(q[b, h], k[b, h], v[b, h], pq[0, h], pk[0, h], dout[b, h])
        got = [host(g[b, h]) for g in grads]
        for name, g, r in zip(("dq", "dk", "dv"), got, (dq, dk, dv)):
            _close(name, g, r)
        # the last column of dphi_q is a sum that cancels against 1e16
        _close("dphi_q", got[3][:, :R - 1], dpq[:, :R - 1])
        _close("dphi_k", got[4], dpk)
