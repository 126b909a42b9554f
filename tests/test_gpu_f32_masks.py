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


@pytest.mark.parametrize("offset", [30.0, 300.0, 3000.0])
@pytest.mark.parametrize("C,causal", [(16, True), (64, False), (128, False)])
def test_dense_bias_with_a_common_offset(C, causal, offset):
    """Softmax does not see a row's common offset; the scores do, by one rounding: the products are summed at their own
    size and the bias is added once.  With u half a last place at the scores' size, a score is off by u (and 1e-6 of
    products), lse by u more, so P = exp(S - lse) and dBias = P (dP - D) by 2 u relative, and D, a sum over the row of
    P, by u; 5 u covers both and the products."""
    rng = np.random.default_rng(int(offset) + C)
    f32 = lambda *s: rng.standard_normal(s).astype(np.float32)
    N = 230
    q, k, v, dout = 2 * f32(1, 1, N, C), f32(1, 1, N, C), f32(1, 1, N, C), f32(1, 1, N, C)
    bias = f32(1, 1, N, N) + np.float32(offset)
    d = [_t(q), _t(k), _t(v), _t(bias)]
    out, lse = api.fb_dense_bias_attn_fwd(*d, causal=causal)
    grads = api.fb_dense_bias_attn_bwd(*d, out, lse, _t(dout), causal=causal)
    torch.cuda.synchronize()
    ro, rl = O.attention_with_bias(q[0, 0], k[0, 0], v[0, 0], bias[0, 0], causal=causal)
    u = float(np.spacing(np.float32(rl.max()))) / 2 + 1e-6
    elo = np.abs(host(lse[0, 0]) - rl).max()
    eo = np.abs(host(out[0, 0]) - ro).max()
    print(f"offset {offset} C {C}: u {u:.2e} lse {elo:.2e} out {eo:.2e}", flush=True)
    assert elo <= 2 * u
    assert eo <= u * np.abs(v).max()
    ref = O.attention_with_bias_grads(q[0, 0], k[0, 0], v[0, 0], bias[0, 0], dout[0, 0], causal=causal)
    for name, g, r in zip(("dq", "dk", "dv", "dbias"), grads, ref):
        e = np.abs(host(g[0, 0]) - r).max()
        print(f"  {name} {e:.2e} of {np.abs(r).max():.2e}: {e / np.abs(r).max() / u:.2f} u", flush=True)
        assert e <= 5 * u * np.abs(r).max(), name
