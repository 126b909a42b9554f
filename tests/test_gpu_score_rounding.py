"""The backward recomputes the scores that the forward's lse belongs to, so both have to round the query operand alike;
otherwise the rows of P = exp(S - lse) do not sum to one, and the rows of dS not to zero.  With unit vectors as upstream
gradient of as many rows as there are channels, dv is those rows of P.  Their sums may be off by what rounding P for the
forward's sum, for dv's contraction and dv itself to bf16 leaves: three independent errors per element, each of standard
deviation at most 2^-8 / sqrt(3) relative, six standard deviations allowed.  Keys with a common part let a different
rounding of the query in the two passes show as a shift of the whole row (up to thirty times the bound's unit)."""
import numpy as np
import pytest
import torch

from paper_2505_12044_amd import api, workloads as W
from tests._gpu_util import dev, host

pytestmark = pytest.mark.gpu


def _row_sums(N, M, H, C, R, phi, scale, qb):
    rng = np.random.default_rng(N + M + C + R)
    mk = lambda *s: rng.standard_normal(s).astype(np.float32)
    q, k, v = W.round_bf16(mk(1, H, N, C)), W.round_bf16(mk(1, H, M, C) + 1), W.round_bf16(mk(1, H, M, C))
    pq, pk = 0.5 * mk(1, H, N, R), 0.5 * mk(1, H, M, R)
    rows = rng.permutation(N)[:C]
    dout = np.zeros((1, H, N, C), np.float32)
    dout[:, :, rows, np.arange(len(rows))] = 1.0
    d = [dev(q, "bf16"), dev(k, "bf16"), dev(v, "bf16"), dev(pq, phi), dev(pk, phi)]
    try:
        api.fb_tune_set("fwd_qb", qb)
        out, lse = (api.fb_lowrank_attn_fwd if N == M else api.fb_lowrank_xattn_fwd)(*d, scale=scale)
    finally:
        api.fb_tune_set("fwd_qb", 0)
    bwd = api.fb_lowrank_attn_bwd if N == M else api.fb_lowrank_xattn_bwd
    dv = bwd(*d, out, lse, dev(dout, "bf16"), scale=scale)[2]
    _check_rows(dv, len(rows), f"N {N} M {M} C {C} R {R} {phi} scale {scale} form {qb}")


def _check_rows(dv, n, label):
    P = host(dv)[0][:, :, :n]
    err = np.abs(P.sum(1) - 1.0)
    sigma = 2.0 ** -8 / 3 ** 0.5 * np.sqrt(3 * (P ** 2).sum(1))
    print(f"{label}: worst row sum off by {err.max():.2e}, {(err / sigma).max():.1f} sigma", flush=True)
    assert (err <= 6 * sigma).all()


FACTORS = [(16, 2, "f32"), (16, 9, "f32"), (16, 2, "bf16"), (32, 2, "f32"), (32, 9, "f32"), (32, 8, "bf16"),
           (64, 2, "f32"), (64, 2, "bf16"), (128, 9, "f32"), (128, 8, "bf16")]


@pytest.mark.parametrize("N,H", [(8, 16), (64, 4)])         # few queries; 128-row tiles
@pytest.mark.parametrize("scale", [0.0, 0.3])
@pytest.mark.parametrize("C,R,phi", FACTORS)
def test_rows_of_p_sum_to_one(N, H, scale, C, R, phi):
    _row_sums(N, 4096, H, C, R, phi, scale, 0)


@pytest.mark.parametrize("N,H", [(96, 8), (180, 8), (384, 208)])      # heads that one workgroup takes whole
@pytest.mark.parametrize("C,R,phi", [(16, 8, "bf16"), (16, 20, "bf16"), (32, 8, "bf16"), (32, 24, "bf16")])
@pytest.mark.parametrize("scale", [0.0, 0.3])
def test_rows_of_p_sum_to_one_in_short_heads(N, H, C, R, phi, scale):
    _row_sums(N, N, H, C, R, phi, scale, 0)


@pytest.mark.parametrize("qb", [1, 2, 8, 16])               # every forward kernel, as many queries as keys
@pytest.mark.parametrize("C,R,phi", FACTORS)
def test_rows_of_p_sum_to_one_after_each_forward(qb, C, R, phi):
    _row_sums(2048, 2048, 2, C, R, phi, 0.0, qb)


@pytest.mark.parametrize("C", [16, 32, 64, 128])
@pytest.mark.parametrize("form", ["alibi", "dense", "cosmul"])
def test_rows_of_p_sum_to_one_other_entry_points(form, C):
    N, H = 1000, 2
    rng = np.random.default_rng(C)
    mk = lambda *s: rng.standard_normal(s).astype(np.float32)
    q, k, v = W.round_bf16(mk(1, H, N, C)), W.round_bf16(mk(1, H, N, C) + 1), W.round_bf16(mk(1, H, N, C))
    rows = rng.permutation(N)[:C]
    dout = np.zeros((1, H, N, C), np.float32)
    dout[:, :, rows, np.arange(C)] = 1.0
    d, do = [dev(x, "bf16") for x in (q, k, v)], dev(dout, "bf16")
    if form == "alibi":
        m = dev(np.array([0.01, 0.002], np.float32), "f32")
        out, lse = api.fb_alibi_attn_fwd(*d, m, causal=True)
        dv = api.fb_alibi_attn_bwd(*d, m, out, lse, do, causal=True)[2]
    elif form == "dense":
        b = dev(W.round_bf16(mk(1, H, N, N)), "bf16")
        out, lse = api.fb_dense_bias_attn_fwd(*d, b)
        dv = api.fb_dense_bias_attn_bwd(*d, b, out, lse, do)[2]
    else:
        R = 1 if C == 128 else 2
        f = [dev(mk(1, H, N, R), "f32") for _ in range(2)]
        out, lse = api.fb_lowrank_mulbias_attn_fwd(*d, *f)
        dv = api.fb_lowrank_mulbias_attn_bwd(*d, *f, out, lse, do)[2]
    torch.cuda.synchronize()
    _check_rows(dv, C, f"{form} C {C}")
