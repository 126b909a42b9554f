"""The dense-bias backward whose key side writes dBias and whose query side reads it back as dS: lengths with 8, 16 and 24
keys in the last block, causal, a shared bias, scales that go onto the key rows (powers of two) and others, short heads in
large calls, against the float64 oracle at the bounds of the other dense gradients."""
import numpy as np
import pytest
import torch

from oracle import fb_oracle as O
from paper_2505_12044_amd import api, workloads as W
from tests._gpu_util import check_grad, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("B,H,N,C,shared,scale", [
    (2, 4, 1024, 32, True, 0.0), (2, 4, 1032, 64, False, 0.0), (4, 2, 1040, 128, True, 0.0), (1, 8, 1048, 64, True, 0.2),
    (2, 4, 1144, 32, False, 0.25), (1, 8, 1160, 128, False, 0.125), (16, 16, 392, 64, True, 0.0), (64, 16, 136, 128, True, 0.0)])
def test_dense_stored(B, H, N, C, shared, scale, causal):
    rng = np.random.default_rng(N + C)
    rd = lambda *s: W.round_bf16(rng.standard_normal(s, dtype=np.float32))
    q, k, v, dout = rd(B, H, N, C), rd(B, H, N, C), rd(B, H, N, C), rd(B, H, N, C)
    bias = rd(1 if shared else B, H, N, N)
    d = [dev(x, "bf16") for x in (q, k, v, bias)]
    out, lse = api.fb_dense_bias_attn_fwd(*d, causal=causal, scale=scale)
    got = api.fb_dense_bias_attn_bwd(*d, out, lse, dev(dout, "bf16"), causal=causal, scale=scale)
    torch.cuda.synchronize()
    for b, h in ((0, 0), (B - 1, H - 1)):
        ref = O.attention_with_bias_grads(q[b, h], k[b, h], v[b, h], bias[0 if shared else b, h], dout[b, h], causal=causal,
                                          scale=scale or None)
        for name, g, r in zip(("dq", "dk", "dv", "dbias"), got, ref):
            check_grad(f"dense stored B{B} H{H} N{N} C{C} causal={causal} ({b},{h})", name, host(g[b, h]), r)
        if causal:
            assert float(np.abs(np.triu(host(got[3][b, h]), 1)).max()) == 0.0
