"""CPU-side checks of the boundary: the shared library loads, exports every symbol the
header declares, and rejects bad arguments on the host before touching a device."""
import ctypes
import os
import re

import pytest

from paper_2505_12044_amd import api

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "flashbias.h")


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(api.LIB_PATH):
        from paper_2505_12044_amd import build
        build.build(force=False)
    return api.load_library()


def _declared_symbols():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(fb_[a-z0-9_]+)\s*\(", text)))


def test_header_symbols_exported(lib):
    names = _declared_symbols()
    assert set(names) == set(api.EXPORTS)
    for n in names:
        assert hasattr(lib, n), n


def test_version_and_status_strings(lib):
    assert lib.fb_version() >= 100
    assert lib.fb_status_string(0) == b"ok"
    seen = {lib.fb_status_string(i) for i in range(8)}
    assert len(seen) == 8
    assert lib.fb_status_string(99) == b"unknown status"


def _fwd(lib, **kw):
    a = dict(q=64, k=64, v=64, phi_q=64, phi_k=64, out=64, lse=64, B=1, H=1, N=16, C=64, R=4,
             causal=0, dtype=api.FB_BF16, phi_dtype=api.FB_BF16, bcast=0, scale=0.0)
    a.update(kw)
    return lib.fb_lowrank_attn_fwd(a["q"], a["k"], a["v"], a["phi_q"], a["phi_k"], a["out"], a["lse"],
                                   a["B"], a["H"], a["N"], a["C"], a["R"], a["causal"], a["dtype"],
                                   a["phi_dtype"], a["bcast"], a["scale"], None)


def test_forward_argument_errors(lib):
    # fake non-null addresses: every case below must be rejected before any device access
    assert _fwd(lib, q=None) == 1
    assert _fwd(lib, phi_k=None) == 1
    assert _fwd(lib, N=0) == 2
    assert _fwd(lib, R=-1) == 2
    assert _fwd(lib, B=1 << 20, H=1 << 10, N=1 << 12) == 2          # index overflow
    assert _fwd(lib, C=48) == 3
    assert _fwd(lib, R=65) == 3                                      # padded width > 64
    assert _fwd(lib, R=11, phi_dtype=api.FB_F32) == 3                # 6 R > 64 columns
    assert _fwd(lib, dtype=api.FB_F32, phi_dtype=api.FB_BF16) == 3
    assert _fwd(lib, dtype=7) == 3
    assert _fwd(lib, k=72) == 4                                      # misaligned


def test_dense_and_backward_argument_errors(lib):
    f = lib.fb_dense_bias_attn_fwd
    assert f(64, 64, 64, None, 64, 64, 1, 1, 16, 64, 0, api.FB_BF16, 0, 0.0, None) == 1
    assert f(64, 64, 64, 64, 64, 64, 1, 1, 16, 96, 0, api.FB_BF16, 0, 0.0, None) == 3
    assert f(64, 64, 64, 68, 64, 64, 1, 1, 16, 64, 0, api.FB_BF16, 0, 0.0, None) == 4
    db = lib.fb_dense_bias_attn_bwd
    wsd = lib.fb_dense_bias_attn_bwd_workspace_bytes(1, 1, 64, 64, api.FB_BF16)
    assert wsd == 64 * 8 + 2 * 64 * 64 * 2
    # head dimension 16: 32-channel operand rows plus widened copies of v and dO
    assert lib.fb_dense_bias_attn_bwd_workspace_bytes(1, 1, 64, 16, api.FB_BF16) == 64 * 8 + 2 * 64 * (32 + 32) * 2
    assert db(*([64] * 10), None, 1, 1, 64, 64, 0, api.FB_BF16, 0, 0.0, 64, wsd, None) == 1         # dbias NULL
    assert db(*([64] * 11), 1, 1, 60, 64, 0, api.FB_BF16, 0, 0.0, 64, wsd, None) == 3               # N % 8 != 0
    assert db(*([64] * 11), 1, 1, 64, 64, 0, api.FB_BF16, 0, 0.0, 64, wsd - 1, None) == 5
    a = lib.fb_alibi_attn_fwd
    assert a(64, 64, 64, None, 64, 64, 1, 1, 16, 64, 1, api.FB_BF16, 0.0, None) == 1      # slopes NULL
    assert a(64, 64, 64, 64, 64, 64, 1, 1, 16, 64, 1, api.FB_F32, 0.0, None) == 3         # bf16 only
    assert a(64, 64, 64, 66, 64, 64, 1, 1, 16, 64, 1, api.FB_BF16, 0.0, None) == 4        # slopes not 4-byte aligned
    assert a(64, 64, 64, 64, 64, 64, 1, 1, 0, 64, 1, api.FB_BF16, 0.0, None) == 2
    ws = lib.fb_lowrank_attn_bwd_workspace_bytes(2, 3, 100, 64, 8, api.FB_BF16)
    # (lse, D) pairs plus the two concatenated operand copies of width up to C + 64
    assert ws == 2 * 3 * 100 * 8 + 2 * (2 * 3 * 100) * (64 + 64) * 2
    assert lib.fb_lowrank_attn_bwd_workspace_bytes(0, 3, 100, 64, 8, api.FB_BF16) == 0
    # head dimension 16: 32-channel operand rows plus widened copies of v and dO
    assert lib.fb_lowrank_attn_bwd_workspace_bytes(1, 1, 10, 16, 9, api.FB_F32) == 10 * 8 + 2 * 10 * (32 + 64 + 32) * 2
    g = lib.fb_lowrank_attn_bwd
    ptrs = [64] * 13

    def bwd(ptrs=ptrs, B=2, H=3, N=100, C=64, R=8, dtype=api.FB_BF16, phi=api.FB_BF16, w=64, wb=ws):
        return g(*ptrs, B, H, N, C, R, 0, dtype, phi, 0, 0.0, w, wb, None)

    assert bwd(ptrs=[None] + [64] * 12) == 1
    assert bwd(dtype=api.FB_F32) == 3          # fp32 tensors need fp32 factors
    assert bwd(dtype=api.FB_F32, phi=api.FB_F32, R=70) == 3
    assert bwd(R=70) == 3                      # padded width > 64
    assert bwd(w=None) == 5
    assert bwd(wb=ws - 1) == 5
    assert bwd(w=72) == 4


def test_mulbias_argument_errors(lib):
    f = lib.fb_lowrank_mulbias_attn_fwd
    need = lib.fb_lowrank_mulbias_attn_fwd_workspace_bytes(1, 2, 100, 64, 2, api.FB_BF16)
    assert need == 4 * 1 * 2 * 100 * 64 * 2
    assert lib.fb_lowrank_mulbias_attn_fwd_workspace_bytes(1, 2, 100, 64, 0, api.FB_BF16) == 0

    def call(ptrs=None, C=64, R=2, dtype=api.FB_BF16, w=64, wb=need):
        ptrs = ptrs or [64] * 7
        return f(*ptrs, 1, 2, 100, C, R, 0, dtype, api.FB_F32, 0, 0.0, w, wb, None)

    assert call(ptrs=[64, 64, 64, None, 64, 64, 64]) == 1      # factors are required
    assert call(R=0) == 2
    assert call(R=4) == 3                                      # C (R - 1) = 192 > 128
    assert call(C=128, R=2) == 3                               # C = 128 takes no extra channels
    assert call(dtype=api.FB_F32) == 3
    assert call(ptrs=[64, 64, 64, 66, 64, 64, 64]) == 4        # factors not 4-byte aligned
    assert call(w=None) == 5
    assert call(wb=need - 1) == 5
    assert call(w=72) == 4


def test_mulbias_backward_argument_errors(lib):
    f = lib.fb_lowrank_mulbias_attn_bwd
    need = lib.fb_lowrank_mulbias_attn_bwd_workspace_bytes(1, 2, 100, 32, 3, api.FB_BF16)
    # q', k' in bf16, their gradients in float, and the additive backward's scratch for 64 extra channels
    assert need == 2 * 200 * 32 * 3 * (2 + 4) + lib.fb_lowrank_attn_bwd_workspace_bytes(1, 2, 100, 32, 64, api.FB_BF16)
    # more than 64 extra channels: operand rows of width C + 128
    need5 = lib.fb_lowrank_mulbias_attn_bwd_workspace_bytes(1, 2, 100, 32, 5, api.FB_BF16)
    assert need5 == 2 * 200 * 32 * 5 * 6 + 200 * 8 + 2 * 200 * (32 + 128) * 2

    def call(ptrs=None, C=32, R=3, dtype=api.FB_BF16, w=64, wb=need):
        ptrs = ptrs or [64] * 13
        return f(*ptrs, 1, 2, 100, C, R, 0, dtype, api.FB_BF16, 0, 0.0, w, wb, None)

    assert call(ptrs=[64] * 12 + [None]) == 1
    assert call(R=0) == 2
    assert call(R=6) == 3                      # C (R - 1) = 160 > 128
    assert call(dtype=api.FB_F32) == 3
    assert call(ptrs=[64] * 11 + [66, 64]) == 4
    assert call(wb=need - 1) == 5
    assert call(w=None) == 5


def test_alibi_backward_argument_errors(lib):
    f = lib.fb_alibi_attn_bwd
    need = lib.fb_alibi_attn_bwd_workspace_bytes(1, 2, 100, 64, api.FB_BF16)
    assert need == lib.fb_lowrank_attn_bwd_workspace_bytes(1, 2, 100, 64, 2, api.FB_BF16)

    def call(ptrs=None, C=64, dtype=api.FB_BF16, w=64, wb=need, N=100):
        ptrs = ptrs or [64] * 10 + [None]                       # dslope_rows NULL: not wanted
        if len(ptrs) == 10:
            ptrs = ptrs + [None]
        return f(*ptrs, 1, 2, N, C, 1, dtype, 0.0, w, wb, None)

    assert call(ptrs=[64, 64, 64, None] + [64] * 6) == 1       # slopes
    assert call(ptrs=[64] * 10 + [66]) == 4                    # dslope_rows not 4-byte aligned
    assert call(N=0) == 2
    assert call(C=48) == 3
    assert call(dtype=api.FB_F32) == 3
    assert call(ptrs=[64, 64, 64, 66] + [64] * 6) == 4
    assert call(wb=need - 1) == 5


def test_size_limits_follow_the_indexing(lib):
    """Offsets above the head level are 64-bit: tensors of 2^31 elements and more are accepted
    (the calls below pass the shape check and stop at the deliberately misaligned pointer);
    what is limited is the row count (32-bit counters) and the extent of one head (32-bit byte
    offsets)."""
    assert _fwd(lib, B=2, H=8, N=1 << 17, C=128, R=8, k=72) == 4        # 2^31 elements per tensor
    assert _fwd(lib, B=64, H=64, N=1 << 16, C=128, R=8, k=72) == 4      # 2^35 elements, 2^28 rows
    assert _fwd(lib, B=1 << 10, H=1 << 5, N=1 << 16, C=32, R=0, k=72) == 2     # 2^31 rows
    assert _fwd(lib, B=1, H=1, N=1 << 23, C=128, R=0, k=72) == 2        # one head: N C = 2^30 elements
    assert _fwd(lib, B=1, H=1, N=1 << 22, C=128, R=0, k=72) == 4
    assert _fwd(lib, B=1, H=1, N=1 << 26, C=16, R=16, k=72) == 2        # N R = 2^30 factor values
    a = lib.fb_alibi_attn_fwd
    assert a(64, 64, 64, 64, 64, 64, 1, 1, (1 << 24) + 1, 16, 1, api.FB_BF16, 0.0, None) == 3   # fp32 positions


@pytest.mark.parametrize("C", [32, 64, 128])
@pytest.mark.parametrize("dtype", [api.FB_F32, api.FB_BF16])
def test_backward_size_queries_take_any_length(lib, C, dtype):
    """The queries run ahead of the limits: padding a length next to the largest int must not wrap (it did, to a head of
    zero bytes that the query then divided by).  Such heads have no room for dS, so the plain formula is the answer."""
    for N in (2 ** 31 - 32, 2 ** 31 - 31, 2 ** 31 - 1):
        for M in (N, 64):
            need = N * 8 + 15 & ~15
            need += (N + M) * (C + 64) * 2
            assert lib.fb_lowrank_xattn_bwd_workspace_bytes(1, 1, N, M, C, 8, dtype) == need
        assert lib.fb_lowrank_attn_bwd_workspace_bytes(1, 1, N, C, 8, dtype) == (N * 8 + 15 & ~15) + 2 * N * (C + 64) * 2


def _least(B, H, N, M, C, R):
    return (B * H * N * 8 + 15 & ~15) + B * H * (N + M) * (C + (64 if R else 0)) * 2


def _stored_heads_bf16(heads, N, M, causal):
    """The launch's rule, every chunk of heads tried: what the pairs save against the extra launch, then rounds of 256
    workgroups of the key side against one launch over all heads."""
    up = lambda n: -(-n // 128) * 128
    per = up(N) * up(M) * 2
    fit = (1 << 30) // per
    if fit == 0 or heads * N * ((0.5 if causal else 1.0) * M - 768.0) < 1 << 24:
        return 0, per
    if fit >= heads:
        return heads, per
    tiles = up(M) // 128
    units = (tiles + 1) // 2 if causal else tiles
    rounds = lambda h: -(-h * units // 256)
    best, cost = 0, 1.1 * rounds(heads)
    for c in range(fit, 0, -1):
        if c * 4 < fit:
            break
        t = heads // c * rounds(c) + rounds(heads % c)
        if t < cost:
            best, cost = c, t
    return best, per


def _stored_heads_f32(heads, N, M, C, causal, room=1 << 30):
    """Parts of equal size; where a part's tiles spill a little into another round of 2048, parts of full rounds."""
    up = lambda n: -(-n // 32) * 32
    per, nq, nk = up(N) * up(M) * 4, -(-N // 32), -(-M // 32)
    fit = room // per
    if fit == 0 or heads * nq * nk * C < 262144:
        return 0, per
    while True:
        parts = -(-heads // fit)
        chunk = -(-heads // parts)
        tiles = chunk * min(nq, nk)
        if parts == 1:
            return heads, per
        if tiles < (4096 if causal and C <= 64 else 512):
            return 0, per
        rounds = tiles / 2048
        if causal or rounds < 1 or rounds >= 0.6 * (int(rounds) + 1) or rounds == int(rounds) or int(rounds) * 2048 < min(nq, nk):
            return chunk, per
        fit = int(rounds) * 2048 // min(nq, nk)


SIZES = [(1, 1, 100), (4, 16, 256), (16, 16, 1000), (4, 16, 1024), (64, 4, 1024), (8, 8, 1100), (64, 4, 1536), (4, 16, 1500), (16, 60, 1100), (1, 16, 2048),
         (4, 16, 4096), (3, 5, 3000), (40, 40, 800), (100, 50, 900), (33, 33, 1900), (19, 4, 3700), (30, 4, 3716), (24, 3, 3000), (2, 8, 8192), (1, 16, 8800), (2, 8, 10000), (1, 16, 12000), (1, 2, 16000), (2, 8, 16384),
         (1, 1, 23168), (1, 1, 23169), (2, 8, 30000), (1 << 16, 4, 8), (1 << 18, 1, 1)]


@pytest.mark.parametrize("B,H,N", SIZES)
def test_backward_asks_for_no_room_it_does_not_use(lib, B, H, N):
    """Beyond the formula the size of a call is what the launch's rule for its mask stores, to the byte (bf16: up to the
    next multiple of 256 behind the formula), and the query, which does not know the mask, the larger of the two."""
    call = lib.fb_attn_bwd_call_workspace_bytes
    for M in (N, N // 2 + 1):
        for R in (0, 8):
            least = _least(B, H, N, M, 128, R)
            assert call(B, H, N, M, 128, R, -1, api.FB_BF16) == least
            sizes = []
            for causal in (0, 1):
                chunk, per = _stored_heads_bf16(B * H, N, M, causal)
                sizes.append(least + (256 + chunk * per if chunk else 0))
                assert call(B, H, N, M, 128, R, causal, api.FB_BF16) == sizes[-1], (M, R, causal)
            assert lib.fb_lowrank_xattn_bwd_workspace_bytes(B, H, N, M, 128, R, api.FB_BF16) == (max(sizes) if M == N else sizes[0])
            for C in (32, 64, 128):
                sizes = []
                for causal in (0, 1):
                    chunk, per = _stored_heads_f32(B * H, N, M, C, causal)
                    # the launch finds the same part in that room
                    assert chunk == 0 or _stored_heads_f32(B * H, N, M, C, causal, chunk * per)[0] == chunk
                    sizes.append(max(_least(B, H, N, M, C, R), (B * H * N * 4 + 255 & ~255) + chunk * per if chunk else 0))
                    assert call(B, H, N, M, C, R, causal, api.FB_F32) == sizes[-1], (C, causal)
                assert lib.fb_lowrank_xattn_bwd_workspace_bytes(B, H, N, M, C, R, api.FB_F32) == (max(sizes) if M == N else sizes[0])
    assert call(B, H, N, N, 64, 8, 0, api.FB_BF16) == _least(B, H, N, N, 64, 8)
    assert lib.fb_alibi_attn_bwd_workspace_bytes(B, H, N, 128, api.FB_BF16) == lib.fb_lowrank_attn_bwd_workspace_bytes(B, H, N, 128, 2, api.FB_BF16)
    room = lib.fb_lowrank_attn_bwd_workspace_bytes(B, H, N, 128, 0, api.FB_BF16) - _least(B, H, N, N, 128, 0)
    assert lib.fb_lowrank_mulbias_attn_bwd_workspace_bytes(B, H, N, 128, 1, api.FB_BF16) == 2 * B * H * N * 128 * 6 + _least(B, H, N, N, 128, 0) + room


def test_noalloc_backward_host_checks(lib):
    """The allocation-free backward rejects bad shapes and problems beyond its static scratch on
    the host, before any device call."""
    g = lib.fb_lowrank_attn_bwd_noalloc
    ptrs = [64] * 13
    assert g(*ptrs, 0, 1, 16, 64, 4, 0, api.FB_BF16, api.FB_BF16, 0, 0.0, None) == 2
    assert g(*ptrs, 1, 1, 16, 48, 4, 0, api.FB_BF16, api.FB_BF16, 0, 0.0, None) == 3
    B, H, N, C, R = 4, 16, 4096, 128, 2
    assert lib.fb_lowrank_attn_bwd_workspace_bytes(B, H, N, C, R, api.FB_BF16) > api.FB_STATIC_SCRATCH_BYTES
    st = g(*ptrs, B, H, N, C, R, 1, api.FB_BF16, api.FB_F32, 1, 0.0, None)
    assert st == 7 and b"static scratch" in lib.fb_status_string(st)
    text = open(HEADER).read()
    m = re.search(r"#define FB_STATIC_SCRATCH_BYTES \(\(size_t\)(\d+) << (\d+)\)", text)
    assert m and int(m.group(1)) << int(m.group(2)) == api.FB_STATIC_SCRATCH_BYTES


def test_only_the_c_abi_is_exported():
    """Built with hidden visibility: the dynamic symbol table defines the header's functions and
    nothing else of this library's own."""
    import subprocess
    out = subprocess.run(["nm", "-D", "--defined-only", api.LIB_PATH], capture_output=True, text=True, check=True).stdout
    defined = {line.split()[-1] for line in out.splitlines() if line.strip()}
    ours = {n for n in defined if not n.startswith("__hip") and n not in ("_init", "_fini")}
    assert ours == set(api.EXPORTS), sorted(ours ^ set(api.EXPORTS))


def test_tune_knob(lib):
    assert lib.fb_tune_set(b"fwd_qb", 2) == 0
    assert lib.fb_tune_set(b"fwd_qb", 0) == 0
    assert lib.fb_tune_set(b"fwd_qb", 3) == 2
    assert lib.fb_tune_set(b"fwd_qb", 4) == 2
    assert lib.fb_tune_set(b"fwd_qb", 8) == 0
    assert lib.fb_tune_set(b"fwd_qb", 0) == 0
    assert lib.fb_tune_set(b"fwd_causal_up", 0) == 0
    assert lib.fb_tune_set(b"fwd_causal_up", 2) == 2
    assert lib.fb_tune_set(b"fwd_causal_up", 1) == 0
    assert lib.fb_tune_set(b"fwd_lds_pad", 0) == 3          # probe knob removed
    assert lib.fb_tune_set(b"nope", 1) == 3
    assert lib.fb_tune_set(None, 1) == 1


def test_missing_library_fails_loudly(tmp_path):
    with pytest.raises(api.FlashBiasError):
        api.load_library(str(tmp_path / "libflashbias.so"))


def test_hand_placed_mfma_forms_keep_their_wait_states():
    """The backward's inline-assembly MFMA forms are invisible to the compiler's hazard padding: the
    generated code must show no instruction touching such a result inside its wait-state window
    (compiles one source to assembly, about a minute and a half).  The scanner itself is checked on
    a planted violation first."""
    from paper_2505_12044_amd import check_mfma_hazards as chk
    planted = ("_Zk:\n\tv_mfma_f32_32x32x16_bf16 v[0:15], v[16:19], v[20:23], v[0:15]\n"
               "\tv_mfma_f32_32x32x16_bf16 v[0:15], v[24:27], v[20:23], v[0:15]\n"
               "\tv_add_f32_e32 v40, v3, v41\n")
    seen, found = chk.scan_asm(planted)
    assert seen == 2 and len(found) == 1
    fenced = planted.replace("\tv_add_f32", "\ts_nop 7\n\ts_nop 2\n\tv_add_f32")
    assert chk.scan_asm(fenced)[1] == []
    seen, found = chk.check()
    assert seen > 0 and found == [], found[:3]


def test_scratch_falls_back_to_the_least_size(monkeypatch):
    """A backward that fits without the room for dS runs without it; any other shortage is reported as before."""
    import torch
    real, limit = torch.empty, 100 << 20

    def empty(n, **kw):
        if n > limit:
            raise torch.OutOfMemoryError(f"{n} bytes")
        return real(n, **kw)
    monkeypatch.setattr(torch, "empty", empty)
    lib = api.load_library()
    shape = (1, 4, 4096, 4096, 128, 8)
    need, least = (lib.fb_attn_bwd_call_workspace_bytes(*shape, m, api.FB_BF16) for m in (0, -1))
    assert least < limit < need
    assert api._bwd_scratch(lib, *shape, False, api.FB_BF16, "cpu", None).numel() == least
    for nbytes, small in ((limit + 1, None), (limit + 1, limit + 1), (limit + 2, limit + 1)):
        with pytest.raises(torch.OutOfMemoryError):
            api._scratch(nbytes, "cpu", None, small and (lambda: small))
    assert api._scratch(limit, "cpu", None, lambda: 64).numel() == limit


def test_scratch_is_recorded_on_the_stream_that_uses_it(monkeypatch):
    """A workspace the binding allocates is dropped when the call returns: the allocator has to know the stream the kernels
    run on, also where the caller passes its raw handle."""
    import torch

    class Stream:
        def __init__(self, handle, device=None):
            self.cuda_stream = handle
    seen = []
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: Stream(7))
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 7, raising=False)
    monkeypatch.setattr(torch.cuda, "ExternalStream", Stream)
    monkeypatch.setattr(torch.Tensor, "record_stream", lambda t, s: seen.append(s.cuda_stream))
    for stream in (None, 7, Stream(7)):
        api._scratch(64, "cpu", stream)
    assert seen == []
    for stream in (11, Stream(12), 0):
        api._scratch(64, "cpu", stream)
    assert seen == [11, 12, 0]
