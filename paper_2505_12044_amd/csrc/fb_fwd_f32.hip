// fp32 forward: attention with a factorised or dense additive bias, every product and sum in fp32
// (v_mfma_f32_32x32x2_f32 for the two contractions).  The full-precision path: 1e-4 against float64.
//
// Orientation as in the bf16 kernels: a query is a lane, the 32 keys of a block sit in that lane's
// sixteen accumulator registers and those of the lane 32 away,
//   S^T[key][query]   = [k | phi_k] . [q*scale | phi_q]      (A = key rows, B = query rows, in registers)
//   O^T[chan][query] += V^T . P^T                            (B = the registers S^T was left in)
// so the softmax is per lane plus one exchange, and P needs no data movement at all: k-step r of the
// second contraction pairs the keys that register r of the two halves stands for.
//
// Waves work on their own: one wave owns 32 queries (and, when the launch has too few tiles, every KW-th
// key block of them: the KW partial results are merged through LDS at the end).  Operands come straight
// from global memory, one phase ahead: key rows of the next block are requested when the score chain has
// released their registers and land under the value chain, value rows under the score chain.  No barrier and no
// staging in the loop.  Bound: the matrix pipe, (C + RP + C) / 2 k-steps of 64 cycles per 32 x 32 block.
// Measured, against the one-thread-per-query FMA kernel this replaced: B 2, H 8, N 1500, C 64, R 8 2725 -> 102 us
// (98 TFLOP/s of executed matrix work, 143 reached by a large fp32 matrix product on the same card); B 1, H 2,
// N 256, R 4 (16 tiles, eight waves each) 437 -> 11 us.  Requests pinned ahead of their chains instead of where the
// compiler sinks them, and buffer addressing (one address register per row block), were 135 -> 102 us of that.
#include <hip/hip_runtime.h>

#include "fb_f32_tiles.h"
#include "fb_launch.h"
#include "fb_params.h"

namespace {

constexpr int BK = 32;       // keys per block

template <int C, int RP>
struct Cfg {
    static constexpr int W = C + RP;
    static constexpr int NCH = W / 8;                      // 8-column chunks of the score contraction
    static constexpr int NPF = NCH <= 9 ? NCH : 8;         // chunks of key rows held in registers
    static constexpr int NCB = (C + 31) / 32;              // 32-channel tiles of the output
    static constexpr bool kTwo = W <= 144;                 // fits 256 registers: two waves per SIMD, eight waves per workgroup
    static constexpr int kMaxKw = kTwo ? 8 : 4;
    static constexpr int OP = C + 4;                       // row pitch of a partial result in LDS
    static constexpr int kSlot = 32 * OP + 64;             // floats: partial O, row maxima, row sums
};

template <int C, int RP, bool DENSE>
__global__ __launch_bounds__((Cfg<C, RP>::kTwo ? 512 : 256), (Cfg<C, RP>::kTwo ? 2 : 1)) void fwd_f32_kernel(FwdParams p, int kw_log2) {
    using K = Cfg<C, RP>;
    extern __shared__ __align__(16) float fsm[];
    const int L = (blockIdx.x & 7) * p.tiles_per_xcd + (blockIdx.x >> 3);      // contiguous runs of units per XCD
    if (L >= p.total_tiles) return;
    const int bh = L / p.n_units;
    const int u0 = L - bh * p.n_units;
    const int u = p.causal ? p.n_units - 1 - u0 : u0;      // causal: the tiles with the most keys first
    const int b = bh / p.H, h = bh - b * p.H;
    const int N = p.N, M = p.M, R = p.R;                   // N queries, M keys

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hf = lane >> 5;
    const int KW = 1 << kw_log2;
    const int part = wave & (KW - 1);                      // this wave's share of the keys
    const int qw = (int)(blockDim.x >> 6) >> kw_log2;      // tiles per workgroup
    const int q0 = (u * qw + (wave >> kw_log2)) * 32;
    const int qi = q0 + l32;
    const int qc = min(qi, N - 1);                         // rows past the end compute on the last row and are not stored

    const float* qrow = (const float*)p.q + ((size_t)bh * N + qc) * C;
    const float* pqrow = nullptr;
    F32Rows ks;
    ks.x = make_buf((const float*)p.k + (size_t)bh * M * C, (size_t)M * C * 4);
    ks.phi = ks.x;
    ks.R = R;
    if (RP > 0) {
        pqrow = (const float*)p.phi_q + (size_t)b * p.phi_bstride + ((size_t)h * N + qc) * R;
        ks.phi = make_buf((const float*)p.phi_k + (size_t)b * p.phik_bstride + (size_t)h * M * R, (size_t)M * R * 4);
    }
    const f32_buf vbuf = make_buf((const float*)p.v + (size_t)bh * M * C, (size_t)M * C * 4);
    const float* brow = nullptr;                           // this lane's bias row
    if (DENSE) brow = (const float*)p.bias + (size_t)b * p.bias_bstride + (size_t)h * N * M + (size_t)qc * M;

    f32x4 qr[K::NCH];
#pragma unroll
    for (int i = 0; i < K::NCH; i++) {
        qr[i] = own_chunk<C>(qrow, pqrow, R, i, hf);
        if (8 * i < C) qr[i] *= p.scale;
    }

    f32x16 o[K::NCB];
#pragma unroll
    for (int cb = 0; cb < K::NCB; cb++)
#pragma unroll
        for (int r = 0; r < 16; r++) o[cb][r] = 0.f;
    float m = -INFINITY, l = 0.f;

    const int n_keys = q0 >= N ? 0 : (p.causal ? min(M, q0 + 32) : M);
    const int nblk = (n_keys + BK - 1) / BK;

    f32x4 kc[K::NPF];
    auto load_k = [&](int blk, int i) __attribute__((always_inline)) {
        return row_chunk<C>(ks, (unsigned)(blk * BK + l32), i, hf);
    };
    float va[2][16];
    const int vcol = l32 & (C < 32 ? C - 1 : 31);
    auto load_v = [&](int blk, int cb) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 16; r++)
            va[cb & 1][r] = buf_f32(vbuf, (unsigned)(blk * BK + 4 * hf) * (C * 4u) + 4u * vcol + (8 * (r / 4) + r % 4) * (C * 4u) + cb * 128u);
    };
    float bv[DENSE ? 16 : 1];
    const bool bias_vec = DENSE && (M & 3) == 0;
    auto load_bias = [&](int blk) __attribute__((always_inline)) {
        if (!DENSE) return;
#pragma unroll
        for (int g = 0; g < 4; g++) {
            const int j = blk * BK + 8 * g + 4 * hf;
            if (bias_vec) {
                const f32x4 t = *(const f32x4*)(brow + min(j, M - 4));
#pragma unroll
                for (int x = 0; x < 4; x++) bv[(4 * g + x) % (DENSE ? 16 : 1)] = t[x];
            } else {
#pragma unroll
                for (int x = 0; x < 4; x++) bv[(4 * g + x) % (DENSE ? 16 : 1)] = brow[min(j + x, M - 1)];
            }
        }
    };

    if (part < nblk) {
#pragma unroll
        for (int i = 0; i < K::NPF; i++) kc[i] = load_k(part, i);
        load_bias(part);
    }
    for (int blk = part; blk < nblk; blk += KW) {
        const int nxt = min(blk + KW, nblk - 1);
        load_v(blk, 0);
        __builtin_amdgcn_sched_barrier(0);      // requests stay ahead of the chain they land under
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; r++) s[r] = 0.f;
#pragma unroll
        for (int i = 0; i < K::NCH; i++) {
            const f32x4 a = kc[i % K::NPF];
            if (i + K::NPF < K::NCH) kc[i % K::NPF] = load_k(blk, i + K::NPF);
#pragma unroll
            for (int e = 0; e < 4; e++) s = mfma32f(a[e], qr[i][e], s);
        }
        if (DENSE) {      // one rounding at the bias's size; a chain started from the bias would round each partial sum there
#pragma unroll
            for (int r = 0; r < 16; r++) s[r] += bv[r % (DENSE ? 16 : 1)];
        }
#pragma unroll
        for (int i = 0; i < K::NPF; i++) kc[i] = load_k(nxt, i);
        load_bias(nxt);
        if (K::NCB > 1) load_v(blk, 1);
        __builtin_amdgcn_sched_barrier(0);

        const int k0 = blk * BK;
        if (k0 + BK > M || (p.causal && k0 + BK - 1 > q0)) {
#pragma unroll
            for (int r = 0; r < 16; r++) {
                const int key = k0 + acc_row(r, hf);
                if (key >= M || (p.causal && key > qi)) s[r] = -INFINITY;
            }
        }
        // The maximum itself, however low it is; a row with no visible key yet (maximum -inf) keeps p = 0
        const float mnew = fmaxf(m, half_max(max16(s)));
        const float msub = mnew == -INFINITY ? 0.f : mnew;
        if (__any(mnew > m)) {
            const float alpha = fast_exp2((m - msub) * kLog2e);
            l *= alpha;
#pragma unroll
            for (int cb = 0; cb < K::NCB; cb++)
#pragma unroll
                for (int r = 0; r < 16; r++) o[cb][r] *= alpha;
            m = mnew;
        }
        float ps[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < 16; r++) {
            s[r] = fast_exp2((s[r] - msub) * kLog2e);
            ps[r & 3] += s[r];
        }
        l += (ps[0] + ps[1]) + (ps[2] + ps[3]);
#pragma unroll
        for (int cb = 0; cb < K::NCB; cb++) {
#pragma unroll
            for (int r = 0; r < 16; r++) o[cb] = mfma32f(va[cb & 1][r], s[r], o[cb]);
            if (cb + 2 < K::NCB) {
                load_v(blk, cb + 2);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    l = half_sum(l);

    float* og = (float*)p.out + (size_t)bh * N * C;
    if (KW == 1) {
        if (qi >= N) return;
        const float inv = 1.f / l;
#pragma unroll
        for (int cb = 0; cb < K::NCB; cb++)
#pragma unroll
            for (int g = 0; g < 4; g++) {
                const int c = cb * 32 + 8 * g;
                if (c >= C) continue;
                f32x4 t;
#pragma unroll
                for (int x = 0; x < 4; x++) t[x] = o[cb][4 * g + x] * inv;
                *(f32x4*)(og + (size_t)qi * C + c + 4 * hf) = t;
            }
        if (hf == 0) p.lse[(size_t)bh * N + qi] = m + __logf(l);
        return;
    }
    // merge the KW partial results of each tile: o = sum_w e^(m_w - m) O_w / sum_w e^(m_w - m) l_w
    float* slot = fsm + wave * K::kSlot;
#pragma unroll
    for (int cb = 0; cb < K::NCB; cb++)
#pragma unroll
        for (int g = 0; g < 4; g++) {
            const int c = cb * 32 + 8 * g;
            if (c >= C) continue;
            *(f32x4*)(slot + l32 * K::OP + c + 4 * hf) = f32x4{o[cb][4 * g], o[cb][4 * g + 1], o[cb][4 * g + 2], o[cb][4 * g + 3]};
        }
    if (hf == 0) {
        slot[32 * K::OP + l32] = m;
        slot[32 * K::OP + 32 + l32] = l;
    }
    __syncthreads();
    const float* tile0 = fsm + (wave - part) * K::kSlot;
    for (int e = part * 64 + lane; e < 32 * (C / 4); e += KW * 64) {
        const int row = e / (C / 4), c = (e % (C / 4)) * 4;
        if (q0 + row >= N) break;
        float mm = -INFINITY;
        for (int w = 0; w < KW; w++) mm = fmaxf(mm, tile0[w * K::kSlot + 32 * K::OP + row]);
        const float msub = mm == -INFINITY ? 0.f : mm;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        float lt = 0.f;
        for (int w = 0; w < KW; w++) {
            const float* t = tile0 + w * K::kSlot;
            const float a = fast_exp2((t[32 * K::OP + row] - msub) * kLog2e);
            lt = fmaf(a, t[32 * K::OP + 32 + row], lt);
            acc += a * *(const f32x4*)(t + row * K::OP + c);
        }
        acc *= 1.f / lt;
        *(f32x4*)(og + (size_t)(q0 + row) * C + c) = acc;
        if (c == 0) p.lse[(size_t)bh * N + q0 + row] = mm + __logf(lt);
    }
}

template <int C, int RP, bool DENSE>
int launch(const FwdParams& pin, hipStream_t stream) {
    using K = Cfg<C, RP>;
    auto kern = fwd_f32_kernel<C, RP, DENSE>;
    static FbLdsOnce once;
    FwdParams p = pin;
    const int tiles = (p.N + 31) / 32;
    const int kw = f32_split((long long)p.B * p.H * tiles, (p.M + BK - 1) / BK, K::kMaxKw);
    int kw_log2 = 0;
    while ((1 << kw_log2) < kw) kw_log2++;
    // four tiles a workgroup (two, one where waves share them), but no more than a head has: heads of up to 32 queries
    // are workgroups of one wave, of which a launch takes 2^26
    const int most = kw > 4 ? 1 : 4 / kw;
    const int qw = tiles < most ? tiles : most;
    const int waves = qw * kw;
    const size_t lds = kw > 1 ? (size_t)waves * K::kSlot * 4 : 0;
    if (lds > 0 && !fb_raise_lds_limit((const void*)kern, (size_t)K::kMaxKw * K::kSlot * 4, once)) return 1;
    p.n_units = (tiles + qw - 1) / qw;
    p.total_tiles = p.B * p.H * p.n_units;
    p.tiles_per_xcd = (p.total_tiles + 7) / 8;
    hipLaunchKernelGGL(kern, dim3(8 * p.tiles_per_xcd), dim3(waves * 64), lds, stream, p, kw_log2);
    return hipGetLastError() == hipSuccess ? 0 : 1;
}

template <int C>
int dispatch_c(const FwdParams& p, bool dense, hipStream_t stream) {
    if (dense) return launch<C, 0, true>(p, stream);
    if (p.R == 0) return launch<C, 0, false>(p, stream);
    if (p.R <= 8) return launch<C, 8, false>(p, stream);
    if (p.R <= 16) return launch<C, 16, false>(p, stream);
    if (p.R <= 32) return launch<C, 32, false>(p, stream);
    return launch<C, 64, false>(p, stream);
}

}  // namespace

// Returns 0 on success, 1 on launch failure, -1 when no instantiation fits.
int fb_launch_fwd_f32(const FwdParams& p, int C, bool dense, hipStream_t stream) {
    if (p.R > 64) return -1;
    switch (C) {
        case 16: return dispatch_c<16>(p, dense, stream);
        case 32: return dispatch_c<32>(p, dense, stream);
        case 64: return dispatch_c<64>(p, dense, stream);
        case 128: return dispatch_c<128>(p, dense, stream);
        default: return -1;
    }
}
