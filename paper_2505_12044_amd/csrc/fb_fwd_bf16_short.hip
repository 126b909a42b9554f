// bf16 MFMA forward for short key sequences on the 32-channel tiles (head dimensions 16 and 32), gfx950.
//
// At these sizes a query tile of the ring kernel (fb_fwd_bf16_impl.h) walks a dozen 32-key blocks, each with a staging
// step and a barrier around five matrix instructions: no pipe is busy (B 384, H 4, N 384, C 32, R 16: vector ALU 56 %,
// matrix pipe 21 %, a third of the wave time spent waiting).  Here a head's [K | phi_k] and V lie in LDS whole, and one
// workgroup per CU walks the heads: one wave per 32 query rows, no barrier inside a head, and the next head's rows
// travel global -> registers -> the second LDS buffer while this one is computed.  At that shape 71 -> 67 us, vector ALU
// 54 %, matrix pipe 21 %: the softmax mix of a block accounts for half of the time, in the other half the one workgroup of a
// CU loads, drains or waits at its barrier.  Causal, short and single-round calls gain more (see fb_short_fwd).
//
// Orientation, softmax and the rounding of the operands are those of the ring kernel: a query is a lane, the scores of
// a 32-key block sit in its accumulator registers, lazy reference maximum.  A wave takes its rows' first block alone,
// for the reference: key 0's, as the ring kernel does, so P is rounded to bf16 at the same scale and the sums follow in
// the same order (the same bits; full attention), or the diagonal one when causal.  The other blocks follow two at a
// time, so the score chain of one overlaps the exponentials of the other.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "fb_device.h"
#include "fb_launch.h"
#include "fb_params.h"

namespace {

constexpr int kMaxWaves = 12;          // three waves per SIMD: 168 registers, and none saved for a fourth (amdgpu_waves_per_eu)
constexpr size_t kLdsBytes = 160 * 1024;
constexpr float kSumLimit = 256.0f;    // see fb_fwd_bf16_impl.h

// LDS image of a head: K rows, V rows (CG channels, unpadded, in 16-byte pieces whose place in a 64-byte row is swizzled
// so that row reads and transpose reads are conflict-free), factor rows (pitch an odd number of 16-byte pieces).
template <int CG, int RP>
struct Cfg {
    static constexpr int KC = CG / 16, KS = (CG + RP) / 16;            // k-steps of the score contraction: channels, all
    static constexpr int RB = CG * 2;                                  // bytes of a k (or v) row
    static constexpr int PP = RP == 0 ? 0 : RP == 16 ? 32 : RP * 2 + 16;
    static constexpr int PCH = RP / 8;                                 // 16-byte pieces of a factor row
    static constexpr int kRow = 2 * RB + PP;                           // LDS bytes per key and buffer
    FB_DEV static int swz(int row) { return CG == 32 ? (row >> 2) & 3 : 0; }
};

// lane l reads sbase + voff (bytes); its 16 bytes land at LDS byte address lds_addr + 16 * l.  Inline assembly, because
// behind the builtin the compiler makes every LDS read wait for all of them.
FB_DEV void dma16(const void* sbase, unsigned voff, unsigned lds_addr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :: "v"(voff), "s"(sbase), "s"(lds_addr) : "memory", "m0");
}

// PM: 0 = no factors, 1 = bf16 factors in whole 16-byte pieces (R % 8 == 0), 2 = bf16 factors of any R, 3 = fp32 factors
template <int CG, int RP, int PM, bool CAUSAL>
__global__ __launch_bounds__(kMaxWaves * 64) __attribute__((amdgpu_waves_per_eu(3, 3))) void fwd_short_kernel(FwdParams p, int heads) {
    using K = Cfg<CG, RP>;
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr bool F32 = PM == 3;
    constexpr bool FOLD = score_log2e(CG, F32);
    const float emul = FOLD ? 1.f : kLog2e;
    // N = M: a wave to every 32 queries and to every 32 keys, so a head's factor pieces are PIT whole rounds of threads
    const int N = p.N, M = p.M, R = p.R;
    const int NT = blockDim.x, nw = NT >> 6;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hf = lane >> 5;
    const int nkb = (M + 31) >> 5, Mp = nkb * 32;
    const unsigned buf_bytes = (unsigned)(Mp * K::kRow), voff0 = (unsigned)(Mp * K::RB), poff0 = 2 * voff0;
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
    const size_t esz = F32 ? 4 : 2;

    // ---- a head's k and v rows: direct loads of 64 pieces, dealt to the waves (rows past M repeat row M - 1) ----
    constexpr int RPD = 1024 / K::RB;        // rows per direct load
    const unsigned drow = (unsigned)lane / (K::RB / 16);
    const unsigned dcol = (((unsigned)lane % (K::RB / 16)) ^ (unsigned)K::swz((int)drow)) * 16;   // RPD is a multiple of 16: the swizzle repeats
    auto issue_kv = [&](int bh, unsigned buf) __attribute__((always_inline)) {
        const unsigned char* kg = (const unsigned char*)p.k + (size_t)bh * M * K::RB;
        const unsigned char* vg = (const unsigned char*)p.v + (size_t)bh * M * K::RB;
        for (int d = wave; d < Mp / RPD; d += nw) {
            const unsigned off = min((unsigned)(d * RPD) + drow, (unsigned)(M - 1)) * K::RB + dcol;
            dma16(kg, off, lds0 + buf + d * 1024);
            dma16(vg, off, lds0 + buf + voff0 + d * 1024);
        }
    };
    // ---- factor rows, piece by piece through registers ----
    auto phi_piece = [&](int bh, int e) __attribute__((always_inline)) {
        const int b = bh / p.H, h = bh - b * p.H;
        const unsigned row = min((unsigned)e / (K::PCH > 0 ? K::PCH : 1), (unsigned)(M - 1));
        const int c8 = (unsigned)e % (K::PCH > 0 ? K::PCH : 1);
        const unsigned char* src =
            (const unsigned char*)p.phi_k + ((size_t)b * p.phik_bstride + ((size_t)h * M + row) * R) * esz;
        if (PM == 1) return c8 * 8 < R ? *(const u32x4*)(src + c8 * 16) : u32x4{0u, 0u, 0u, 0u};
        return phi_chunk_raw(src, c8, R, F32, true);
    };
    auto phi_store = [&](unsigned buf, int e, const u32x4& raw) __attribute__((always_inline)) {
        const unsigned row = (unsigned)e / (K::PCH > 0 ? K::PCH : 1);
        const int c8 = (unsigned)e % (K::PCH > 0 ? K::PCH : 1);
        *(u32x4*)(smem + buf + poff0 + row * K::PP + c8 * 16) = PM == 1 ? raw : as_uint4(phi_chunk_finish<false>(raw, c8, F32));
    };
    constexpr int PIT = K::PCH / 2;      // pieces of a thread, in flight together
    static_assert(2 * PIT == K::PCH, "whole rounds");

    // ---- query rows: raw in registers while they travel ----
    u32x4 qraw[K::KC];
    bf16x8 qphi[RP / 16 > 0 ? RP / 16 : 1];
    const int qw0 = wave * 32;      // first query row of this wave
    auto load_q = [&](int bh) __attribute__((always_inline)) {
        const int b = bh / p.H, h = bh - b * p.H;
        const int qi = min(qw0 + l32, N - 1);
        const bf16_t* q = (const bf16_t*)p.q + ((size_t)bh * N + qi) * CG + 8 * hf;
#pragma unroll
        for (int ks = 0; ks < K::KC; ks++) qraw[ks] = *(const u32x4*)(q + ks * 16);
        if (RP > 0) {
            const unsigned char* src = (const unsigned char*)p.phi_q + ((size_t)b * p.phi_bstride + ((size_t)h * N + qi) * R) * esz;
#pragma unroll
            for (int ks = 0; ks < RP / 16; ks++) {
                const int c8 = ks * 2 + hf;
                if (PM == 1) qphi[ks] = as_bf16x8(c8 * 8 < R ? *(const u32x4*)(src + c8 * 16) : u32x4{0u, 0u, 0u, 0u});
                else qphi[ks] = phi_chunk_gather<true>(src, c8, R, F32, FOLD ? kLog2e : 1.f);
            }
        }
    };

    int bh = blockIdx.x;
    if (bh >= heads) return;
    issue_kv(bh, 0);
    load_q(bh);
#pragma unroll
    for (int it = 0; it < PIT; it++) phi_store(0, tid + it * NT, phi_piece(bh, tid + it * NT));
    __builtin_amdgcn_s_waitcnt(0x0F70);      // vmcnt(0)
    __syncthreads();

    // ---- LDS operand addresses (bytes inside a 32-key tile) ----
    const int i16 = lane & 15, blk16 = CG == 32 ? l32 >> 4 : 0;
    unsigned krow[K::KC], vtr[2];
#pragma unroll
    for (int ks = 0; ks < K::KC; ks++) krow[ks] = l32 * K::RB + (((2 * ks + hf) ^ K::swz(l32)) << 4);
    const unsigned prow = l32 * K::PP + hf * 16;
#pragma unroll
    for (int hi = 0; hi < 2; hi++) {
        const int row = 8 * hi + 4 * hf + (i16 >> 2);
        vtr[hi] = row * K::RB + (((2 * blk16 + ((i16 & 3) >> 1)) ^ K::swz(row)) << 4) + (i16 & 1) * 8;
    }

    unsigned buf = 0;
    for (;;) {
        const unsigned nbuf = buf_bytes - buf;
        const int next = bh + (int)gridDim.x;
        const bool more = next < heads;                             // workgroup-uniform

        bf16x8 qreg[K::KS];
        const float qscale = FOLD ? p.scale * kLog2e : p.scale;
#pragma unroll
        for (int ks = 0; ks < K::KS; ks++) {
            if (ks < K::KC) {
                const bf16x8 x = as_bf16x8(qraw[ks]);
#pragma unroll
                for (int e = 0; e < 8; e++) qreg[ks][e] = (bf16_t)((float)x[e] * qscale);
            } else {
                qreg[ks] = qphi[ks - K::KC];
            }
        }
        // everything the next head reads is requested here and met at the end of this one
        u32x4 praw[PIT > 0 ? PIT : 1];
        if (more) {
            issue_kv(next, nbuf);
            load_q(next);
#pragma unroll
            for (int it = 0; it < PIT; it++) praw[it] = phi_piece(next, tid + it * NT);
        }

        f32x16 oacc;
        float mref = -INFINITY, lsum = 0.f;
#pragma unroll
        for (int r = 0; r < 16; r++) oacc[r] = 0.f;

        // NB blocks starting at key block kb; FIRST: the one that gives every row its reference; MASK: it may be partial or
        // the diagonal one
        auto step = [&](int kb, auto nb_tag, auto first_tag, auto mask_tag) __attribute__((always_inline)) {
            constexpr int NB = decltype(nb_tag)::value;
            constexpr bool FIRST = decltype(first_tag)::value, MASK = decltype(mask_tag)::value;
            static_assert(NB == 1 || !(FIRST || MASK), "two blocks: plain ones");
            f32x16 s[NB];
            bf16x8 va[NB][2];
            const unsigned char* kt = smem + (buf + kb * 32 * K::RB);
            const unsigned char* pt = smem + (buf + poff0 + kb * 32 * K::PP);
#pragma unroll
            for (int b = 0; b < NB; b++) {
#pragma unroll
                for (int r = 0; r < 16; r++) s[b][r] = 0.f;
#pragma unroll
                for (int ks = 0; ks < K::KS; ks++) {
                    const bf16x8 a = as_bf16x8(ks < K::KC ? *(const u32x4*)(kt + krow[ks < K::KC ? ks : 0] + b * 32 * K::RB)
                                                          : *(const u32x4*)(pt + prow + b * 32 * K::PP + (ks - K::KC) * 32));
                    s[b] = mfma32(a, qreg[ks], s[b]);
                }
            }
#pragma unroll
            for (int b = 0; b < NB; b++)
#pragma unroll
                for (int kk = 0; kk < 2; kk++)
                    va[b][kk] = join_tr(lds_read_tr16((const bf16_t*)(kt + voff0 + vtr[0] + (2 * b + kk) * 16 * K::RB)),
                                        lds_read_tr16((const bf16_t*)(kt + voff0 + vtr[1] + (2 * b + kk) * 16 * K::RB)));
            bf16x8 pb[NB][2];
            // P = exp2(S log2e - mref), packed, and this lane's row sum of block b
            auto exps = [&](int b, float nm) __attribute__((always_inline)) {
                float ps[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int r = 0; r < 16; r += 2) {
                    const bf16x2 pr2 = {(bf16_t)fast_exp2(fmaf(s[b][r], emul, nm)), (bf16_t)fast_exp2(fmaf(s[b][r + 1], emul, nm))};
                    ps[(r >> 1) & 3] = pair_sum(pr2, ps[(r >> 1) & 3]);
                    pb[b][r / 8][r % 8] = pr2[0];
                    pb[b][r / 8][r % 8 + 1] = pr2[1];
                }
                return (ps[0] + ps[1]) + (ps[2] + ps[3]);
            };
            if (MASK && (CAUSAL || kb * 32 + 32 > M)) {
                const int qi = qw0 + l32;
#pragma unroll
                for (int r = 0; r < 16; r++) {
                    const int key = kb * 32 + 8 * (r / 4) + 4 * hf + (r % 4);
                    if (key >= M || (CAUSAL && key > qi)) s[0][r] = -INFINITY;
                }
            }
            if constexpr (FIRST) mref = fmaxf(half_max(max16(s[0])) * emul, -1e30f);
            float psum[NB], all = 0.f;
#pragma unroll
            for (int b = 0; b < NB; b++) {
                psum[b] = exps(b, -mref);
                all += psum[b];
            }
            if (!FIRST && __any(!(all < kSumLimit))) {
                // rare: the scores may have outgrown the reference.  Block by block, as the ring kernel does: where a
                // block's own sum says so, take its true maximum, rescale, redo the exponentials
                asm volatile("" ::: "memory");
#pragma unroll
                for (int b = 0; b < NB; b++) {
                    if (!__any(!(psum[b] < kSumLimit))) continue;
                    const float mx = half_max(max16(s[b])) * emul;
                    if (__any(mx > mref)) {
                        const float mnew = fmaxf(mref, mx);
                        const float alpha = fast_exp2(mref - mnew);
                        mref = mnew;
                        if (b == 1) {      // the block before belongs to what is rescaled
                            lsum += psum[0];
                            psum[0] = 0.f;
#pragma unroll
                            for (int kk = 0; kk < 2; kk++) {
                                oacc = mfma32(va[0][kk], pb[0][kk], oacc);
                                pb[0][kk] = as_bf16x8(u32x4{0u, 0u, 0u, 0u});
                            }
                        }
                        lsum *= alpha;
#pragma unroll
                        for (int r = 0; r < 16; r++) oacc[r] *= alpha;
#pragma unroll
                        for (int x = b + 1; x < NB; x++) psum[x] = exps(x, -mref);
                    }
                    psum[b] = exps(b, -mref);
                }
            }
#pragma unroll
            for (int b = 0; b < NB; b++) {
                lsum += psum[b];
#pragma unroll
                for (int kk = 0; kk < 2; kk++) oacc = mfma32(va[b][kk], pb[b][kk], oacc);
            }
        };
        using One = std::integral_constant<int, 1>;
        using Two = std::integral_constant<int, 2>;

        using Yes = std::true_type;
        using No = std::false_type;
        using Tail = std::integral_constant<bool, !CAUSAL>;
        const int whole = CAUSAL ? wave : M >> 5, end = CAUSAL ? wave : nkb;      // blocks without masks; all blocks but the first one taken
        step(CAUSAL ? wave : 0, One{}, Yes{}, Yes{});
        int kb = CAUSAL ? 0 : 1;
        for (; kb + 2 <= whole; kb += 2) step(kb, Two{}, No{}, No{});
        for (; kb < end; kb++) step(kb, One{}, No{}, Tail{});
        if (more) {
            // the next head's rows have landed before anyone reads them; the stores of the results follow behind the
            // barrier, so nothing waits for them until the next head ends
#pragma unroll
            for (int it = 0; it < PIT; it++) phi_store(nbuf, tid + it * NT, praw[it]);
            __builtin_amdgcn_s_waitcnt(0x0F70);      // vmcnt(0)
            __syncthreads();
        }
        // ---- epilogue: o = O / l, lse = m + ln l ----
        const int qi = qw0 + l32;
        const float ltot = half_sum(lsum);
        const float inv = 1.f / ltot;
        if (qi < N) {
            bf16_t* og = (bf16_t*)p.out + ((size_t)bh * N + qi) * CG;
#pragma unroll
            for (int g = 0; g < 4; g++) {
                if (8 * g >= CG) continue;
                bf16x4 o4;
#pragma unroll
                for (int x = 0; x < 4; x++) o4[x] = (bf16_t)(oacc[4 * g + x] * inv);
                *(u32x2*)(og + 8 * g + 4 * hf) = __builtin_bit_cast(u32x2, o4);
            }
            if (hf == 0) p.lse[(size_t)bh * N + qi] = (mref + __log2f(ltot)) * kLn2;
        }
        if (!more) break;
        buf = nbuf;
        bh = next;
    }
}

template <int CG, int RP, int PM, bool CAUSAL>
int launch(const FwdParams& p, int nw, int cus, hipStream_t stream) {
    using K = Cfg<CG, RP>;
    auto kern = fwd_short_kernel<CG, RP, PM, CAUSAL>;
    static FbLdsOnce once;
    if (!fb_raise_lds_limit((const void*)kern, kLdsBytes, once)) return 1;
    const int heads = p.B * p.H;
    const size_t lds = (size_t)2 * (32 * nw) * K::kRow;
    // workgroups that stay resident: by LDS and by the twelve waves that the registers allow
    const long long per_cu = kMaxWaves / nw < (int)(kLdsBytes / lds) ? kMaxWaves / nw : (long long)(kLdsBytes / lds);
    const long long most = (long long)cus * (per_cu < 1 ? 1 : per_cu);
    hipLaunchKernelGGL(kern, dim3((unsigned)(heads < most ? heads : most)), dim3(64 * nw), lds, stream, p, heads);
    return hipGetLastError() == hipSuccess ? 0 : 1;
}

template <int CG, int RP, int PM>
int dispatch_causal(const FwdParams& p, int nw, int cus, hipStream_t stream) {
    return p.causal ? launch<CG, RP, PM, true>(p, nw, cus, stream) : launch<CG, RP, PM, false>(p, nw, cus, stream);
}
template <int CG, int RP>
int dispatch_pm(const FwdParams& p, int nw, int cus, hipStream_t stream) {
    if (p.phi_f32) return p.causal ? launch<CG, RP, 3, true>(p, nw, cus, stream) : -1;
    if (p.R % 8 == 0) return dispatch_causal<CG, RP, 1>(p, nw, cus, stream);
    return dispatch_causal<CG, RP, 2>(p, nw, cus, stream);
}
template <int CG>
int dispatch_rp(const FwdParams& p, int rp, int nw, int cus, hipStream_t stream) {
    switch (rp) {
        case 0: return dispatch_causal<CG, 0, 0>(p, nw, cus, stream);
        case 16: return dispatch_pm<CG, 16>(p, nw, cus, stream);
        case 32: return dispatch_pm<CG, 32>(p, nw, cus, stream);
        default: return -1;
    }
}

}  // namespace

// Self-attention whose keys fit LDS twice.  Kernel times against the ring kernel's (ring / this), 16 to 4096 heads of every
// length in steps of 32, 256 CUs.  Heads are dealt one at a time to a workgroup that stays, so what counts beyond one head a
// CU is how full the last round is; the ring kernel's tiles have rounds of their own, three times finer.
// Full attention, bf16 factors:
//   up to 128 keys it is the faster one throughout (C 32, R 16 1.0-1.7; C 16 1.0-2.1; no factors 1.0);
//   C 32 beyond: below five eighths of the CUs 0.94-1.0; one round 1.13-1.24 (up to 192 keys 1.20); two rounds 0.85-0.96
//   where the second is nearly empty (280 heads), 1.04-1.10 where it is full; then up to 192 keys 0.97-1.12, up to 256 keys
//   1.0-1.05 in a full third round and 0.91-0.98 after it, beyond 256 keys 1.0-1.13 in full rounds and 0.85-0.97 in others;
//   C 16: the same shape of line, some 5 % (up to 256 keys) and 15 % (beyond) higher;
//   32 factor columns at C 32: only where the heads fill one round (1.10-1.35; beyond it 0.90-0.94, some registers spill);
//   no factors, or C 16 with R 8: 0.95-1.02, not beyond 128 keys (at 128 in many rounds 0.93-0.96).
//   fp32 factors are split once a head, but only by one workgroup: 0.7-0.95, never.
// Causal the ring kernel's 128-row tiles do up to twice the work: 1.04-1.9 throughout, but for 32 factor columns at many
// heads (0.95-0.98) and fp32 factors (N 256: 256 heads 18.6 / 12.9 us, 400 heads 21.4 / 21.7).
bool fb_short_fwd(const FwdParams& p, int C, int rp) {
    if (C > 32 || rp > 32 || p.N != p.M || p.slopes != nullptr) return false;
    const long long BH = (long long)p.B * p.H;
    const int nkb = (p.M + 31) / 32;
    if (nkb > kMaxWaves || BH >= (1LL << 30)) return false;
    const size_t row = C == 16 ? (rp == 0 ? Cfg<16, 0>::kRow : rp == 16 ? Cfg<16, 16>::kRow : Cfg<16, 32>::kRow)
                               : (rp == 0 ? Cfg<32, 0>::kRow : rp == 16 ? Cfg<32, 16>::kRow : Cfg<32, 32>::kRow);
    if ((size_t)2 * nkb * 32 * row > kLdsBytes) return false;
    const int cus = fb_cu_count();
    if (cus <= 0) return false;
    if (rp > 0 && p.phi_f32) return p.causal && (nkb > 8 || (nkb > 4 && BH <= cus));
    const bool wide = C == 32 && rp == 32;
    if (p.causal) return !wide || nkb <= 4 || nkb > 8 || BH <= 2LL * cus;
    const FbHeadRounds r = fb_head_rounds(BH, cus);
    const bool light = rp == 0 || (C == 16 && rp == 16 && p.R % 8 == 0);
    if (nkb <= 4) return nkb <= 3 || !light || r.rounds <= 8;
    if (light) return false;
    if (wide) return BH * 8 >= 5LL * cus && BH <= cus;
    if (C == 32 ? BH * 8 < 5LL * cus : nkb > 8 && BH * 2 < cus) return false;
    if (r.rounds == 1) return true;
    if (C == 16) return r.fill >= (nkb > 8 ? 0.72 : r.rounds == 2 ? 0.76 : r.rounds == 3 ? 0.8 : 0.92);
    if (nkb <= 6) return r.rounds > 2 || r.fill >= 0.76;
    if (nkb <= 8) return r.rounds <= 3 && r.fill >= (r.rounds == 2 ? 0.76 : 0.85);
    return r.fill >= (r.rounds == 2 ? 0.75 : 0.97);
}

int fb_launch_fwd_bf16_short(const FwdParams& p, int C, int rp, hipStream_t stream) {
    const int cus = fb_cu_count(), nw = (p.N + 31) / 32;
    if (cus <= 0) return 1;
    return C == 16 ? dispatch_rp<16>(p, rp, nw, cus, stream) : dispatch_rp<32>(p, rp, nw, cus, stream);
}
