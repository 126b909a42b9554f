// fp32 backward of attention with a factorised (or materialised) additive bias, every product and sum in
// fp32 (v_mfma_f32_32x32x2_f32); the full-precision companion of fb_fwd_f32.hip.
//
// With S = [q*scale | phi_q] . [k | phi_k]^T (FlashBias Eq. 3), P = exp(S - lse) and
// D_i = sum_c dout_ic out_ic, the gradient of the scores is dS = P o (dout V^T - D), and
//   [dq / scale | dphi_q] = dS   [k | phi_k]          (query-side launch, one pass over the keys)
//   [dk / scale | dphi_k / 1] = dS^T [q | phi_q]      (key-side launch, one pass over the queries)
//   dv                    = P^T  dout
// so the factor gradients are the trailing R columns of the contractions that give dq and dk
// (Sec. 3.2 "Speed up training").  Nothing N x N is stored; each launch recomputes S and dP.
// Deterministic: every output element is summed in a fixed order, without atomics.
//
// One wave owns 32 rows of its side (lanes), the streamed side comes in blocks of 32 rows (accumulator
// registers): S and dP take the streamed rows as row operands (16 bytes a lane) and their results are,
// register for register, the second operand of the output contractions, whose first operand is the
// streamed rows read down their columns (4 bytes a lane, 128 bytes in a row).  Both come straight from
// global memory into registers ahead of their use (rows: NPF chunks of four k-steps, columns: one tile of
// sixteen k-steps); a k-step holds the matrix pipe for 64 cycles, so the vector cache keeps up
// and the loop has no barrier and no LDS.  Bound: the matrix pipe.  The query-side launch also writes D
// into the caller's workspace for the key-side launch behind it.
// Measured, B 2, H 8, N 1500, C 64, R 8: 874 -> 169 us (query side) and 955 -> 253 us (key side, whose accumulators
// leave one wave per SIMD) against the four-threads-per-row FMA kernel this replaced.
// Where the tiles are too few to fill the chip, KW waves share one and take every KW-th block each; their
// sums meet in LDS at the end.
#include <hip/hip_runtime.h>

#include <cmath>

#include "fb_f32_tiles.h"
#include "fb_launch.h"
#include "fb_params.h"

namespace {

constexpr int kThreads = 256;
constexpr int BT = 32;       // streamed rows per block
constexpr int OPITCH = 36;   // row pitch of an output tile in LDS (floats)

// dS of one head, whole tiles (any int: the size queries come before the limits are checked).
size_t ds_head_bytes(int N, int M) {
    const size_t pairs = (((size_t)N + 31) & ~(size_t)31) * (((size_t)M + 31) & ~(size_t)31);      // at most 2^62
    return pairs > (SIZE_MAX >> 2) ? SIZE_MAX : pairs * 4;
}
size_t d_bytes(long long rows) { return ((size_t)rows * 4 + 255) & ~(size_t)255; }
// At most this much dS at a time.  (256 MB, what the last-level cache holds, cuts B 16, H 4, N 1500, C 64 into three
// launches whose tiles fill the chip badly: 1514 us; in one 1084, recomputed 1329.)
constexpr size_t kMaxStored = (size_t)1 << 30;
// Heads whose dS the workspace takes at a time, 0 where the query side recomputes it.  Stored against recomputed,
// kernel times (us): C 32, R 8 64 heads of N 1024 333 / 290; C 64 16 heads of N 1500 372 / 301; C 128 790 / 553; from
// the smallest calls on (C 64, 2 heads of 256 34 / 29), where one launch more costs the host what it saves: left to
// recompute below about 60 us.  In one launch neither the mask nor short heads move the line (backward calls, before / now):
// causal C 32, 64 heads of 1024 323 / 263; C 64, 262144 heads of one row 13455 / 10948, 4096 of 65 causal 628 / 525, 4096 of 4 x 512
// 1549 / 1218.  Not at 16 channels: a block's recomputation takes 1300 cycles of the matrix pipe, its
// 8 KB to memory and back more.
// Several launches (C 32 and 64; at 128 channels 1.06-2.0 throughout): each has a tail of its own.  Of 2048 waves at a time
// (f32_split) one tile each, a launch of 2204 tiles takes two rounds: C 64, 76 heads of N 3700 9554 / 10385 us, cut smaller 9528 / 8305.
// Causal tiles differ in length, and a launch's few heads fall unevenly on the XCDs: N 3700, 38 to 120 heads 0.77-0.92, N 8192,
// 16 heads 0.83, N 2500 and 3000 0.95-1.13, up to N 2000 (4096 tiles a launch) 0.98-1.26: from there on.
int stored_heads(long long heads, int N, int M, int C, bool causal, size_t avail) {
    if (avail > kMaxStored) avail = kMaxStored;
    long long fit = (long long)(avail / ds_head_bytes(N, M));
    if (fit <= 0) return 0;
    const long long nq = ((long long)N + 31) / 32, nk = ((long long)M + 31) / 32, tiles = nq < nk ? nq : nk;
    if ((double)heads * nq * nk * C < 262144.0) return 0;
    for (;;) {
        const long long parts = (heads + fit - 1) / fit, chunk = (heads + parts - 1) / parts;
        if (parts == 1) return (int)heads;
        // worth filling the chip (four waves to a 32-row tile)
        if (chunk * tiles < (causal && C <= 64 ? 4096 : 512)) return 0;
        const long long whole = chunk * tiles / 2048 * 2048;
        if (causal || whole == 0 || chunk * tiles * 10 >= (whole + 2048) * 6 || chunk * tiles == whole || whole < tiles) return (int)chunk;
        fit = whole / tiles;      // fewer heads, full rounds
    }
}

template <int C, int RP, bool KEYSIDE>
struct Cfg {
    static constexpr int W = C + RP;
    static constexpr int NCH = W / 8, NC2 = C / 8;         // row chunks of S and of dP
    static constexpr int NALL = NCH + NC2;
    static constexpr int NPF = NALL < 6 ? NALL : 6;        // row chunks in flight
    static constexpr int TA = (W + 31) / 32;               // 32-column tiles of d[x | phi]
    static constexpr int TE = KEYSIDE ? (C + 31) / 32 : 0; // ... of dv
    static constexpr int kRegs = (W + C) / 2 + 16 * (TA + TE) + 32 + 4 * NPF + 32 + (KEYSIDE ? 32 : 0);
    static constexpr int kMinWaves = kRegs <= (C == 16 ? 190 : 225) ? 2 : 1;      // waves per SIMD the registers allow
};

// KEYSIDE = false: lanes are queries, keys are streamed; outputs dq, dphi_q, D (and dBias when DENSE).
// KEYSIDE = true:  lanes are keys, queries are streamed; outputs dk, dv, dphi_k.
// DENSE: the bias is a materialised [N, M] matrix per head, added to the scores (the
// training-side baseline of Sec. 4.3); dBias = dS is written by the query-side launch, zero where masked.
// dS: the heads head0.. of this launch, dS transposed, [keys][queries] padded to whole tiles (STORE: written; the query
// side's second contraction is then a launch of its own, bwd_f32_dq_kernel).
// QSCALE (key side): the scale is multiplied into the streamed q rows, as the forward and the query side do, so that both
// sides hold the same scores to the bit; without it the lane's k row carries it (a power of two: the same bits).
template <int C, int RP, bool KEYSIDE, bool DENSE = false, bool STORE = false, bool QSCALE = false>
__global__ __launch_bounds__(kThreads, (Cfg<C, RP, KEYSIDE>::kMinWaves)) void bwd_f32_kernel(BwdParams p, float* __restrict__ Dws, int kw_log2, float* __restrict__ dS, int head0) {
    static_assert(!(STORE || QSCALE) || (KEYSIDE && !DENSE), "the key side stores dS");
    using K = Cfg<C, RP, KEYSIDE>;
    __shared__ __align__(16) float otile[kThreads / 64][32 * OPITCH];
    const int L = (blockIdx.x & 7) * p.tiles_per_xcd + (blockIdx.x >> 3);      // contiguous runs of units per XCD
    if (L >= p.total_tiles) return;
    const int bhl = L / p.n_tiles;                         // p.n_tiles: workgroups per (b, h)
    const int u0 = L - bhl * p.n_tiles, bh = head0 + bhl;
    const int u = (p.causal && !KEYSIDE) ? p.n_tiles - 1 - u0 : u0;      // causal: long tiles first
    const int b = bh / p.H, h = bh - b * p.H;
    const int N = p.N, M = p.M, R = p.R;                   // N queries, M keys
    const int NL = KEYSIDE ? M : N;                        // rows on the lane side
    const int NO = KEYSIDE ? N : M;                        // rows on the streamed side

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hf = lane >> 5;
    const int KW = 1 << kw_log2;
    const int part = wave & (KW - 1);
    const int tile = u * ((kThreads / 64) >> kw_log2) + (wave >> kw_log2);
    const int row0 = tile * 32;
    const int row = row0 + l32;
    const int rowc = min(row, NL - 1);                     // rows past the end compute on the last row and are not stored

    const size_t qbase = (size_t)bh * N * C, kbase = (size_t)bh * M * C;
    const float* pq = RP > 0 ? (const float*)p.phi_q + (size_t)b * p.phi_bstride + (size_t)h * N * R : nullptr;
    const float* pk = RP > 0 ? (const float*)p.phi_k + (size_t)b * p.phik_bstride + (size_t)h * M * R : nullptr;
    const float* qg = (const float*)p.q + qbase;
    const float* kg = (const float*)p.k + kbase;
    const float* vg = (const float*)p.v + kbase;
    const float* dog = (const float*)p.dout + qbase;
    const float* lseg = p.lse + (size_t)bh * N;
    float* Dg = Dws + (size_t)bh * N;
    // lane-side rows
    const float* xrow = (KEYSIDE ? kg : qg) + (size_t)rowc * C;
    const float* prow = RP > 0 ? (KEYSIDE ? pk : pq) + (size_t)rowc * R : nullptr;
    const float* erow = (KEYSIDE ? vg : dog) + (size_t)rowc * C;
    // streamed arrays
    F32Rows oth;
    oth.x = make_buf(KEYSIDE ? qg : kg, (size_t)NO * C * 4);
    oth.phi = RP > 0 ? make_buf(KEYSIDE ? pq : pk, (size_t)NO * R * 4) : oth.x;
    oth.R = R;
    const f32_buf eoth = make_buf(KEYSIDE ? dog : vg, (size_t)NO * C * 4);
    const f32_buf lbuf = make_buf(lseg, (size_t)N * 4), dbuf = make_buf(Dg, (size_t)N * 4);
    const float* bg = nullptr;
    float* dbg = nullptr;
    if (DENSE) {
        bg = (const float*)p.bias + (size_t)b * p.bias_bstride + (size_t)h * N * M;
        dbg = (float*)p.dbias + (size_t)bh * N * M;
    }

    // ---- lane-side operands: the scale sits on the lane side's x columns (QSCALE: on the streamed side's) ----
    f32x4 ar[K::NCH], er[K::NC2];
#pragma unroll
    for (int i = 0; i < K::NCH; i++) {
        ar[i] = own_chunk<C>(xrow, prow, R, i, hf);
        if (8 * i < C && !QSCALE) ar[i] *= p.scale;
    }
#pragma unroll
    for (int i = 0; i < K::NC2; i++) er[i] = *(const f32x4*)(erow + 8 * i + 4 * hf);
    float lse_r = 0.f, d_r = 0.f;
    if (!KEYSIDE) {
        const float* orow = (const float*)p.out + qbase + (size_t)rowc * C;
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < K::NC2; i++) {
            const f32x4 x = *(const f32x4*)(orow + 8 * i + 4 * hf);
#pragma unroll
            for (int e = 0; e < 4; e++) sum = fmaf(er[i][e], x[e], sum);
        }
        d_r = half_sum(sum);
        lse_r = lseg[rowc];
        if (part == 0 && hf == 0 && row < NL) Dg[row] = d_r;
    }

    f32x16 acca[K::TA], acce[K::TE > 0 ? K::TE : 1];
#pragma unroll
    for (int r = 0; r < 16; r++) {
#pragma unroll
        for (int t = 0; t < K::TA; t++) acca[t][r] = 0.f;
#pragma unroll
        for (int t = 0; t < (K::TE > 0 ? K::TE : 1); t++) acce[t][r] = 0.f;
    }

    // ---- streamed blocks [b0, b1): with a causal mask (N = M) the tile's own block is the diagonal one ----
    const int nall = (NO + BT - 1) / BT;
    int b0 = 0, b1 = nall;
    if (p.causal) {
        if (KEYSIDE) b0 = min(tile, nall);
        else b1 = min(nall, tile + 1);
    }
    if (row0 >= NL) b1 = b0 = 0;

    // row operands, chunk n of a block: S chunks, then dP chunks
    f32x4 rc[K::NPF];
    auto load_row = [&](int blk, int n) __attribute__((always_inline)) {
        const unsigned r = (unsigned)(blk * BT + l32);
        return n < K::NCH ? row_chunk<C>(oth, r, n, hf) : buf_f32x4(eoth, r * (C * 4u) + 16u * hf + 32u * (n - K::NCH));
    };
    // column operands, tile t of a block: dv tiles (of the streamed dout rows), then d[x | phi] tiles.  Columns
    // past C + R read some real element (computed, never stored).
    constexpr int NT = K::TE + K::TA;
    float cc[2][16];
    auto load_cols = [&](int blk, int t) __attribute__((always_inline)) {
        const unsigned r0 = (unsigned)(blk * BT + 4 * hf);
        const int c0 = (t < K::TE ? t : t - K::TE) * 32;
        if (t < K::TE || c0 < C) {
            const unsigned off = r0 * (C * 4u) + 4u * (l32 & (C < 32 ? C - 1 : 31)) + 4u * c0;
#pragma unroll
            for (int r = 0; r < 16; r++) cc[t & 1][r] = buf_f32(t < K::TE ? eoth : oth.x, off + (8 * (r / 4) + r % 4) * (C * 4u));
        }
        if (RP > 0 && t >= K::TE && c0 + 32 > C) {
            const int pc = min(max(c0 + l32 - C, 0), R - 1);
            unsigned off = (r0 * (unsigned)R + (unsigned)pc) * 4u;
#pragma unroll
            for (int r = 0; r < 16; r++) {
                const float x = buf_f32(oth.phi, off);
                cc[t & 1][r] = c0 < C && l32 < C ? cc[t & 1][r] : x;      // (head dimension 16: a tile of both)
                off += (r & 3) == 3 ? 20u * (unsigned)R : 4u * (unsigned)R;
            }
        }
    };
    float lq[KEYSIDE ? 16 : 1], dqv[KEYSIDE ? 16 : 1];      // key side: lse and D of the streamed queries
    auto load_vec = [&](int blk) __attribute__((always_inline)) {
        if (!KEYSIDE) return;
        const unsigned off = (unsigned)(blk * BT + 4 * hf) * 4u;
#pragma unroll
        for (int r = 0; r < 16; r++) {
            lq[r % (KEYSIDE ? 16 : 1)] = buf_f32(lbuf, off + (8 * (r / 4) + r % 4) * 4u);
            dqv[r % (KEYSIDE ? 16 : 1)] = buf_f32(dbuf, off + (8 * (r / 4) + r % 4) * 4u);
        }
    };
    float bv[DENSE ? 16 : 1];
    const bool vec_m = DENSE && (M & 3) == 0;
    auto load_bias = [&](int blk) __attribute__((always_inline)) {
        if (!DENSE) return;
        if (KEYSIDE) {
#pragma unroll
            for (int r = 0; r < 16; r++)
                bv[r % (DENSE ? 16 : 1)] = bg[(size_t)min(blk * BT + acc_row(r, hf), N - 1) * M + rowc];
        } else {
            const float* brow = bg + (size_t)rowc * M;
#pragma unroll
            for (int g = 0; g < 4; g++) {
                const int j = blk * BT + 8 * g + 4 * hf;
                if (vec_m) {
                    const f32x4 t = *(const f32x4*)(brow + min(j, M - 4));
#pragma unroll
                    for (int x = 0; x < 4; x++) bv[(4 * g + x) % (DENSE ? 16 : 1)] = t[x];
                } else {
#pragma unroll
                    for (int x = 0; x < 4; x++) bv[(4 * g + x) % (DENSE ? 16 : 1)] = brow[min(j + x, M - 1)];
                }
            }
        }
    };

    if (b0 + part < b1) {
        const int blk = b0 + part;
#pragma unroll
        for (int n = 0; n < K::NPF; n++) rc[n] = load_row(blk, n);
        load_vec(blk);
        load_bias(blk);
        load_cols(blk, 0);
    }
    for (int blk = b0 + part; blk < b1; blk += KW) {
        const int nxt = min(blk + KW, b1 - 1);
        if (NT > 1) load_cols(blk, 1);
        __builtin_amdgcn_sched_barrier(0);      // requests stay ahead of the chains they land under
        f32x16 s, dp;
#pragma unroll
        for (int r = 0; r < 16; r++) {
            s[r] = 0.f;
            dp[r] = 0.f;
        }
#pragma unroll
        for (int n = 0; n < K::NALL; n++) {
            f32x4 a = rc[n % K::NPF];
            if (QSCALE && 8 * n < C) a *= p.scale;
            if (n + K::NPF < K::NALL) rc[n % K::NPF] = load_row(blk, n + K::NPF);
#pragma unroll
            for (int e = 0; e < 4; e++) {
                if (n < K::NCH) s = mfma32f(a[e], ar[n][e], s);
                else dp = mfma32f(a[e], er[n - K::NCH][e], dp);
            }
        }
        if (DENSE) {      // behind the products, as the forward adds it
#pragma unroll
            for (int r = 0; r < 16; r++) s[r] += bv[r % (DENSE ? 16 : 1)];
        }
#pragma unroll
        for (int n = 0; n < K::NPF; n++) rc[n] = load_row(nxt, n);
        load_bias(nxt);
        __builtin_amdgcn_sched_barrier(0);
        // P in s, dS in dp
#pragma unroll
        for (int r = 0; r < 16; r++) {
            s[r] = fast_exp2((s[r] - (KEYSIDE ? lq[r % (KEYSIDE ? 16 : 1)] : lse_r)) * kLog2e);
            dp[r] = s[r] * (dp[r] - (KEYSIDE ? dqv[r % (KEYSIDE ? 16 : 1)] : d_r));
        }
        if (blk * BT + BT > NO || (p.causal && blk == tile)) {
#pragma unroll
            for (int r = 0; r < 16; r++) {
                const int o = blk * BT + acc_row(r, hf);
                if (o >= NO || (p.causal && (KEYSIDE ? o < row : o > row))) { s[r] = 0.f; dp[r] = 0.f; }
            }
        }
        load_vec(nxt);
        if (STORE) {
            const size_t pitch = (size_t)nall * BT, rows = (size_t)((NL + 31) & ~31);
            float* drow = dS + ((size_t)bhl * rows + row) * pitch + blk * BT + 4 * hf;
#pragma unroll
            for (int g = 0; g < 4; g++) *(f32x4*)(drow + 8 * g) = f32x4{dp[4 * g], dp[4 * g + 1], dp[4 * g + 2], dp[4 * g + 3]};
        }
        if (DENSE && !KEYSIDE && row < NL) {
            float* drow = dbg + (size_t)row * M;
#pragma unroll
            for (int g = 0; g < 4; g++) {
                const int j = blk * BT + 8 * g + 4 * hf;
                if (vec_m) {
                    if (j < M) *(f32x4*)(drow + j) = f32x4{dp[4 * g], dp[4 * g + 1], dp[4 * g + 2], dp[4 * g + 3]};
                } else {
#pragma unroll
                    for (int x = 0; x < 4; x++)
                        if (j + x < M) drow[j + x] = dp[4 * g + x];
                }
            }
        }
#pragma unroll
        for (int t = 0; t < NT; t++) {
#pragma unroll
            for (int r = 0; r < 16; r++) {
                if (t < K::TE) acce[t < K::TE ? t : 0] = mfma32f(cc[t & 1][r], s[r], acce[t < K::TE ? t : 0]);
                else acca[t < K::TE ? 0 : t - K::TE] = mfma32f(cc[t & 1][r], dp[r], acca[t < K::TE ? 0 : t - K::TE]);
            }
            if (t + 2 < NT) load_cols(blk, t + 2);
            __builtin_amdgcn_sched_barrier(0);
        }
        load_cols(nxt, 0);
    }
    if (DENSE && !KEYSIDE && p.causal && row < NL) {
        // keys past the tile's diagonal block were never visited: their dBias entries are zero
        float* drow = dbg + (size_t)row * M;
        for (int blk = b1 + part; blk < nall; blk += KW)
            for (int x = hf; x < BT; x += 2)
                if (blk * BT + x < M) drow[blk * BT + x] = 0.f;
    }

    // ---- epilogue: tile by tile through LDS, where the KW partial sums meet; rows leave 16 bytes a thread ----
    float* dxg = (float*)(KEYSIDE ? p.dk : p.dq) + (KEYSIDE ? kbase : qbase);
    float* dvg = KEYSIDE ? (float*)p.dv + kbase : nullptr;
    float* dphig = (float*)(KEYSIDE ? p.dphi_k : p.dphi_q);      // [B,H,N or M,R], per batch element; may be NULL
    if (dphig) dphig += (size_t)bh * NL * R;
#pragma unroll
    for (int t = 0; t < NT; t++) {
        __syncthreads();
#pragma unroll
        for (int g = 0; g < 4; g++) {
            f32x4 w;
#pragma unroll
            for (int x = 0; x < 4; x++) w[x] = t < K::TE ? acce[t < K::TE ? t : 0][4 * g + x] : acca[t < K::TE ? 0 : t - K::TE][4 * g + x];
            *(f32x4*)(&otile[wave][l32 * OPITCH + 8 * g + 4 * hf]) = w;
        }
        __syncthreads();
        for (int e = part * 64 + lane; e < 32 * 8; e += KW * 64) {
            const int rr = e >> 3, c4 = (e & 7) * 4;
            if (row0 + rr >= NL) break;
            f32x4 w = {0.f, 0.f, 0.f, 0.f};
            for (int x = 0; x < KW; x++) w += *(const f32x4*)(&otile[wave - part + x][rr * OPITCH + c4]);
            const int c = (t < K::TE ? t : t - K::TE) * 32 + c4;
            const size_t orow = (size_t)(row0 + rr);
            if (t < K::TE) {
                if (c < C) *(f32x4*)(dvg + orow * C + c) = w;
            } else if (c < C) {
                w *= p.scale;
                *(f32x4*)(dxg + orow * C + c) = w;
            } else if (dphig) {
#pragma unroll
                for (int x = 0; x < 4; x++)
                    if (c + x - C < R) dphig[orow * R + (c + x - C)] = w[x];
            }
        }
    }
}

// D_i = sum_c dout_ic out_ic of `rows` rows: two threads a row, each summing as a lane of the query side does where that
// runs first, so the two forms agree to the bit.  Bound by its reads.
template <int C>
__global__ __launch_bounds__(256) void bwd_f32_d_kernel(const float* __restrict__ out, const float* __restrict__ dout, float* __restrict__ D, long long rows) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x, row = i >> 1;
    const int hf = (int)(i & 1);
    if (row >= rows) return;                 // both threads of a row leave together
    const size_t off = (size_t)row * C + 4 * hf;
    float s = 0.f;
#pragma unroll
    for (int n = 0; n < C / 8; n++) {
        const f32x4 a = *(const f32x4*)(dout + off + 8 * n), b = *(const f32x4*)(out + off + 8 * n);
#pragma unroll
        for (int e = 0; e < 4; e++) s = fmaf(a[e], b[e], s);
    }
    s += __shfl_xor(s, 1);
    if (hf == 0) D[row] = s;
}

// d[q | phi_q] = dS [k | phi_k] from the dS that the key side stored: lanes are queries, both operands of a k-step are 4
// bytes a lane and 128 in a row, one block ahead.  Bound by the matrix pipe (48 instructions of 64 cycles a 32 x 32
// block at C 64, R 8) with the read of dS, 4 KB a block, behind it.
template <int C, int RP>
__global__ __launch_bounds__(kThreads, 2) void bwd_f32_dq_kernel(BwdParams p, const float* __restrict__ dS, int head0, int kw_log2) {
    using K = Cfg<C, RP, false>;
    __shared__ __align__(16) float otile[kThreads / 64][32 * OPITCH];
    const int L = (blockIdx.x & 7) * p.tiles_per_xcd + (blockIdx.x >> 3);
    if (L >= p.total_tiles) return;
    const int bhl = L / p.n_tiles;
    const int u0 = L - bhl * p.n_tiles, bh = head0 + bhl;
    const int u = p.causal ? p.n_tiles - 1 - u0 : u0;      // causal: long tiles first
    const int b = bh / p.H, h = bh - b * p.H;
    const int N = p.N, M = p.M, R = p.R;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int l32 = lane & 31, hf = lane >> 5;
    const int KW = 1 << kw_log2;
    const int part = wave & (KW - 1);
    const int tile = u * ((kThreads / 64) >> kw_log2) + (wave >> kw_log2);
    const int row0 = tile * 32;
    const int nkb = (M + BT - 1) / BT, pitch = (N + 31) & ~31;

    const f32_buf kb = make_buf((const float*)p.k + (size_t)bh * M * C, (size_t)M * C * 4);
    const f32_buf pb = RP > 0 ? make_buf((const float*)p.phi_k + (size_t)b * p.phik_bstride + (size_t)h * M * R, (size_t)M * R * 4) : kb;
    const f32_buf sb = make_buf(dS + (size_t)bhl * nkb * BT * pitch, (size_t)nkb * BT * pitch * 4);

    f32x16 acc[K::TA];
#pragma unroll
    for (int t = 0; t < K::TA; t++)
#pragma unroll
        for (int r = 0; r < 16; r++) acc[t][r] = 0.f;
    int b1 = p.causal ? min(nkb, tile + 1) : nkb;
    if (row0 >= N) b1 = 0;

    auto load_ds = [&](int blk, float (&x)[16]) __attribute__((always_inline)) {
        const unsigned off = ((unsigned)(blk * BT + 4 * hf) * (unsigned)pitch + (unsigned)(row0 + l32)) * 4u;
#pragma unroll
        for (int r = 0; r < 16; r++) x[r] = buf_f32(sb, off + (8 * (r / 4) + r % 4) * ((unsigned)pitch * 4u));
    };
    // column tile t of block blk of [k | phi_k]; rows past M read zero, columns past C + R some real element
    auto load_cols = [&](int blk, int t, float (&x)[16]) __attribute__((always_inline)) {
        const unsigned r0 = (unsigned)(blk * BT + 4 * hf);
        const int c0 = t * 32;
        if (c0 < C) {
            const unsigned off = r0 * (C * 4u) + 4u * (c0 + l32);
#pragma unroll
            for (int r = 0; r < 16; r++) x[r] = buf_f32(kb, off + (8 * (r / 4) + r % 4) * (C * 4u));
        } else {
            unsigned off = (r0 * (unsigned)R + (unsigned)min(c0 + l32 - C, R - 1)) * 4u;
#pragma unroll
            for (int r = 0; r < 16; r++) {
                x[r] = buf_f32(pb, off);
                off += (r & 3) == 3 ? 20u * (unsigned)R : 4u * (unsigned)R;
            }
        }
    };
    float ds[2][16], cc[2][16];
    if (part < b1) {
        load_ds(part, ds[0]);
        load_cols(part, 0, cc[0]);
    }
    // two blocks at a time: the register sets change roles without copies
    auto block = [&](int blk, float (&cur)[16], float (&nxt)[16], int c0) __attribute__((always_inline)) {
        const int next = min(blk + KW, b1 - 1);
        load_ds(next, nxt);
#pragma unroll
        for (int t = 0; t < K::TA; t++) {
            load_cols(t + 1 < K::TA ? blk : next, t + 1 < K::TA ? t + 1 : 0, cc[(c0 + t + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < 16; r++) acc[t] = mfma32f(cc[(c0 + t) & 1][r], cur[r], acc[t]);
        }
    };
    int blk = part;
    for (; blk + KW < b1; blk += 2 * KW) {
        block(blk, ds[0], ds[1], 0);
        block(blk + KW, ds[1], ds[0], K::TA & 1);
    }
    if (blk < b1) block(blk, ds[0], ds[1], 0);

    // ---- epilogue: tile by tile through LDS, where the KW partial sums meet ----
    float* dxg = (float*)p.dq + (size_t)bh * N * C;
    float* dphig = (float*)p.dphi_q;
    if (dphig) dphig += (size_t)bh * N * R;
#pragma unroll
    for (int t = 0; t < K::TA; t++) {
        __syncthreads();
#pragma unroll
        for (int g = 0; g < 4; g++)
            *(f32x4*)(&otile[wave][l32 * OPITCH + 8 * g + 4 * hf]) = f32x4{acc[t][4 * g], acc[t][4 * g + 1], acc[t][4 * g + 2], acc[t][4 * g + 3]};
        __syncthreads();
        for (int e = part * 64 + lane; e < 32 * 8; e += KW * 64) {
            const int rr = e >> 3, c = t * 32 + (e & 7) * 4;
            if (row0 + rr >= N) break;
            f32x4 w = {0.f, 0.f, 0.f, 0.f};
            for (int x = 0; x < KW; x++) w += *(const f32x4*)(&otile[wave - part + x][rr * OPITCH + (e & 7) * 4]);
            const size_t orow = (size_t)(row0 + rr);
            if (c < C) {
                w *= p.scale;
                *(f32x4*)(dxg + orow * C + c) = w;
            } else if (dphig) {
#pragma unroll
                for (int x = 0; x < 4; x++)
                    if (c + x - C < R) dphig[orow * R + (c + x - C)] = w[x];
            }
        }
    }
}

// Heads a launch of this call is laid out for: those that the room a size query asks for takes at a time.  The split of a
// tile over waves, which orders the sums, follows from them and not from the heads that the given workspace leaves to one
// launch, so the gradients do not depend on the workspace.
template <int C, bool DENSE>
long long planned_heads(const BwdParams& p) {
    const long long heads = (long long)p.B * p.H;
    const int chunk = C < 32 || DENSE ? 0 : stored_heads(heads, p.N, p.M, C, p.causal != 0, kMaxStored);
    return chunk > 0 ? chunk : heads;
}

// Tiles of one launch over `heads` heads, `rows` rows a head: p's counters, the split of a tile over waves.
int set_tiles(BwdParams& p, int heads, long long planned, int rows, int other) {
    const int tiles = (rows + 31) / 32;
    const int kw = f32_split(planned * tiles, (other + BT - 1) / BT, 4);
    int kw_log2 = 0;
    while ((1 << kw_log2) < kw) kw_log2++;
    const int qw = (kThreads / 64) / kw;
    p.n_tiles = (tiles + qw - 1) / qw;
    p.total_tiles = heads * p.n_tiles;
    p.tiles_per_xcd = (p.total_tiles + 7) / 8;
    return kw_log2;
}

template <int C, int RP, bool KEYSIDE, bool DENSE, bool QSCALE = false>
int launch_side(const BwdParams& pin, hipStream_t stream) {
    BwdParams p = pin;
    const int kw_log2 = set_tiles(p, p.B * p.H, planned_heads<C, DENSE>(p), KEYSIDE ? p.M : p.N, KEYSIDE ? p.N : p.M);
    hipLaunchKernelGGL((bwd_f32_kernel<C, RP, KEYSIDE, DENSE, false, QSCALE>), dim3(8 * p.tiles_per_xcd), dim3(kThreads), 0, stream, p,
                       (float*)p.workspace, kw_log2, (float*)nullptr, 0);
    return hipGetLastError() == hipSuccess ? 0 : 1;
}

// Key side first, leaving dS for the query side, `chunk` heads at a time.
template <int C, int RP, bool QSCALE>
int launch_stored(const BwdParams& pin, float* dS, int chunk, hipStream_t stream) {
    const long long rows = (long long)pin.B * pin.H * pin.N, planned = planned_heads<C, false>(pin);
    hipLaunchKernelGGL((bwd_f32_d_kernel<C>), dim3((unsigned)((rows * 2 + 255) / 256)), dim3(256), 0, stream, (const float*)pin.out,
                       (const float*)pin.dout, (float*)pin.workspace, rows);
    if (hipGetLastError() != hipSuccess) return 1;
    const int heads = pin.B * pin.H;
    for (int h0 = 0; h0 < heads; h0 += chunk) {
        const int n = heads - h0 < chunk ? heads - h0 : chunk;
        BwdParams p = pin;
        int kw_log2 = set_tiles(p, n, planned, p.M, p.N);
        hipLaunchKernelGGL((bwd_f32_kernel<C, RP, true, false, true, QSCALE>), dim3(8 * p.tiles_per_xcd), dim3(kThreads), 0, stream, p,
                           (float*)p.workspace, kw_log2, dS, h0);
        kw_log2 = set_tiles(p, n, planned, p.N, p.M);
        hipLaunchKernelGGL((bwd_f32_dq_kernel<C, RP>), dim3(8 * p.tiles_per_xcd), dim3(kThreads), 0, stream, p, (const float*)dS, h0, kw_log2);
        if (hipGetLastError() != hipSuccess) return 1;
    }
    return 0;
}

template <int C, int RP, bool DENSE = false>
int launch(const BwdParams& p, hipStream_t stream) {
    if constexpr (C >= 32 && !DENSE) {
        int exponent = 0;
        const bool pow2 = std::frexp(p.scale, &exponent) == 0.5f;
        const size_t off = d_bytes((long long)p.B * p.H * p.N);
        const int chunk = stored_heads((long long)p.B * p.H, p.N, p.M, C, p.causal != 0, p.workspace_bytes > off ? p.workspace_bytes - off : 0);
        float* const dS = (float*)((unsigned char*)p.workspace + off);
        if (chunk > 0) return pow2 ? launch_stored<C, RP, false>(p, dS, chunk, stream) : launch_stored<C, RP, true>(p, dS, chunk, stream);
        if (!pow2) {
            const int rc = launch_side<C, RP, false, DENSE>(p, stream);
            return rc != 0 ? rc : launch_side<C, RP, true, DENSE, true>(p, stream);
        }
    }
    const int rc = launch_side<C, RP, false, DENSE>(p, stream);      // also leaves D for the key side
    return rc != 0 ? rc : launch_side<C, RP, true, DENSE>(p, stream);
}

template <int C>
int dispatch_c(const BwdParams& p, hipStream_t stream) {
    if (p.R == 0) return launch<C, 0>(p, stream);
    if (p.R <= 8) return launch<C, 8>(p, stream);
    if (p.R <= 16) return launch<C, 16>(p, stream);
    if (p.R <= 32) return launch<C, 32>(p, stream);
    return launch<C, 64>(p, stream);
}

}  // namespace

// Workspace with which the query side takes dS from the key side, by the rule and in the parts of the launch; 0 where it
// recomputes dS in any case.
size_t fb_bwd_f32_workspace_bytes(long long heads, int N, int M, int C, bool causal) {
    const int chunk = C < 32 ? 0 : stored_heads(heads, N, M, C, causal, kMaxStored);
    return chunk > 0 ? d_bytes(heads * N) + (size_t)chunk * ds_head_bytes(N, M) : 0;
}

// fp32 tensors and fp32 factors (N queries, M keys; causal needs N = M); p.workspace: at least
// 4 B H N bytes (the D row sums), and room for dS as far as p.workspace_bytes says.
// Returns 0 on success, 1 on launch failure, -1 when no instantiation fits.
int fb_launch_bwd_f32(const BwdParams& p, int C, hipStream_t stream) {
    if (p.R > 64 || (p.causal && p.N != p.M)) return -1;
    switch (C) {
        case 16: return dispatch_c<16>(p, stream);
        case 32: return dispatch_c<32>(p, stream);
        case 64: return dispatch_c<64>(p, stream);
        case 128: return dispatch_c<128>(p, stream);
        default: return -1;
    }
}

// Dense-bias backward in fp32 (p.bias, p.dbias, p.bias_bstride set; p.R = 0; N = M).
int fb_launch_bwd_dense_f32(const BwdParams& p, int C, hipStream_t stream) {
    if (p.N != p.M) return -1;
    switch (C) {
        case 16: return launch<16, 0, true>(p, stream);
        case 32: return launch<32, 0, true>(p, stream);
        case 64: return launch<64, 0, true>(p, stream);
        case 128: return launch<128, 0, true>(p, stream);
        default: return -1;
    }
}
