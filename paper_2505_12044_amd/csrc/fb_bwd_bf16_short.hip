// bf16 MFMA backward for short key sequences on the 32-channel tiles (head dimensions 16 and 32), gfx950.
//
// The two kernels of fb_bwd_bf16.hip recompute S and dP twice, because a query's dQ and a key's dK, dV are sums over
// what other workgroups hold.  Where a head's keys fit one workgroup (up to twelve waves of 32 keys) they are not:
// here S, P, dP and dS are formed once, keys on the lanes as in the dkv kernel, dV and d[K | phi_k] stay in the wave's
// accumulators, and the dS tiles of all waves meet in LDS, from where d[Q | phi_q] = dS [K | phi_k] is contracted
// over all keys: 5 contractions instead of 7, half the exponentials, q, k, v, dO and out read once, no workspace.
// B 384, H 4, N 384, C 32, R 16: 208 -> 195 us; vector ALU 51 % of the cycles (16 exponentials, multiply-adds, conversions a
// 32 x 32 block against 11 + 3 matrix instructions), matrix pipe 23 %, LDS 15 %; between them two barriers a pair of query
// blocks, with nothing else on the CU.
//
// One workgroup walks heads; queries come in pairs of 32-row blocks.  Pair p:
//     request the rows of pair p + 1 (registers) | block a: S, dP | P, dS | dV, dK chains |
//     barrier | dS of a -> LDS | block b the same | rows of pair p + 1 -> LDS | barrier | dQ of both blocks
// The dQ work of a pair is 2 x 2 x KS tiles of 16 queries x 16 columns, dealt to the waves.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "fb_device.h"
#include "fb_launch.h"
#include "fb_params.h"

namespace {

constexpr int kMaxWaves = 12;            // three waves per SIMD: 168 registers
constexpr int kMinWaves = 6;             // the rows of a query block are staged by up to six waves
constexpr size_t kLdsBytes = 160 * 1024;

FB_DEV int swz64(int r) { return (((r >> 1) & 1) << 2) | ((r >> 2) & 3); }
FB_DEV int swz32(int r) { return (r >> 2) & 3; }

// LDS tiles of 32 rows: WT = 32 or 64 columns unpadded, 16-byte pieces swizzled so that row and transpose reads are
// conflict-free (as in fb_bwd_bf16.hip).
template <int CG, int RP>
struct Cfg {
    static constexpr int KC = CG / 16, KS = (CG + RP) / 16;
    static constexpr int WT = CG + RP <= 32 ? 32 : 64;
    static constexpr int T1 = 32 * WT * 2, T2 = 32 * 32 * 2, kVec = 256;
    static constexpr int kSlot = T1 + T2 + kVec;
    static constexpr int kTile = 32 * 32 * 2;          // a wave's dS tile
    static constexpr int MB = (CG + RP + 31) / 32;     // 32-column blocks of d[K | phi_k]
    static constexpr int NU = 2 * KC + RP / 16;        // staging roles of a query block: q, (dO, out), phi_q in 64-piece units
    static size_t lds(int nkb) { return (size_t)nkb * T1 + (size_t)2 * nkb * kTile + 4 * kSlot; }
    static_assert(CG + RP <= 64 && NU <= kMinWaves, "shape");
};
template <int WT>
FB_DEV int tile_off(int row, int chunk) {
    return WT == 64 ? row * 128 + ((chunk ^ swz64(row)) << 4) : row * 64 + ((chunk ^ swz32(row)) << 4);
}

FB_DEV f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }

// Sixteen bytes of a factor row at byte offset `row`: columns [8 c8, 8 c8 + 8), zero from R on.  R4: R is a multiple of
// four and not of eight (rows start on 8 bytes).
template <bool R4>
FB_DEV u32x4 phi_piece(const unsigned char* base, unsigned row, int c8, int R) {
    u32x4 x = {0u, 0u, 0u, 0u};
    if (!R4) {
        if (c8 * 8 < R) x = *(const u32x4*)(base + (row + c8 * 16));
    } else {
        if (c8 * 8 < R) { const u32x2 t = *(const u32x2*)(base + (row + c8 * 16)); x.x = t.x; x.y = t.y; }
        if (c8 * 8 + 4 < R) { const u32x2 t = *(const u32x2*)(base + (row + c8 * 16 + 8)); x.z = t.x; x.w = t.y; }
    }
    return x;
}

// Opaque copy: what is computed from it is computed where it is used and not kept in registers over the whole kernel
// (a spilled address costs more than its few instructions: a scratch reload waits for every load in flight).
FB_DEV int here(int x) {
    asm volatile("" : "+v"(x));
    return x;
}

// four consecutive gradient values at columns col.. of a row [channels | R factor columns]; the bases are wave-uniform
FB_DEV void store4(bf16x4 v, int col, int CG, int R, unsigned row, bf16_t* chan, bf16_t* phi) {
    if (col < CG) *(u32x2*)(chan + (row * (unsigned)CG + col)) = __builtin_bit_cast(u32x2, v);
    else if (phi != nullptr && col - CG < R) *(u32x2*)(phi + (row * (unsigned)R + (col - CG))) = __builtin_bit_cast(u32x2, v);
}

template <int CG, int RP, bool R4, bool CAUSAL>
__global__ __launch_bounds__(kMaxWaves * 64) void bwd_short_kernel(BwdParams p, int heads) {
    using K = Cfg<CG, RP>;
    extern __shared__ __align__(16) unsigned char smem[];
    const int N = p.N, M = p.M, R = p.R;
    const int nw = blockDim.x >> 6;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hf = lane >> 5;
    const int nkb = (M + 31) >> 5, nqb = (N + 31) >> 5, npair = (nqb + 1) >> 1;
    const bool keys = wave < nkb;                     // waves beyond the key tiles stage rows and contract dQ
    const int dsbase = nkb * K::T1, ring = dsbase + 2 * nkb * K::kTile;      // K tiles, dS tiles, ring of query blocks
    const int ri = wave * 32 + l32;                   // this lane's key
    const float emul = kLog2e, qscale = p.scale;

    // ---- lane-side operands: [k | phi_k] and v rows of this lane's key (byte offsets inside a head are 32-bit) ----
    bf16x8 l1reg[K::KS], l2reg[K::KC];
    auto load_keys = [&](int head) __attribute__((always_inline)) {
        const int b = head / p.H, h = head - b * p.H;
        const unsigned char* kg = (const unsigned char*)p.k + (size_t)head * M * (CG * 2);
        const unsigned char* vg = (const unsigned char*)p.v + (size_t)head * M * (CG * 2);
        const int ln = here(lane), key = min(wave * 32 + (ln & 31), M - 1), half = ln >> 5;
        const unsigned off = (unsigned)key * (CG * 2) + 16 * half;
#pragma unroll
        for (int ks = 0; ks < K::KC; ks++) {
            l1reg[ks] = as_bf16x8(*(const u32x4*)(kg + (off + ks * 32)));
            l2reg[ks] = as_bf16x8(*(const u32x4*)(vg + (off + ks * 32)));
        }
        if (RP > 0) {
            const unsigned char* pg = (const unsigned char*)p.phi_k + ((size_t)b * p.phik_bstride + (size_t)h * M * R) * 2;
#pragma unroll
            for (int ks = K::KC; ks < K::KS; ks++) l1reg[ks] = as_bf16x8(phi_piece<R4>(pg, (unsigned)(key * R) * 2, (ks - K::KC) * 2 + half, R));
        }
    };

    // ---- staging of a query block's rows: the first KC waves take q, the next KC dO with out and lse, the next phi_q ----
    u32x4 r0 = {0u, 0u, 0u, 0u}, r1 = r0;       // one block's rows on their way
    float rl = 0.f;
    const bool q_role = wave < K::KC, o_role = wave >= K::KC && wave < 2 * K::KC, p_role = wave >= 2 * K::KC && wave < K::NU;
    const int unit = wave - (q_role ? 0 : o_role ? K::KC : 2 * K::KC);
    auto load_rows = [&](int head, int qblk) __attribute__((always_inline)) {
        if (wave >= K::NU) return;
        const int piece = unit * 64 + here(lane);
        if (q_role || o_role) {
            const unsigned qi = (unsigned)min(qblk * 32 + piece / (CG / 8), N - 1);
            const unsigned off = qi * (CG * 2) + piece % (CG / 8) * 16;
            const size_t hoff = (size_t)head * N * (CG * 2);
            const unsigned char* g0 = (const unsigned char*)(q_role ? p.q : p.dout) + hoff;
            r0 = *(const u32x4*)(g0 + off);
            if (o_role) {
                const unsigned char* g1 = (const unsigned char*)p.out + hoff;
                r1 = *(const u32x4*)(g1 + off);
                const float* lg = p.lse + (size_t)head * N;
                rl = lg[qi];
            }
        } else if (RP > 0) {
            const int b = head / p.H, h = head - b * p.H;
            const unsigned qi = (unsigned)min(qblk * 32 + piece / (RP / 8), N - 1);
            const unsigned char* pg = (const unsigned char*)p.phi_q + ((size_t)b * p.phi_bstride + (size_t)h * N * R) * 2;
            r0 = phi_piece<R4>(pg, qi * (unsigned)R * 2, piece % (RP / 8), R);
        }
    };
    auto store_rows = [&](int slot) __attribute__((always_inline)) {
        if (wave >= K::NU) return;
        unsigned char* t = smem + (ring + slot * K::kSlot);
        const int piece = unit * 64 + here(lane);
        if (q_role) {
            bf16x8 a = as_bf16x8(r0);
#pragma unroll
            for (int e = 0; e < 8; e++) a[e] = (bf16_t)((float)a[e] * qscale);     // as the forward rounds it
            *(u32x4*)(t + tile_off<K::WT>(piece / (CG / 8), piece % (CG / 8))) = as_uint4(a);
        } else if (o_role) {
            const int row = piece / (CG / 8), chunk = piece % (CG / 8);
            *(u32x4*)(t + K::T1 + tile_off<32>(row, chunk)) = r0;
            // D in the order of the two-kernel form: one chain over the even pieces of a row, one over the odd ones, added
            const bf16x8 d8 = as_bf16x8(r0), o8 = as_bf16x8(r1);
            float dsum = 0.f;
#pragma unroll
            for (int c = 0; c < CG / 16; c++) {
                if (c > 0) dsum = __shfl_xor(dsum, 2);
#pragma unroll
                for (int e = 0; e < 8; e++) dsum = fmaf((float)o8[e], (float)d8[e], dsum);
            }
            dsum += __shfl_xor(dsum, 1);
            if (chunk == CG / 8 - 2) {
                float* v = (float*)(t + K::T1 + K::T2);
                v[row] = -(rl * kLog2e);
                v[32 + row] = -dsum;
            }
        } else if (RP > 0) {
            *(u32x4*)(t + tile_off<K::WT>(piece / (RP > 0 ? RP / 8 : 1), CG / 8 + piece % (RP > 0 ? RP / 8 : 1))) = r0;
        }
    };

    // ---- per-lane LDS offsets.  The swizzle makes every other operand of a tile this offset with address bits 4..6
    // flipped (tiles start on multiples of 128 bytes) and a constant added, so one register serves each kind of read.
    const int i16 = lane & 15, blk16 = l32 >> 4;
    const int row1 = tile_off<K::WT>(l32, hf), row2 = tile_off<32>(l32, hf);                   // row reads: k-step ks is ^ 32 ks
    const int trow = 4 * hf + (i16 >> 2), tchunk = 2 * blk16 + ((i16 & 3) >> 1), tsub = (i16 & 1) * 8;
    const int tr1 = tile_off<K::WT>(trow, tchunk) + tsub, tr2 = tile_off<32>(trow, tchunk) + tsub;   // transpose reads
    auto tr_pair = [&](int lo, int hi) __attribute__((always_inline)) {
        return join_tr(lds_read_tr16((const bf16_t*)(smem + lo)), lds_read_tr16((const bf16_t*)(smem + hi)));
    };
    auto row_op = [&](int addr) __attribute__((always_inline)) { return as_bf16x8(*(const u32x4*)(smem + addr)); };

    f32x16 acc1[K::MB], acc2;                        // d[K | phi_k]^T, dV^T
    auto clear_acc = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 16; r++) {
#pragma unroll
            for (int mb = 0; mb < K::MB; mb++) acc1[mb][r] = 0.f;
            acc2[r] = 0.f;
        }
    };
    clear_acc();

    // ---- first pair into slots 0, 1; first rows of the second requested ----
    int bh = blockIdx.x, pair = 0;
    if (bh >= heads) return;
    load_keys(bh);
#pragma unroll 1
    for (int j = 0; j < 2; j++) {
        load_rows(bh, j);
        store_rows(j);
    }
    int nhead = npair > 1 ? bh : bh + (int)gridDim.x, npr = npair > 1 ? 1 : 0;        // the pair behind this one
    if (nhead < heads) load_rows(nhead, 2 * npr);
    __syncthreads();

    // d[Q | phi_q] of pair dpair of head dbh: tile (block, query half, column group) = sum over the key tiles
    int dbh = -1, dpair = 0;
    auto contract_dq = [&]() __attribute__((always_inline)) {
        for (int t = wave; t < 4 * K::KS; t += nw) {
            const int j = t / (2 * K::KS), rem = t - j * (2 * K::KS), qh = rem & 1, cg = rem >> 1;
            const int qblk = 2 * dpair + j;
            if (qblk >= nqb) break;
            const int nt = CAUSAL ? min(nkb, qblk + 1) : nkb;
            // lane group g16 takes keys 8 g16 + 0..7 of a tile
            const int ln = here(lane), g16 = ln >> 4, c16 = ln & 15, krow = 8 * g16 + (c16 >> 2), kchunk = (c16 & 3) >> 1;
            const int kt16 = tile_off<K::WT>(krow, kchunk) + (c16 & 1) * 8, ds16 = tile_off<32>(krow, kchunk) + (c16 & 1) * 8;
            const int ka = kt16 ^ (32 * cg), da = (dsbase + j * nkb * K::kTile + ds16) ^ (32 * qh);
            f32x4 c0 = {0.f, 0.f, 0.f, 0.f}, c1 = c0;
            // two key tiles at a time, the operands of the next two in flight; an odd last tile is met twice, the second
            // time unused
            struct Ops { bf16x8 k[2], d[2]; };
            auto read2 = [&](int w, Ops& x) __attribute__((always_inline)) {
#pragma unroll
                for (int u = 0; u < 2; u++) {
                    const int wu = min(w + u, nt - 1);
                    const int a = ka + wu * K::T1, d = da + wu * K::kTile;
                    x.k[u] = tr_pair(a, (a ^ 16) + 4 * K::WT * 2);
                    x.d[u] = tr_pair(d, (d ^ 16) + 256);
                }
            };
            auto mul2 = [&](int w, const Ops& x) __attribute__((always_inline)) {
                c0 = mfma16(x.k[0], x.d[0], c0);
                if (w + 1 < nt) c1 = mfma16(x.k[1], x.d[1], c1);
            };
            Ops x, y;
            read2(0, x);
            for (int w = 0; w < nt; w += 4) {
                read2(w + 2, y);
                mul2(w, x);
                if (w + 2 < nt) {
                    read2(w + 4, x);
                    mul2(w + 2, y);
                }
            }
            const int qi = qblk * 32 + qh * 16 + c16;
            if (qi < N) {
                const float mul = cg < K::KC ? p.scale : 1.f;
                bf16x4 v;
#pragma unroll
                for (int x = 0; x < 4; x++) v[x] = (bf16_t)((c0[x] + c1[x]) * mul);
                store4(v, cg * 16 + 4 * g16, CG, R, (unsigned)qi, (bf16_t*)p.dq + (size_t)dbh * N * CG,
                       p.dphi_q == nullptr ? nullptr : (bf16_t*)p.dphi_q + (size_t)dbh * N * R);
            }
        }
    };

    int par = 0;
    bool first = true;       // first pair of a head: [k | phi_k] goes to LDS
    for (;;) {
        const bool last_pair = pair == npair - 1;
        const bool more = nhead < heads;                                 // workgroup-uniform
#pragma unroll
        for (int j = 0; j < 2; j++) {
            const int qblk = 2 * pair + j;
            const bool live = keys && qblk < nqb && !(CAUSAL && qblk < wave);     // wave-uniform
            bf16x8 dsb[2];
            if (j == 0 && dbh >= 0) contract_dq();
            if (live) {
                const int t1 = ring + (2 * par + j) * K::kSlot, t2 = t1 + K::T1;
                const int ra = t1 + row1, rb = t2 + row2, ta = t1 + tr1, tb = t2 + tr2;
                // S is formed as the forward forms it and P = exp2(S log2e - lse log2e), so P sums to one as far as the
                // forward's did; the dP chain starts from -D of the block's rows.  Operands are read LA matrix instructions
                // ahead: S, dP, dV, d[K | phi_k] in this order.
                constexpr int NA = K::KS + K::KC, NOPS = NA + 2 + 2 * K::MB, LA = 3;
                bf16x8 opr[LA + 1];
                auto read_op = [&](int n) __attribute__((always_inline)) {
                    if (n < K::KS) return row_op(ra ^ (32 * n));
                    if (n < NA) return row_op(rb ^ (32 * (n - K::KS)));
                    if (n < NA + 2) return tr_pair(tb + (n - NA) * 1024, (tb ^ 32) + (n - NA) * 1024 + 512);
                    const int mb = (n - NA - 2) >> 1, o = ((n - NA) & 1) * 16 * K::WT * 2;
                    return tr_pair((ta ^ (64 * mb)) + o, (ta ^ (64 * mb) ^ 32) + o + 8 * K::WT * 2);
                };
                f32x16 s, dp;
                const unsigned char* vp = smem + (t2 + K::T2 + 16 * hf);
#pragma unroll
                for (int r = 0; r < 16; r++) s[r] = 0.f;
#pragma unroll
                for (int n = 0; n < LA; n++) opr[n] = read_op(n);
#pragma unroll
                for (int g = 0; g < 4; g++) {
                    const f32x4 nd = *(const f32x4*)(vp + 32 * g + 128);
#pragma unroll
                    for (int x = 0; x < 4; x++) dp[4 * g + x] = nd[x];
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int n = 0; n < NA; n++) {
                    opr[(n + LA) % (LA + 1)] = read_op(n + LA);
                    if (n < K::KS) s = mfma32(opr[n % (LA + 1)], l1reg[n], s);
                    else dp = mfma32(opr[n % (LA + 1)], l2reg[n - K::KS], dp);
                    __builtin_amdgcn_sched_barrier(0);
                }
                bf16x8 pb[2];
                f32x4 nl;
#pragma unroll
                for (int r = 0; r < 16; r++) {
                    if (r % 4 == 0) nl = *(const f32x4*)(vp + 8 * r);
                    const float pr = fast_exp2(fmaf(s[r], emul, nl[r % 4]));
                    pb[r / 8][r % 8] = (bf16_t)pr;
                    dsb[r / 8][r % 8] = (bf16_t)(pr * dp[r]);
                }
                if (qblk * 32 + 32 > N || wave * 32 + 32 > M || (CAUSAL && qblk == wave)) {
                    // rare: zero what is not there (rows past N repeat row N - 1, keys past M key M - 1) or not seen
                    asm volatile("" ::: "memory");
#pragma unroll
                    for (int r = 0; r < 16; r++) {
                        const int qi = qblk * 32 + 8 * (r / 4) + 4 * hf + (r % 4);
                        if (qi >= N || ri >= M || (CAUSAL && qi < ri)) {
                            pb[r / 8][r % 8] = (bf16_t)0.f;
                            dsb[r / 8][r % 8] = (bf16_t)0.f;
                        }
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int n = NA; n < NOPS; n++) {
                    if (n + LA < NOPS) opr[(n + LA) % (LA + 1)] = read_op(n + LA);
                    if (n < NA + 2) acc2 = mfma32(opr[n % (LA + 1)], pb[n - NA], acc2);
                    else acc1[(n - NA - 2) >> 1] = mfma32(opr[n % (LA + 1)], dsb[(n - NA) & 1], acc1[(n - NA - 2) >> 1]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if (j == 0) {
                __syncthreads();         // everyone has left the dQ work of the pair before: its dS, K and row tiles may be written
                if (first && keys) {
#pragma unroll
                    for (int ks = 0; ks < K::KS; ks++)
                        *(u32x4*)(smem + ((wave * K::T1 + row1) ^ (32 * ks))) = as_uint4(l1reg[ks]);
                }
            }
            if (more) {                  // rows of the next pair: what was requested is stored, the other block requested
                store_rows(2 * (par ^ 1) + j);
                if (j == 0) load_rows(nhead, 2 * npr + 1);
            }
            if (live) {
                const int ln = here(lane), key = ln & 31;
                unsigned char* t = smem + (dsbase + (j * nkb + wave) * K::kTile) + key * 64 + (ln >> 5) * 8;
#pragma unroll
                for (int g = 0; g < 4; g++) {
                    const bf16x8 d = dsb[g >> 1];
                    const bf16x4 v = (g & 1) ? __builtin_shufflevector(d, d, 4, 5, 6, 7) : __builtin_shufflevector(d, d, 0, 1, 2, 3);
                    *(u32x2*)(t + ((g ^ swz32(key)) << 4)) = __builtin_bit_cast(u32x2, v);
                }
            }
        }
        if (last_pair) {
            // this head's key gradients leave, the next head's keys arrive
            if (keys) {
                if (more) load_keys(nhead);
                const int key = wave * 32 + (here(lane) & 31);
                if (key < M) {
                    bf16_t* dvg = (bf16_t*)p.dv + (size_t)bh * M * CG;
                    bf16_t* dkg = (bf16_t*)p.dk + (size_t)bh * M * CG;
                    bf16_t* dpg = p.dphi_k == nullptr ? nullptr : (bf16_t*)p.dphi_k + (size_t)bh * M * R;
                    const int half = here(lane) >> 5;
#pragma unroll
                    for (int mb = 0; mb < K::MB; mb++)
#pragma unroll
                        for (int g = 0; g < 4; g++) {
                            bf16x4 a4, b4;
#pragma unroll
                            for (int x = 0; x < 4; x++) { a4[x] = (bf16_t)acc1[mb][4 * g + x]; b4[x] = (bf16_t)acc2[4 * g + x]; }
                            if (mb * 32 + 8 * g < CG + RP) store4(a4, mb * 32 + 8 * g + 4 * half, CG, R, (unsigned)key, dkg, dpg);
                            if (mb == 0 && 8 * g < CG) *(u32x2*)(dvg + ((unsigned)key * CG + 8 * g + 4 * half)) = __builtin_bit_cast(u32x2, b4);
                        }
                }
                clear_acc();
            }
        }
        __syncthreads();                 // dS tiles, K tiles and the next rows are in place
        // the pair behind the next one: its first block is requested now
        int n2head = nhead, n2pr = npr + 1;
        if (n2pr == npair) { n2head += (int)gridDim.x; n2pr = 0; }
        if (more && n2head < heads) load_rows(n2head, 2 * n2pr);

        dbh = bh;
        dpair = pair;
        if (!more) break;
        first = last_pair;
        bh = nhead;
        pair = npr;
        nhead = n2head;
        npr = n2pr;
        par ^= 1;
    }
    contract_dq();
}

template <int CG, int RP, bool R4, bool CAUSAL>
int launch(const BwdParams& p, int cus, hipStream_t stream) {
    using K = Cfg<CG, RP>;
    auto kern = bwd_short_kernel<CG, RP, R4, CAUSAL>;
    static FbLdsOnce once;
    if (!fb_raise_lds_limit((const void*)kern, kLdsBytes, once)) return 1;
    const int nkb = (p.M + 31) / 32, nw = nkb < kMinWaves ? kMinWaves : nkb;
    const size_t lds = K::lds(nkb);
    const int heads = p.B * p.H;
    int per_cu = kMaxWaves / nw;
    if ((size_t)per_cu * lds > kLdsBytes) per_cu = (int)(kLdsBytes / lds);
    const long long most = (long long)cus * per_cu;
    hipLaunchKernelGGL(kern, dim3((unsigned)(heads < most ? heads : most)), dim3(64 * nw), lds, stream, p, heads);
    return hipGetLastError() == hipSuccess ? 0 : 1;
}
template <int CG, int RP, bool R4>
int dispatch_causal(const BwdParams& p, int cus, hipStream_t stream) {
    return p.causal ? launch<CG, RP, R4, true>(p, cus, stream) : launch<CG, RP, R4, false>(p, cus, stream);
}
template <int CG, int RP>
int dispatch_r(const BwdParams& p, int cus, hipStream_t stream) {
    return p.R % 8 == 0 ? dispatch_causal<CG, RP, false>(p, cus, stream) : dispatch_causal<CG, RP, true>(p, cus, stream);
}
template <int CG>
int dispatch_rp(const BwdParams& p, int rp, int cus, hipStream_t stream) {
    switch (rp) {
        case 0: return p.causal ? launch<CG, 0, false, true>(p, cus, stream) : -1;
        case 16: return dispatch_r<CG, 16>(p, cus, stream);
        case 32: return dispatch_r<CG, 32>(p, cus, stream);
        default: return -1;
    }
}

}  // namespace

// Kernel times against the pair of kernels of fb_bwd_bf16.hip (those / this, pre-pass included), 16 to 4096 heads of every
// length in steps of 32, 256 CUs, bf16 factors.  One workgroup takes a whole head, so longer heads have to be enough of them
// (16 a 32-key tile, 8 at 16 channels), and beyond one head a CU the last round has to be full.
//   C 32, 16 factor columns, full: up to 64 keys 1.06-1.8 (beyond twelve rounds 0.93); 65 to 128 keys 1.3-1.46 in one round, 0.78-1.02 beyond (half of the
//   six waves only stage rows); up to 192 keys 1.05-1.3 in one round, 1.0-1.18 in full rounds, 0.88-0.97 in others; 224 and
//   256 keys the same, but no more than 0.92-1.0 from the fourth and fifth round on; beyond 256 keys 1.02-1.25 in full rounds,
//   0.85-0.98 in others.  Causal: 1.0-1.7, but for 65 to 128 and 224 keys (0.86-1.0 in three rounds and from five on) and 160
//   and 192 keys in many rounds that are not full (0.95).  (Full enough: the other kernels take 128 rows to a workgroup, three a
//   CU, so up to 256 keys 1.5 heads a CU are one round of theirs and 1.6 are two: 384 heads 0.91, 400 heads 1.28.)
//   32 columns: 1.05-1.9 up to 192 keys (65 to 128 in many rounds 0.91-0.95), beyond 1.0-1.4 in rounds that are full enough;
//   causal 1.0-2.0.
//   C 16 (two 16-column groups, no dead rows): 1.07-2.4, but for 65 to 96 keys in many rounds (0.87-0.98).
//   Without factors there is no pre-pass to save and less to recompute: full 0.86-1.2, never; causal from 161 keys on 1.3-1.44
//   in one round, 1.0-1.2 in two, 0.84-1.0 beyond at C 32 up to 256 keys; C 16 and longer heads 1.0-2.
//   Fewer queries than keys 1.0-2.7, once no more than three quarters as many in any number of rounds; more queries than keys
//   stream through one workgroup: 0.3-1.2, never.
static bool rounds_pay(int C, int rp, int nkb, bool causal, const FbHeadRounds r) {
    if (r.rounds == 1) return true;
    if (nkb == 3 && (C == 16 || rp == 32)) return r.rounds <= (causal ? 10 : 6);
    if (C == 16) return true;
    if (rp == 0) return nkb <= 8 ? r.rounds == 2 && (nkb != 7 || r.fill >= 0.75) : r.rounds > 2 || r.fill >= 0.8;
    if (rp == 32) return causal || (nkb <= 6 ? nkb != 4 || r.rounds <= 10 : r.fill >= (r.rounds <= 4 ? 0.8 : 0.9));
    if (nkb <= 2) return r.rounds <= 12;
    if (causal) {
        if (nkb == 3 || nkb == 4 || nkb == 7) return r.rounds == 2 || r.rounds == 4;
        return (nkb != 5 && nkb != 6) || r.rounds < 6 || r.fill >= 0.9;
    }
    if (nkb <= 4) return false;
    const double least = r.rounds == 2 ? 0.76 : r.rounds > 3 ? 1.0 - 0.33 / (double)r.rounds : nkb <= 6 || nkb == 8 ? 0.8 : 0.9;
    return r.rounds <= (nkb == 7 ? 3 : nkb == 8 ? 4 : r.rounds) && r.fill >= least;
}

bool fb_short_bwd(const BwdParams& p, int C, int rp) {
    if (C > 32 || rp > 32 || p.grad_f32 || p.slopes != nullptr) return false;
    const int nkb = (p.M + 31) / 32, nqb = (p.N + 31) / 32;
    if (nkb > kMaxWaves || nqb > nkb) return false;
    const long long BH = (long long)p.B * p.H;
    if (BH >= (1LL << 30)) return false;
    if (rp == 0 ? !p.causal || nkb <= 5 : p.phi_f32 || p.R % 4 != 0) return false;
    const int cus = fb_cu_count();
    if (cus <= 0) return false;
    if (!p.causal && nkb > 6 && nqb > 4 && BH * 256 < (long long)(C == 16 ? 8 : 16) * nkb * cus) return false;
    return nqb * 4 <= nkb * 3 || rounds_pay(C, rp, nkb, p.causal, fb_head_rounds(BH, cus));
}

int fb_launch_bwd_bf16_short(const BwdParams& p, int C, int rp, hipStream_t stream) {
    const int cus = fb_cu_count();
    if (cus <= 0) return 1;
    return C == 16 ? dispatch_rp<16>(p, rp, cus, stream) : dispatch_rp<32>(p, rp, cus, stream);
}
