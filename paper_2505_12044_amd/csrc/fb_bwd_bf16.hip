// bf16 MFMA backward of attention with a factorised bias, gfx950.
//
// With Aq = [q*scale | phi_q], Ak = [k | phi_k] (FlashBias Eq. 3) and S = Aq Ak^T,
// P = exp(S - lse), the chain rule for L = sum(dO * O) gives
//   dV = P^T dO,  dP = dO V^T,  dS = P o (dP - D),  D_i = sum_c dO_ic O_ic,
//   dAk = dS^T Aq  -> dK = dAk[:, :C],          dphi_k = dAk[:, C:],
//   dAq = dS Ak    -> dQ = scale * dAq[:, :C],  dphi_q = dAq[:, C:].
// The factor gradients are extra columns of the contractions that give dK and dQ; no N x N
// gradient is ever written.  No atomics; results are deterministic.
//
// Kernels:
//   rows  : where dS is stored (below): -lse * log2 e, -D and the scaled q rows, ahead of the other two
//   pre   : writes the factor columns of the operands Aq = [q*scale | phi_q | 0], Ak = [k | phi_k | 0]
//           into the workspace (bf16, 32 to 128 columns; fp32 factors as three bf16 limbs, six product columns
//           per rank as in the forward), once per head where the factors are shared over the batch; the
//           channel columns are read from k, and from q or its scaled copy, in place
//   main<DKV = false> : a lane owns a query; streams 32-key blocks;   accumulates dAq^T; runs first and
//                       leaves -lse * log2 e and -D per query row, and q*scale where it is a rounding, for the other
//   main<DKV = true>  : a lane owns a key;   streams 32-query blocks; accumulates dV^T, dAk^T
// Both main kernels recompute S and dP (7 contractions instead of 5, but no atomic dQ), except at C = 128 where the
// workspace has room: there dkv runs first and leaves dS, and dq is its output contraction alone.  They
// use the transposed orientation of the forward: the lane-side operands stay in registers,
// score-shaped accumulators feed the next MFMA as its B operand without leaving registers,
// and the transposed A operands come from the LDS transpose read.
//
// Streaming.  Because the operand columns exist in memory, a streamed block is a pure
// copy, done with direct-to-LDS loads (global_load_lds_dwordx4 from inline assembly, see
// fb_fwd_bf16_dma.h for why) into a ring of four block slots; nothing passes through
// registers.  One barrier per iteration, in the middle:
//     S, dP chains of block i | exp / dS | wait, barrier | issue block i+3 |
//     output chains of block i, first operand reads of block i+1
// A direct load writes 64 consecutive 16-byte pieces, so a 32-row tile of width W is kept as
// W/64 panels [32][64] (and one [32][32] panel if W % 64), each unpadded with an XOR chunk
// swizzle that makes both the row reads and the transpose reads bank-conflict free.
#include <hip/hip_runtime.h>

#include <type_traits>

#include <cmath>
#include "fb_device.h"
#include "fb_launch.h"
#include "fb_params.h"

namespace {

constexpr int kWaves = 4;
constexpr int kThreads = kWaves * 64;
constexpr int BT = 32;       // streamed rows per block
constexpr int NSLOT = 4;       // ring slots of the kernels that use a block in one iteration

FB_DEV int swz64(int r) { return (((r >> 1) & 1) << 2) | ((r >> 2) & 3); }
FB_DEV int swz32(int r) { return (r >> 2) & 3; }

// s_waitcnt with only vmcnt constrained
template <int N>
FB_DEV void wait_vmcnt() {
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}
FB_DEV void wait_vmcnt_n(int n) {   // n is wave-uniform; larger values wait for 12 (stricter, still correct)
    switch (n) {
        case 0: wait_vmcnt<0>(); break;
        case 1: wait_vmcnt<1>(); break;
        case 2: wait_vmcnt<2>(); break;
        case 3: wait_vmcnt<3>(); break;
        case 4: wait_vmcnt<4>(); break;
        case 5: wait_vmcnt<5>(); break;
        case 6: wait_vmcnt<6>(); break;
        case 7: wait_vmcnt<7>(); break;
        case 8: wait_vmcnt<8>(); break;
        case 9: wait_vmcnt<9>(); break;
        case 10: wait_vmcnt<10>(); break;
        case 11: wait_vmcnt<11>(); break;
        default: wait_vmcnt<12>(); break;
    }
}

// lane l reads sbase + voff (bytes); its 16 bytes land at LDS byte address lds_addr + 16 * l
FB_DEV void dma16(const void* sbase, unsigned voff, unsigned lds_addr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :: "v"(voff), "s"(sbase), "s"(lds_addr) : "memory", "m0");
}
// the same for bytes that are read once: they leave the caches to the operand tiles
FB_DEV void dma16nt(const void* sbase, unsigned voff, unsigned lds_addr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt"
                 :: "v"(voff), "s"(sbase), "s"(lds_addr) : "memory", "m0");
}

// 32-row tile of W bf16 columns stored as panels (see the header comment)
template <int W>
struct Tile {
    static constexpr int NP64 = W / 64;
    static constexpr bool HAS32 = (W % 64) != 0;
    static constexpr int BYTES = W * 64;
    static constexpr int NDMA = NP64 * 4 + (HAS32 ? 2 : 0);   // direct loads per tile
    // direct load d of the tile: row and 16-byte source chunk fetched by `lane`, LDS offset of the load
    FB_DEV static void dma_map(int d, int lane, int& row, int& chunk, int& dst) {
        if (d < NP64 * 4) {
            row = (d & 3) * 8 + (lane >> 3);
            chunk = (d >> 2) * 8 + ((lane & 7) ^ swz64(row));
            dst = (d >> 2) * 4096 + (d & 3) * 1024;
        } else {
            const int e = d - NP64 * 4;
            row = e * 16 + (lane >> 2);
            chunk = NP64 * 8 + ((lane & 3) ^ swz32(row));
            dst = NP64 * 4096 + e * 1024;
        }
    }
};

// LIMB: the factors are fp32 (or generated), i.e. bf16 limb columns.  Set only where it changes something, see
// FOLD and DL.  CG: channels of the caller's rows, 16 on the 32-channel tiles of head dimension 16, else C.
template <int C, int RP, bool LIMB = false, int CG = C>
struct Cfg {
    static constexpr int RP2 = (RP + 31) / 32 * 32;    // factor columns kept in the workspace rows (0, 32 or 64)
    static constexpr int W = C + RP2;
    static constexpr int KS = (CG + RP) / 16;          // k-steps of the score contraction (channels CG.. are zero: no step)
    static constexpr int CS = CG / 16;                 // k-steps of the dP contraction
    // DL: six to ten fp32 ranks.  A rank's six product columns are kept as three and three, 32 columns apart: the
    // first three pair (a1, b3) (a2, b2) (a3, b1), so they hold every limb of either side once and are all that the
    // factor gradients need: one 32-column output block instead of two (B 1, H 8, N 32186, C 16, R 9: of 12 + 15
    // matrix instructions a block 2 + 2).
    static constexpr bool DL = LIMB && RP == 64;
    // FOLD: the forward at C = 32 carries log2 e on its query columns where the factors are fp32.  Formed the same
    // way here, the exponent of P needs no multiply-add (the score chain starts at -lse log2 e), and the scores round
    // as the forward's did (gradients against 64 bits, N 3001, R 9: 3.3e-3 -> 3.0e-3).  Not at head dimension 16,
    // whose q scale is exact at the default scale: log2 e would round it (dk 2.5e-3 -> 3.6e-3).
    static constexpr bool FOLD = LIMB && score_log2e(CG, true);
    static constexpr int MBP = DL ? 1 : RP2 / 32;      // 32-column blocks of the factor gradients
    static constexpr int MB = C / 32 + MBP;            // 32-column blocks of dAq / dAk
    static constexpr int MBC = C / 32;
    using TC = Tile<C>;                                // channel panels of a streamed operand tile; T2: the dP operand
    using TP = Tile<RP2>;                              // factor panels, behind them
    using T2 = Tile<C>;
    static constexpr int T1_BYTES = TC::BYTES + TP::BYTES, T1_NDMA = TC::NDMA + TP::NDMA;
    static constexpr int kVecBytes = 1024;             // -lse2 of 32 rows, then their -D, in the first 256 bytes
    // Form of the dkv kernel.  Up to 128 operand columns its accumulators leave room for two waves per SIMD (three
    // at C = 32), which fill each other's gaps as they do in the dq kernel; above, one wave per SIMD overlaps
    // matrix and vector work of two blocks in its own instruction stream (PIPE).  PIPE against plain, one launch:
    // B 4, H 16, N 4096, C 64, 64 extra columns 1079 -> 867 us; B 8, H 12, N 1024, C 64, R 32 105 -> 87 us and
    // with a dense bias 109 -> 82 us; B 384, H 4, N 384, C 32, R 16 140 -> 116 us; B 1, H 8, N 32186, C 16, R 9
    // fp32 equal (its vector work, not the overlap, bounds it).
    static constexpr bool PIPE = C >= 128 || C + RP > 128;
    static constexpr int NSLOT_DKV = PIPE ? 5 : NSLOT;         // ring slots (PIPE: a block is used in two iterations)
    static constexpr size_t kEpiLds = (size_t)kWaves * 32 * (MBP * 32 + 1) * sizeof(float);
};

// ------------------------------------------------------------------------------------------
// prep / vec
// ------------------------------------------------------------------------------------------
// The factor columns of the operand rows, RP2 to a row: limbs or copies of phi (or generated ALiBi factors).  The
// channel columns are the caller's q and k, read in place (or, where the scale has to be rounded into q, the scaled
// rows that the dq kernel leaves; head dimension 16: the widened copies below).  Factors shared over the batch, or
// generated from slopes, are written once per head and not once per batch element (B 384, H 4, N 384, C 32, R 16:
// whole rows per batch element 42 us, this 4 us and the scaled q rows inside the dq kernel).
// A workgroup covers kPrepRows whole rows (one thread per 16-byte piece; the few threads past the last whole row
// idle), so a thread's row and piece come from its index by a division by a constant, and the head and position of
// the row from one block-uniform division plus a wrap.
template <int RP2>
constexpr int kPrepRows = 256 / (RP2 > 0 ? RP2 / 8 : 1);

// fmul: factor of the factor columns (1, or 1/scale on the query side of a launch whose q columns
// carry no scale: q k^T scale + phi_q phi_k^T = scale (q k^T + (phi_q / scale) phi_k^T), or log2 e, see FOLD;
// applied to fp32 factors before the limb split, as the forward does, and to bf16 factors only as a power of two).
template <int RP2, bool QSIDE, bool DL>
FB_DEV void bwd_prep_block(const BwdParams& p, bf16_t* __restrict__ dst, const unsigned block, const long long rows,
                           const float fmul) {
    constexpr int CPR = RP2 / 8;
    constexpr int RPB = kPrepRows<RP2>;
    const unsigned len = (unsigned)(QSIDE ? p.N : p.M);
    const unsigned dr = threadIdx.x / CPR;
    const int pc = (int)(threadIdx.x - dr * CPR);
    const long long row0 = (long long)block * RPB;            // block-uniform
    const long long row = row0 + dr;                          // (b*H + h)*len + i; shared factors: h*len + i
    if (dr >= (unsigned)RPB || row >= rows) return;
    bf16x8 a;
    const bool f32 = p.phi_f32 != 0;
    const size_t esz = f32 ? 4 : 2;
    // rows < 2^31: the block's first row splits into head and position once, the thread's row wraps
    const unsigned bh0 = (unsigned)((unsigned long long)row0 / len);
    unsigned bb = bh0 / (unsigned)p.H;
    unsigned h = bh0 - bb * (unsigned)p.H;
    unsigned i = (unsigned)((unsigned long long)row0 - (unsigned long long)bh0 * len) + dr;
    while (i >= len) {
        i -= len;
        if (++h == (unsigned)p.H) { h = 0; ++bb; }
    }
    if (p.slopes != nullptr) {
        // ALiBi factors of Example 3.4 from the head's slope and the row's position (App. D)
        const float m = p.slopes[h];
        float pair[2];
        pair[0] = QSIDE ? -m * (float)i : 1.f;
        pair[1] = QSIDE ? m : (float)i;
        a = phi_chunk_switch<QSIDE>(pair, pc, 2, true, fmul);
    } else {
        const size_t off = ((size_t)bb * (QSIDE ? p.phi_bstride : p.phik_bstride) + ((size_t)h * len + i) * p.R) * esz;
        const unsigned char* src = (const unsigned char*)(QSIDE ? p.phi_q : p.phi_k) + off;
        if (!f32 && (p.R & 7) == 0) {
            // bf16 factors in whole 16-byte pieces: a copy (rows and the batch stride are then multiples of 16 bytes)
            u32x4 raw = u32x4{0u, 0u, 0u, 0u};
            if (pc * 8 < p.R) raw = *(const u32x4*)(src + pc * 16);
            a = as_bf16x8(raw);
        } else if (DL) {
            a = phi_chunk_dl_switch<QSIDE>((const float*)src, pc, p.R, fmul);
        } else {
            a = phi_chunk_switch<QSIDE>(src, pc, p.R, f32, fmul);
        }
        if (!f32 && fmul != 1.f) {      // a power of two: exact
#pragma unroll
            for (int e = 0; e < 8; e++) a[e] = (bf16_t)((float)a[e] * fmul);
        }
    }
    *(u32x4*)(dst + row * RP2 + pc * 8) = as_uint4(a);
}

// Both sides in one launch: the first nb_q workgroups write the query-side rows, the rest the key-side rows.
template <int RP2, bool DL>
__global__ __launch_bounds__(256) void bwd_pre_kernel(BwdParams p, bf16_t* __restrict__ aq, bf16_t* __restrict__ ak,
                                                      unsigned nb_q, long long rows_q, long long rows_k, float qmul) {
    const unsigned blk = blockIdx.x;
    if (blk < nb_q) {
        bwd_prep_block<RP2, true, DL>(p, aq, blk, rows_q, qmul);
    } else {
        bwd_prep_block<RP2, false, DL>(p, ak, blk - nb_q, rows_k, 1.f);
    }
}

// Head dimension 16: rows of 16 channels widened to 32 with zeros (the main kernels stream tiles of 32 channels).
// One thread per 16-byte piece of the destination; blockIdx.y: q (times qscale), dO, k, v.
struct Widen16 {
    bf16_t *q, *dout, *k, *v;
};
__global__ __launch_bounds__(256) void bwd_widen16_kernel(BwdParams p, Widen16 w, long long rows_q, long long rows_k,
                                                          float qscale) {
    const unsigned side = blockIdx.y;
    const bf16_t* src = (const bf16_t*)(side == 0 ? p.q : side == 1 ? p.dout : side == 2 ? p.k : p.v);
    bf16_t* dst = side == 0 ? w.q : side == 1 ? w.dout : side == 2 ? w.k : w.v;
    const long long gid = (long long)blockIdx.x * 256 + threadIdx.x;
    const long long row = gid >> 2;
    const int c = (int)(gid & 3);
    if (row >= (side < 2 ? rows_q : rows_k)) return;
    u32x4 x = u32x4{0u, 0u, 0u, 0u};
    if (c < 2) x = *(const u32x4*)(src + row * 16 + c * 8);
    if (side == 0) {
        bf16x8 a = as_bf16x8(x);
#pragma unroll
        for (int e = 0; e < 8; e++) a[e] = (bf16_t)((float)a[e] * qscale);
        x = as_uint4(a);
    }
    *(u32x4*)(dst + row * 32 + c * 8) = x;
}

// Stored dS: what the dq kernel's prologue leaves where it runs first, -lse log2 e and -D of every query row and, where
// the scale has to be rounded into q, the scaled rows.  Two threads a row, each summing as a lane of that prologue does:
// the two forms of the backward agree to the bit.  Bound by its reads.
template <int C>
__global__ __launch_bounds__(256) void bwd_rows_kernel(BwdParams p, float* __restrict__ vec, bf16_t* __restrict__ q_out, float q_mul, long long rows) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x, row = i >> 1;
    const int hf = (int)(i & 1);
    if (row >= rows) return;                 // both threads of a row leave together
    const size_t off = (size_t)row * C + 8 * hf;
    u32x4 o[C / 16], d[C / 16];
#pragma unroll
    for (int cs = 0; cs < C / 16; cs++) {
        o[cs] = *(const u32x4*)((const bf16_t*)p.out + off + cs * 16);
        d[cs] = *(const u32x4*)((const bf16_t*)p.dout + off + cs * 16);
    }
    float sum = 0.f;
#pragma unroll
    for (int cs = 0; cs < C / 16; cs++) {
        const bf16x8 o8 = as_bf16x8(o[cs]), d8 = as_bf16x8(d[cs]);
#pragma unroll
        for (int e = 0; e < 8; e++) sum = fmaf((float)o8[e], (float)d8[e], sum);
    }
    sum += __shfl_xor(sum, 1);
    if (q_out != nullptr) {
#pragma unroll
        for (int cs = 0; cs < C / 16; cs++) {
            bf16x8 q = as_bf16x8(*(const u32x4*)((const bf16_t*)p.q + off + cs * 16));
#pragma unroll
            for (int e = 0; e < 8; e++) q[e] = (bf16_t)((float)q[e] * q_mul);
            *(u32x4*)(q_out + off + cs * 16) = as_uint4(q);
        }
    }
    if (hf == 0) {
        const unsigned head = (unsigned)((unsigned long long)row / (unsigned)p.N), pos = (unsigned)(row - (long long)head * p.N);
        float* v = vec + (size_t)head * 2 * p.N + pos;
        v[0] = -(p.lse[row] * kLog2e);
        v[p.N] = -sum;
    }
}

// Write one wave's factor-gradient columns to LDS scratch and reduce limb columns.
// acc[mb] holds columns mb*32 + 8*g + 4*hf + x (register 4*g + x) for row l32.
// raw: the R columns are written as float without any limb summing (gradients of bf16 columns
// kept in fp32 for a later reduction).
template <int RP2, bool QSIDE, bool DL>
FB_DEV void store_dphi(const f32x16* acc_phi /* [RP2/32] */, float* scratch /* wave-private [32][RP2+1] */,
                       void* dst_row /* gradient row of this lane's token or null */, int R,
                       bool f32, bool raw, int l32, int hf, float* dslope = nullptr, float pos = 0.f) {
#pragma unroll
    for (int mb = 0; mb < RP2 / 32; mb++)
#pragma unroll
        for (int r = 0; r < 16; r++)
            scratch[l32 * (RP2 + 1) + mb * 32 + 8 * (r / 4) + 4 * hf + (r % 4)] = acc_phi[mb][r];
    __syncthreads();
    if (QSIDE && dslope != nullptr && hf == 0) {
        // ALiBi factors phi_q(i) = [-m i, m] against phi_k(j) = [1, j] (fp32 limb columns): the chain rule
        // onto the slope is dphi_q[i,1] - i dphi_q[i,0] = sum_j dS_ij (j - i).  Both terms come from the same
        // bf16 dS values through fp32 accumulators, so whatever the rows of dS fail to sum to (the error of
        // D = rowsum(dO o O)) cancels here instead of being multiplied by the position.
        const float* s = scratch + l32 * (RP2 + 1);
        const float g0 = s[0] + s[1] + s[3], g1 = s[6] + s[7] + s[9];
        *dslope = g1 - pos * g0;
    }
    if (dst_row != nullptr) {
        for (int r = hf; r < R; r += 2) {
            const float* s = scratch + l32 * (RP2 + 1);
            if (raw) {
                ((float*)dst_row)[r] = s[r];
            } else if (DL) {
                ((float*)dst_row)[r] = QSIDE ? (s[3 * r + 2] + s[3 * r + 1] + s[3 * r])       // b1, b2, b3
                                             : (s[3 * r] + s[3 * r + 1] + s[3 * r + 2]);      // a1, a2, a3
            } else if (f32) {
                // distinct limbs on the other side: query side [a1,a1,a2,a1,a2,a3] -> slots 0,2,5
                // multiply dphi_k; key side [b1,b2,b1,b3,b2,b1] -> slots 0,1,3 multiply dphi_q
                const float val = QSIDE ? (s[6 * r] + s[6 * r + 1] + s[6 * r + 3])
                                        : (s[6 * r] + s[6 * r + 2] + s[6 * r + 5]);
                ((float*)dst_row)[r] = val;
            } else {
                ((bf16_t*)dst_row)[r] = (bf16_t)s[r];
            }
        }
    }
}

// ------------------------------------------------------------------------------------------
// main kernel.  "lane side" = the 128 rows owned by the workgroup (keys when DKV, else
// queries); "streamed side" = the other index, walked in blocks of 32 rows.
//   T1 tile: rows of the streamed operand of S (Aq when DKV, else Ak), width W
//   T2 tile: rows of the streamed operand of dP (dO when DKV, else V), width C
// ------------------------------------------------------------------------------------------
// Operand rows [channels | factor columns] of one side: rows of C channels (the caller's q or k, or copies in the
// workspace) and rows of the RP2 factor columns, one set per batch element or one for all (shared).
struct OperandRows {
    const bf16_t* main;
    const bf16_t* phi;
    int shared;
};
struct MainArgs {
    OperandRows aq;       // B*H*N rows
    OperandRows ak;       // B*H*M rows
    float* vec;           // per head N values of -lse log2 e, then N of -D: written by the dq kernel, read by the dkv kernel
    float exp_mul;        // S exp_mul - lse2 is the exponent of P to base two (not used by FOLD): log2 e, times the scale where the q columns carry none
    bf16_t* q_out;        // not NULL: the dq kernel forms its operand rows as bf16(q q_mul) and leaves them here (= aq.main)
    float q_mul;
    float k_mul;          // dkv kernel, dense bias: its key rows carry the scale (else 1)
    float dkv_mul;        // factor of d[K | phi_k] (the scale, where the q columns carry none; 1 / log2 e for FOLD)
    bf16_t* ds;           // stored dS of the heads head0.. in 32 x 32 tiles (see store_ds)
    unsigned ds_pitch;    // queries and keys of a head, padded to whole tiles of the two kernels
    unsigned ds_rows;
    int head0;
};

// What a main kernel does about dS.  RECOMPUTE: each forms S, P, dP and dS itself.  STORE (dkv) leaves dS in the
// workspace, or in dBias where the bias is a dense matrix, LOAD (dq) takes it from there and is left with its output
// contraction alone.
enum { RECOMPUTE = 0, STORE = 1, LOAD = 2 };

constexpr int kWavesLd = 4;       // of the dq kernel that takes dS from the workspace
template <int C, int RP, bool LIMB, int CG>
constexpr int kSlotBytesLd = Cfg<C, RP, LIMB, CG>::T1_BYTES + kWavesLd * 32 * 32 * 2;
template <int C, int RP, bool LIMB, int CG>
constexpr int kSlotsLd = 80 * 1024 / kSlotBytesLd<C, RP, LIMB, CG>;      // two workgroups a CU

// DENSE (RP = 0 only): the bias is a dense [N][M] matrix instead of factors.  Every wave also
// copies the 32 x 32 bias tile of (its lane rows) x (the streamed block) into the slot, two
// direct loads per block; the S chain starts from those values; the dq kernel (STORE: the dkv kernel, turned in LDS) writes
// dS = dBias from its packed operand registers.
template <int C, int RP, bool CAUSAL, bool DKV, bool DENSE, bool LIMB, int CG, int MODE>
FB_DEV void bwd_tile(const BwdParams& p, const MainArgs& a, unsigned char* smem, const int bh, const int tile) {
    static_assert(!DENSE || RP == 0, "dense bias and factors are exclusive");
    constexpr bool ST = MODE == STORE, LD = MODE == LOAD;
    static_assert(!ST || DENSE || (DKV && Cfg<C, RP, LIMB, CG>::PIPE), "dS is stored by the PIPE form alone");
    constexpr int WV = LD ? kWavesLd : kWaves, kRows = WV * 32;      // waves and lane-side rows of the workgroup
    static_assert((!ST || DKV) && (!LD || !DKV) && (MODE == RECOMPUTE || CG == C), "stored dS");
    using K = Cfg<C, RP, LIMB, CG>;
    using TC = typename K::TC;
    using TP = typename K::TP;
    using T2 = typename K::T2;
    constexpr int kBiasTile = 32 * 32 * 2;     // one wave's tile: 32 rows of 64 bytes
    constexpr int kOffT2 = K::T1_BYTES, kOffVec = K::T1_BYTES + (LD ? 0 : T2::BYTES);
    constexpr int kOffBias = kOffVec + (DKV ? K::kVecBytes : 0);      // this wave's 32 x 32 tile of the dense bias, or of dS (LD)
    constexpr int kSlotBytes = kOffBias + (DENSE || LD ? WV * kBiasTile : 0);
    constexpr int ND = K::T1_NDMA + (LD ? 0 : T2::NDMA) + (DKV ? 1 : 0);       // direct loads per block
    constexpr int NDW = (ND + WV - 1) / WV;               // ... per wave, at most
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;

    // NL rows on the lane side (keys when DKV, else queries), NS rows on the streamed side
    const int NL = DKV ? p.M : p.N, NS = DKV ? p.N : p.M, R = p.R;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hf = lane >> 5;
    const int r0 = tile * kRows;          // first lane-side row of the workgroup
    const int rw0 = r0 + wave * 32;       // ... of this wave
    const int ri = rw0 + l32;             // this lane's row
    const int rc = min(ri, NL - 1);       // rows past the end compute on the last row and are not stored

    const size_t lbase = (size_t)bh * NL, sbase_rows = (size_t)bh * NS;
    const OperandRows& L1 = DKV ? a.ak : a.aq;                                      // lane-side operand of S
    const OperandRows& S1 = DKV ? a.aq : a.ak;                                      // streamed operand of S
    const int b_ = bh / p.H, h_ = bh - b_ * p.H;
    const bool q_scaled_here = !DKV && !LD && a.q_out != nullptr;                          // wave-uniform
    const bf16_t* l1m = (q_scaled_here ? (const bf16_t*)p.q : L1.main) + lbase * C;
    const bf16_t* l1p = L1.phi + (size_t)(L1.shared ? h_ : bh) * NL * K::RP2;
    const bf16_t* l2g = (const bf16_t*)(DKV ? p.v : p.dout) + lbase * C;            // lane-side operand of dP
    const bf16_t* t1m = S1.main + sbase_rows * C;
    const bf16_t* t1p = S1.phi + (size_t)(S1.shared ? h_ : bh) * NS * K::RP2;
    const float emul = a.exp_mul;
    const bf16_t* t2g = (const bf16_t*)(DKV ? p.dout : p.v) + sbase_rows * C;
    float* vecg = a.vec + (size_t)bh * 2 * p.N;                                     // per query row

    // ---- lane-side operands, loop invariant ----
    bf16x8 l1reg[K::KS], l2reg[K::CS];
#pragma unroll
    for (int ks = 0; ks < (LD ? 0 : K::KS); ks++)
        l1reg[ks] = as_bf16x8(*(const u32x4*)(ks * 16 < CG ? l1m + (size_t)rc * C + ks * 16 + 8 * hf
                                                           : l1p + (size_t)rc * K::RP2 + (ks * 16 - CG) + 8 * hf));
    if (CG == C && q_scaled_here) {
        bf16_t* qo = a.q_out + (lbase + rc) * C + 8 * hf;
#pragma unroll
        for (int ks = 0; ks < C / 16; ks++) {
#pragma unroll
            for (int e = 0; e < 8; e++) l1reg[ks][e] = (bf16_t)((float)l1reg[ks][e] * a.q_mul);
            if (ri < NL) *(u32x4*)(qo + ks * 16) = as_uint4(l1reg[ks]);
        }
    }
    if (DENSE && ST && a.k_mul != 1.f) {      // wave-uniform
#pragma unroll
        for (int ks = 0; ks < C / 16; ks++)
#pragma unroll
            for (int e = 0; e < 8; e++) l1reg[ks][e] = (bf16_t)((float)l1reg[ks][e] * a.k_mul);
    }
#pragma unroll
    for (int cs = 0; cs < (LD ? 0 : K::CS); cs++)
        l2reg[cs] = as_bf16x8(*(const u32x4*)(l2g + (size_t)rc * C + cs * 16 + 8 * hf));
    float my_nl = 0.f, my_nd = 0.f;     // dq kernel: -lse2 and -D of this lane's row (formed below, behind the first block loads)

    f32x16 acc1[K::MB];                 // dAk^T or dAq^T
    f32x16 acc2[DKV ? K::MBC : 1];      // dV^T
#pragma unroll
    for (int r = 0; r < 16; r++) {
#pragma unroll
        for (int mb = 0; mb < K::MB; mb++) acc1[mb][r] = 0.f;
#pragma unroll
        for (int mb = 0; mb < (DKV ? K::MBC : 1); mb++) acc2[mb][r] = 0.f;
    }

    // ---- streamed block range ----
    const int nblk_all = (NS + BT - 1) / BT;
    int b_begin = 0, b_end = nblk_all;
    if (CAUSAL) {
        if (DKV) b_begin = r0 / BT;                            // queries before the first key see nothing
        else b_end = min(nblk_all, (min(NS, r0 + kRows) + BT - 1) / BT);
    }
    const int nIt = b_end - b_begin;
    auto blk_of = [&](int i) __attribute__((always_inline)) { return min(b_begin + i, nblk_all - 1); };

    // ---- this wave's share of a block's direct loads: load d = wave + 4*j, j < NDW ----
    // Every wave issues NDW loads per block so that the vmcnt waits are compile-time constants and
    // the issue code carries no per-load guards: where ND is not a multiple of four the surplus
    // slots repeat load ND-1 (same source, same destination, same bytes as the wave that owns it).
    // wave-uniform per load: running source pointer of the block being issued, bytes per block,
    // LDS offset inside a slot, row-offset limit for the sequence's last (partial) block;
    // per lane: byte offset of its source row (a chunk of four values for the vec rows) and of its
    // 16 bytes inside the row
    unsigned dma_rowoff[NDW], dma_col[NDW], dma_taillim[NDW];
    const unsigned char* dma_ptr[NDW];
    int dma_bstride[NDW], dma_dst[NDW];
    const int tail_left = NS - (nblk_all - 1) * BT - 1;      // last valid row of the sequence's last block
    int dma_blk = blk_of(0);                                 // block the running pointers stand at
#pragma unroll
    for (int j = 0; j < NDW; j++) {
        const int d = min(wave + WV * j, ND - 1);
        const unsigned char* dma_src_j;
        int dma_pitch_j, dma_lshift_j;
        int row = 0, chunk = 0, dst = 0;
        if (d < K::T1_NDMA) {
            const bool fpart = d >= TC::NDMA;      // a load takes channel or factor columns, never both
            if (fpart) TP::dma_map(d - TC::NDMA, lane, row, chunk, dst);
            else TC::dma_map(d, lane, row, chunk, dst);
            const int pitch_el = fpart ? K::RP2 : C;
            dma_src_j = (const unsigned char*)(fpart ? t1p : t1m);
            dma_bstride[j] = BT * pitch_el * 2; dma_pitch_j = pitch_el * 2; dma_lshift_j = 0;
            dma_col[j] = (unsigned)chunk * 16u;
            dma_dst[j] = fpart ? TC::BYTES + dst : dst;
        } else if (d < K::T1_NDMA + T2::NDMA) {
            T2::dma_map(d - K::T1_NDMA, lane, row, chunk, dst);
            dma_src_j = (const unsigned char*)t2g;
            dma_bstride[j] = BT * C * 2; dma_pitch_j = C * 2; dma_lshift_j = 0;
            dma_col[j] = (unsigned)chunk * 16u;
            dma_dst[j] = kOffT2 + dst;
        } else {
            // vec: eight chunks of four -lse2, eight of four -D; the other lanes repeat the last chunk.  A chunk that
            // holds the head's last row may end in up to three values of whatever follows (inside the workspace).
            row = min(lane, 15) & 7;
            dma_src_j = (const unsigned char*)vecg;
            dma_bstride[j] = BT * 4; dma_pitch_j = 16; dma_lshift_j = 2;
            dma_col[j] = lane >= 8 ? (unsigned)p.N * 4u : 0u;
            dma_dst[j] = kOffVec;
        }
        dma_dst[j] = __builtin_amdgcn_readfirstlane(dma_dst[j]);     // wave-uniform by construction: keep it scalar
        dma_rowoff[j] = (unsigned)(row * dma_pitch_j);
        dma_taillim[j] = (unsigned)__builtin_amdgcn_readfirstlane((tail_left >> dma_lshift_j) * dma_pitch_j);
        dma_ptr[j] = dma_src_j + (size_t)dma_blk * dma_bstride[j];
    }
    // Blocks are issued in ascending order of i (the clamp in blk_of makes the index stall at the
    // last block), so the source pointers advance by at most one block per call.
    auto issue_block = [&](int i, int slot) __attribute__((always_inline)) {
        const int blk = blk_of(i);
        const bool adv = blk != dma_blk;       // wave-uniform; false once the index is clamped (and on the first call)
        dma_blk = blk;
        const bool tail = blk == nblk_all - 1; // rows past the sequence end repeat the last valid row
        const unsigned sbase = lds0 + slot * kSlotBytes;
#pragma unroll
        for (int j = 0; j < NDW; j++) {
            dma_ptr[j] += adv ? dma_bstride[j] : 0;
            const unsigned voff = min(dma_rowoff[j], tail ? dma_taillim[j] : ~0u) + dma_col[j];
            dma16(dma_ptr[j], voff, sbase + dma_dst[j]);
        }
    };
    // ---- dense bias tile of this wave: rows = queries, columns = keys, 64-byte rows; lane l of
    // load i covers tile row 16*i + l/4; chunk position l%4 holds 8-key chunk (l%4) ^ ((row>>2)&3)
    const unsigned char* bias_src = nullptr;   // wave-uniform base of this wave's tiles
    size_t bias_bstep = 0;                     // bytes per streamed block
    int bias_var[2], bias_pitch = 0, bias_lshift = 0;
    unsigned bias_fix[2];
    if (DENSE) {
        const bf16_t* bg = LD ? (const bf16_t*)p.dbias + (size_t)bh * p.N * p.M
                              : (const bf16_t*)p.bias + (size_t)b_ * p.bias_bstride + (size_t)h_ * p.N * p.M;
        const int Mk = p.M;
#pragma unroll
        for (int i = 0; i < 2; i++) {
            const int trow = 16 * i + (lane >> 2);
            const int c = (lane & 3) ^ ((trow >> 2) & 3);
            if (!DKV) {
                // lane side = queries: fixed row per lane; the key chunk is clamped at the sequence end
                const int rbase = min(rw0, NL - 1);
                bias_fix[i] = (unsigned)(min(rw0 + trow, NL - 1) - rbase) * (unsigned)(Mk * 2);
                bias_var[i] = c;
                bias_src = (const unsigned char*)(bg + (size_t)rbase * Mk);
            } else {
                // lane side = keys: fixed 8-key chunk per lane; the query row is clamped at the end
                const int kb = min(rw0, Mk - 8);
                bias_fix[i] = (unsigned)(min(rw0 + 8 * c, Mk - 8) - kb) * 2u;
                bias_var[i] = trow;
                bias_src = (const unsigned char*)(bg + kb);
            }
        }
        bias_pitch = DKV ? Mk * 2 : 16;
        bias_lshift = DKV ? 0 : 3;
        bias_bstep = DKV ? (size_t)BT * Mk * 2 : (size_t)BT * 2;
    }
    if (LD && !DENSE) {
        // tile (streamed block, this wave's queries), see store_ds; rows of the LDS tile = keys
#pragma unroll
        for (int i = 0; i < 2; i++) {
            const int trow = 16 * i + (lane >> 2), c = (lane & 3) ^ ((trow >> 2) & 3);
            bias_fix[i] = (unsigned)((c >> 1) * 1024 + trow * 32 + (c & 1) * 16);
        }
        bias_src = (const unsigned char*)(a.ds + (size_t)(bh - a.head0) * a.ds_rows * a.ds_pitch + (size_t)rw0 * 32);
        bias_bstep = (size_t)BT * a.ds_pitch * 2;
    }
    auto issue_bias = [&](int i, int slot) __attribute__((always_inline)) {
        if (!DENSE && !LD) return;
        const int blk = blk_of(i);
        const int left = NS - blk * BT - 1;
        const unsigned dst = lds0 + slot * kSlotBytes + kOffBias + wave * kBiasTile;
#pragma unroll
        for (int x = 0; x < 2; x++) {
            if (LD && !DENSE) dma16nt(bias_src + (size_t)blk * bias_bstep, bias_fix[x], dst + x * 1024);
            else dma16(bias_src + (size_t)blk * bias_bstep, (unsigned)(min(bias_var[x], left >> bias_lshift) * bias_pitch) + bias_fix[x], dst + x * 1024);
        }
    };
    // all but the newest block's loads (plus `stores` global stores issued since) may remain
    auto wait_prev_loads = [&](int stores) __attribute__((always_inline)) {
        // (ST: behind them also the two stores of each of the last two blocks, which every wave issues)
        constexpr int NLD = NDW + (DENSE || LD ? 2 : 0) + (ST && !DENSE ? 4 : 0);
        if (stores == 0) wait_vmcnt<NLD>();
        else wait_vmcnt_n(NLD + stores);
    };
    // per-lane offsets of the bias values of this lane's accumulator registers inside a tile:
    // group g <-> registers 4g..4g+3
    int boff[4];
#pragma unroll
    for (int g = 0; g < 4; g++) {
        if (!DKV) {
            boff[g] = l32 * 64 + ((g ^ ((l32 >> 2) & 3)) << 4) + hf * 8;             // row = query l32, keys 8g+4hf..
        } else {
            const int trow = 8 * g + 4 * hf + ((lane & 15) >> 2);                       // transpose read
            const int chunk = 2 * (l32 >> 4) + (((lane & 15) & 3) >> 1);
            boff[g] = trow * 64 + ((chunk ^ ((trow >> 2) & 3)) << 4) + (lane & 1) * 8;
        }
    }
    auto bias_init = [&](f32x16& s, int slot_off) __attribute__((always_inline)) {
        const unsigned char* tp = smem + (slot_off + kOffBias + wave * kBiasTile);
#pragma unroll
        for (int g = 0; g < 4; g++) {
            bf16x4 bv;
            if (!DKV) bv = __builtin_bit_cast(bf16x4, *(const u32x2*)(tp + boff[g]));
            else bv = __builtin_bit_cast(bf16x4, lds_read_tr16((const bf16_t*)(tp + boff[g])));
#pragma unroll
            for (int x = 0; x < 4; x++) s[4 * g + x] = (float)bv[x];
        }
    };

    // ---- per-lane LDS read offsets (bytes inside a panel) ----
    int rb64[4], rb32[2];                 // row operand, k-step j of a panel: 16 bytes at row l32
#pragma unroll
    for (int j = 0; j < 4; j++) rb64[j] = l32 * 128 + (((2 * j + hf) ^ swz64(l32)) << 4);
#pragma unroll
    for (int j = 0; j < 2; j++) rb32[j] = l32 * 64 + (((2 * j + hf) ^ swz32(l32)) << 4);
    const int i16 = lane & 15, blk16 = l32 >> 4;
    int tr64[2][2], tr32[2];              // transpose reads: 32-column block m of a panel, half hi
#pragma unroll
    for (int hi = 0; hi < 2; hi++) {
        const int row = 8 * hi + 4 * hf + (i16 >> 2);
#pragma unroll
        for (int m = 0; m < 2; m++)
            tr64[m][hi] = row * 128 + (((m * 4 + 2 * blk16 + ((i16 & 3) >> 1)) ^ swz64(row)) << 4) + (i16 & 1) * 8;
        tr32[hi] = row * 64 + (((2 * blk16 + ((i16 & 3) >> 1)) ^ swz32(row)) << 4) + (i16 & 1) * 8;
    }
    // The same offsets with a slot's byte offset added, built once per block instead of once per
    // read (the slot is a run-time value, the rest of a read's address is an immediate).
    constexpr bool ANY64 = TC::NP64 > 0 || TP::NP64 > 0;
    constexpr bool ANY32 = TC::HAS32 || TP::HAS32;
    struct RowBase { int b64[4]; int b32[2]; };
    struct TrBase { int t64[2][2]; int t32[2]; };
    auto mk_row = [&](int off) __attribute__((always_inline)) {
        RowBase r;
#pragma unroll
        for (int j = 0; j < 4; j++) r.b64[j] = ANY64 ? rb64[j] + off : 0;
#pragma unroll
        for (int j = 0; j < 2; j++) r.b32[j] = ANY32 ? rb32[j] + off : 0;
        return r;
    };
    auto mk_tr = [&](int off) __attribute__((always_inline)) {
        TrBase t;
#pragma unroll
        for (int hi = 0; hi < 2; hi++) {
#pragma unroll
            for (int m = 0; m < 2; m++) t.t64[m][hi] = ANY64 ? tr64[m][hi] + off : 0;
            t.t32[hi] = ANY32 ? tr32[hi] + off : 0;
        }
        return t;
    };
    // operand n of a block, in consumption order:
    //   [0, KS)            S   k-step n          row read of T1
    //   [KS, KS+CS)        dP  k-step n-KS       row read of T2
    //   then NO1 = 2*MB    output 1, (mb, kk)    transpose read of T1
    //   then NO2 = 2*MBC   output 2 (DKV only)   transpose read of T2   (LAZY_DS: output 2 before output 1)
    constexpr int NO1 = 2 * K::MB, NO2 = DKV ? 2 * K::MBC : 0;
    constexpr int NA = K::KS + K::CS;          // operands of the first half
    // dkv kernel, one wave per SIMD: a wave hides about five vector instructions under each MFMA.
    // With eight or more dV MFMAs (C = 128) the dS arithmetic of a block (sub, mul, convert: 40
    // instructions) fits under them, which leaves only the exponentials under the S / dP chains;
    // smaller head dimensions have too few dV MFMAs and keep everything under the first half.
    constexpr bool PIPE = DKV && K::PIPE;
    constexpr int NSLOT_DKV = K::NSLOT_DKV;
    constexpr bool LAZY_DS = PIPE && NO2 >= 8;
    constexpr int NOPS = NA + NO1 + NO2;
    // LDS operand reads run LA MFMAs ahead of their use; the first half never reads past its own block
    // (PIPE: 5..12 run within 1 %.  Plain, three against five ahead, kernel times: B 1, H 8, N 32186, C 16, R 9 dkv
    // 3179 -> 3071 us; B 4, H 16, N 4096, C 64, 64 columns dq 673 -> 658 us; C = 128 dq -1 %; N <= 1024 equal)
    constexpr int LA_WANT = PIPE ? 6 : 5;
    constexpr int LA_CAP = (NO1 + NO2) < NA ? (NO1 + NO2) : NA;
    constexpr int LA = LA_CAP < LA_WANT ? LA_CAP : LA_WANT;
    bf16x8 opr[LA + 1];
    auto row_read = [&](const RowBase& rb, int toff, int np64, int ks) __attribute__((always_inline)) {
        if (ks < np64 * 4) return as_bf16x8(*(const u32x4*)(smem + rb.b64[ks & 3] + (toff + (ks >> 2) * 4096)));
        return as_bf16x8(*(const u32x4*)(smem + rb.b32[ks - np64 * 4] + (toff + np64 * 4096)));
    };
    auto tr_read = [&](const TrBase& tb, int toff, int np64, int mb, int kk) __attribute__((always_inline)) {
        if (mb < np64 * 2) {
            const int imm = toff + (mb >> 1) * 4096 + kk * 2048;
            return join_tr(lds_read_tr16((const bf16_t*)(smem + tb.t64[mb & 1][0] + imm)),
                           lds_read_tr16((const bf16_t*)(smem + tb.t64[mb & 1][1] + imm)));
        }
        const int imm = toff + np64 * 4096 + kk * 1024;
        return join_tr(lds_read_tr16((const bf16_t*)(smem + tb.t32[0] + imm)),
                       lds_read_tr16((const bf16_t*)(smem + tb.t32[1] + imm)));
    };
    auto tr_read1 = [&](const TrBase& tb, int mb, int kk) __attribute__((always_inline)) {
        return mb < C / 32 ? tr_read(tb, 0, TC::NP64, mb, kk) : tr_read(tb, TC::BYTES, TP::NP64, mb - C / 32, kk);
    };
    // operand n of a block whose slot offset is folded into rb (row reads) / tb (transpose reads);
    // callers keep a rolling window opr[n % (LA + 1)]
    auto read_op = [&](const RowBase& rb, const TrBase& tb, int n) __attribute__((always_inline)) {
        if (n < CG / 16) return row_read(rb, 0, TC::NP64, n);
        if (n < K::KS) return row_read(rb, TC::BYTES, TP::NP64, n - CG / 16);
        if (n < NA) return row_read(rb, kOffT2, T2::NP64, n - K::KS);
        if (LAZY_DS) {
            // the P-side output (dV) first: its operand is complete when the first half ends, while dS
            // is still being formed under these MFMAs
            if (n < NA + NO2) return tr_read(tb, kOffT2, T2::NP64, (n - NA) >> 1, (n - NA) & 1);
            return tr_read1(tb, (n - NA - NO2) >> 1, (n - NA - NO2) & 1);
        }
        if (n < NA + NO1) return tr_read1(tb, (n - NA) >> 1, (n - NA) & 1);
        return tr_read(tb, kOffT2, T2::NP64, (n - NA - NO1) >> 1, (n - NA - NO1) & 1);
    };

    // Stored dS: 32 x 32 tiles of 2 KB, [key tile][query tile], so that a wave's store and load of one is contiguous (rows
    // of a whole matrix, 64 bytes a wave and block at a stride of N: B 2, H 8, N 16384 training 14.8 ms).  In a tile, piece
    // (gp, key, hf) of 16 bytes holds the queries 16 gp + 8 hf + 0..7 of a key: a lane's packed registers after one
    // exchange across the halves per register pair.  Keys past the last are zero.
    bf16_t* const ds_row = ST && !DENSE ? a.ds + (size_t)(bh - a.head0) * a.ds_rows * a.ds_pitch + (size_t)(rw0 >> 5) * 32 * a.ds_pitch + l32 * 16 + 8 * hf : nullptr;
    auto store_ds = [&](const bf16x8 (&dsb)[2], int sb0) __attribute__((always_inline)) {
        if (!ST || DENSE) return;
#pragma unroll
        for (int gp = 0; gp < 2; gp++) {
            u32x4 w = as_uint4(dsb[gp]);
            const auto r0 = __builtin_amdgcn_permlane32_swap(w.x, w.z, false, false);
            const auto r1 = __builtin_amdgcn_permlane32_swap(w.y, w.w, false, false);
            w = u32x4{(unsigned)r0[0], (unsigned)r1[0], (unsigned)r0[1], (unsigned)r1[1]};
            if (rw0 + 31 >= NL && ri >= NL) w = u32x4{0u, 0u, 0u, 0u};
            // read once, by the next launch: past the caches, which the streamed operands need (B 2, H 8, N 16384 training
            // 9256 -> 8984 us, B 4, H 16, N 4096 causal 1374 -> 1302 us with the loads marked alike)
            __builtin_nontemporal_store(w, (u32x4*)(ds_row + (size_t)sb0 * 32 + 512 * gp));
        }
    };

    // dBias = dS, by the dq kernel (dsb: keys 8g + 4 hf + 0..3 of this lane's query) or, ST, by the dkv kernel, whose lanes
    // hold queries of a key: its 32 x 32 tile is turned in LDS, in the bias tile of the block, which this wave alone reads
    // and has read.  One exchange across the halves per register pair makes whole 16-byte pieces, group 2 gp + hf in half hf.
    bf16_t* const dbg = DENSE ? (bf16_t*)p.dbias + (size_t)bh * p.N * p.M : nullptr;
    auto store_dbias = [&](const bf16x8 (&dsb)[2], int sb0, int slot_off) __attribute__((always_inline)) {
        if (!DENSE || (DKV && !ST)) return;
        u32x4 w[2] = {as_uint4(dsb[0]), as_uint4(dsb[1])};
        if (DKV) {
            unsigned char* tp = smem + (slot_off + kOffBias + wave * kBiasTile);
#pragma unroll
            for (int g = 0; g < 4; g++) {
                const u32x4 v = w[g >> 1];
                *(u32x2*)(tp + l32 * 64 + ((g ^ ((l32 >> 2) & 3)) << 4) + hf * 8) = (g & 1) ? u32x2{v.z, v.w} : u32x2{v.x, v.y};
            }
            asm volatile("" ::: "memory");
#pragma unroll
            for (int gp = 0; gp < 2; gp++)
                w[gp] = as_uint4(join_tr(lds_read_tr16((const bf16_t*)(tp + boff[2 * gp])), lds_read_tr16((const bf16_t*)(tp + boff[2 * gp + 1]))));
            asm volatile("" ::: "memory");
        }
        u32x4 piece[2];
#pragma unroll
        for (int gp = 0; gp < 2; gp++) {
            const auto r0 = __builtin_amdgcn_permlane32_swap(w[gp].x, w[gp].z, false, false);
            const auto r1 = __builtin_amdgcn_permlane32_swap(w[gp].y, w[gp].w, false, false);
            piece[gp] = u32x4{(unsigned)r0[0], (unsigned)r1[0], (unsigned)r0[1], (unsigned)r1[1]};
        }
        const int row = DKV ? sb0 + l32 : ri, col = (DKV ? rw0 : sb0) + 8 * hf;
        if (row < p.N) {
            bf16_t* drow = dbg + (size_t)row * p.M + col;
#pragma unroll
            for (int gp = 0; gp < 2; gp++)
                if (col + 16 * gp < p.M) *(u32x4*)(drow + 16 * gp) = piece[gp];
        }
    };
    // what wait_prev_loads has to allow for it (whole blocks, so all stores have issued where the wave's rows are all inside)
    const int dbias_stores = DENSE && (!DKV || ST) && rw0 + 31 < NL ? 4 : 0;

    using Yes = std::true_type;
    using No = std::false_type;
    // P and dS of one accumulator element r (streamed row sb0 + 8*(r/4) + 4*hf + (r%4), lane row ri)
    // SADD, DADD: nl and nd are still to be added (else the tiles started from them)
    auto elem = [&](int r, const f32x16& s, const f32x16& dp, float nl, float nd, auto sadd, auto dadd,
                    bf16x8 (&pb)[2], bf16x8 (&dsb)[2]) __attribute__((always_inline)) {
        const float pr = fast_exp2(sadd.value ? fmaf(s[r], emul, nl) : s[r]);
        const float ds = pr * (dadd.value ? dp[r] + nd : dp[r]);
        if (DKV) pb[r / 8][r % 8] = (bf16_t)pr;
        dsb[r / 8][r % 8] = (bf16_t)ds;
    };

    if constexpr (PIPE) {
        // One wave per SIMD (at C = 128 the accumulators alone take 144 registers), so the overlap of
        // matrix and vector work is written into the instruction stream: while the S and dP
        // chains of block i+1 run, the exponentials and dS of block i are computed, one
        // accumulator element per MFMA.  Iteration i:
        //     S, dP chains of block i+1  ||  P, dS of block i
        //     wait, barrier, issue block i+4
        //     output chains of block i, first operand reads of block i+2, (lse2, D) of block i+1
        // (LAZY_DS: only P under the first chains, dS under the dV chains, then the dK chains)
        // Ring of five slots: blocks i (transpose reads), i+1 (row reads), i+2 (prefetch),
        // i+3 (landing), i+4 (being issued).
        static_assert(NSLOT_DKV == 5, "slot arithmetic below assumes five slots");
        // SV: the S and dP tiles are produced by hand-placed MFMA forms with VGPR results (the
        // vector ALU reads them next); the compiler's own choice at one wave per SIMD is an AGPR
        // result and a v_accvgpr_read per element, 32 per block (-4 % per backward on the headline
        // shape together with the copy-free swap of the tile pairs below).  Not with a dense bias,
        // whose tile is the chain's start value.
        // Only where the kernel leaves the register allocator room (operand rows of at most 144
        // columns): in the wider instantiations every VGPR is taken, the allocator parks values in
        // spare AGPRs around the statements it cannot see into, and a copy of a tile placed right
        // behind an inner link of a chain would read it too early (seen as a wrong dK at C = 128,
        // R = 9 fp32 factors; those instantiations keep the compiler's forms).
        constexpr bool SV = !DENSE && C + RP <= 144;
        // one link of the S (n < KS) or dP chain of a block into the VGPR tiles st / dt
        auto chain_link = [&](int n, f32x16& st, f32x16& dt, bf16x8 o) __attribute__((always_inline)) {
            // the last link of each chain
            const bool last_s = n == K::KS - 1, last_d = n == NA - 1;
            if (n < K::KS) {
                if (n == 0) mfma32_vdst_first(st, o, l1reg[n]);
                else if (last_s) mfma32_vdst_last(st, o, l1reg[n]);
                else mfma32_vdst(st, o, l1reg[n]);
            } else {
                if (n == K::KS) mfma32_vdst_first(dt, o, l2reg[n - K::KS]);
                else if (last_d) mfma32_vdst_last(dt, o, l2reg[n - K::KS]);
                else mfma32_vdst(dt, o, l2reg[n - K::KS]);
            }
        };
        static_assert(!SV || (K::KS >= 2 && NA - K::KS >= 2), "a first and a last link per chain");
        issue_block(0, 0); issue_bias(0, 0);
        issue_block(1, 1); issue_bias(1, 1);
        issue_block(2, 2); issue_bias(2, 2);
        issue_block(3, 3); issue_bias(3, 3);
        wait_vmcnt<0>();
        __syncthreads();
        f32x16 sA, dA, sB, dB;
        {
            const RowBase r0 = mk_row(0);
            const TrBase t0 = mk_tr(0);
#pragma unroll
            for (int r = 0; r < 16; r++) { sA[r] = 0.f; dA[r] = 0.f; }
            if (DENSE) bias_init(sA, 0);
#pragma unroll
            for (int n = 0; n < NA; n++) {
                const bf16x8 o = read_op(r0, t0, n);
                if (SV) {
                    chain_link(n, sA, dA, o);
                } else {
                    if (n < K::KS) sA = mfma32(o, l1reg[n], sA);
                    else dA = mfma32(o, l2reg[n - K::KS], dA);
                }
            }
        }
        RowBase rb1 = mk_row(kSlotBytes);     // rows of block i+1
#pragma unroll
        for (int n = 0; n < LA; n++) opr[n] = read_op(rb1, TrBase{}, n);
        // -lse2 and -D of the 16 streamed rows this lane's accumulator registers belong to, one block ahead
        f32x4 vq[4], vd[4];
        const int vlane = kOffVec + 16 * hf;
        auto read_vec = [&](int off) __attribute__((always_inline)) {
            const unsigned char* vp = smem + (vlane + off);
#pragma unroll
            for (int g = 0; g < 4; g++) {
                vq[g] = *(const f32x4*)(vp + 32 * g);
                vd[g] = *(const f32x4*)(vp + 32 * g + 128);
            }
        };
        read_vec(0);
        int sl = 0;   // slot of block i
        const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        auto body = [&](int i, const f32x16& sc, const f32x16& dc, f32x16& sn, f32x16& dn)
                        __attribute__((always_inline)) {
            const int sl1 = sl + 1 >= NSLOT_DKV ? sl + 1 - NSLOT_DKV : sl + 1;
            const int sl2 = sl + 2 >= NSLOT_DKV ? sl + 2 - NSLOT_DKV : sl + 2;
            const int sl4 = sl == 0 ? NSLOT_DKV - 1 : sl - 1;
            const TrBase tb0 = mk_tr(sl * kSlotBytes);          // transpose reads of block i
            const RowBase rb2 = mk_row(sl2 * kSlotBytes);       // rows of block i+2
            const int sb0 = blk_of(i) * BT;
            const bool need_mask = (sb0 + BT > NS) || (CAUSAL && sb0 < rw0 + 31);
            bf16x8 pb[2], dsb[2];
            float prf[16];                                      // P of block i in fp32, until dS is formed
            f32x16 sinit = zero;
            if (DENSE) bias_init(sinit, sl1 * kSlotBytes);      // S of block i+1 starts from its bias tile
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int n = 0; n < NA; n++) {
                opr[(n + LA) % (LA + 1)] = read_op(rb1, tb0, n + LA);   // past NA: output operands of block i
                if (SV) {
                    chain_link(n, sn, dn, opr[n % (LA + 1)]);
                } else {
                    if (n < K::KS) sn = mfma32(opr[n % (LA + 1)], l1reg[n], n == 0 ? sinit : sn);
                    else dn = mfma32(opr[n % (LA + 1)], l2reg[n - K::KS], n == K::KS ? zero : dn);
                }
#pragma unroll
                for (int e = (n * 16) / NA; e < ((n + 1) * 16) / NA; e++) {
                    if (LAZY_DS) {
                        prf[e] = fast_exp2(fmaf(sc[e], emul, vq[e >> 2][e & 3]));
                        pb[e / 8][e % 8] = (bf16_t)prf[e];
                    } else {
                        elem(e, sc, dc, vq[e >> 2][e & 3], vd[e >> 2][e & 3], Yes{}, Yes{}, pb, dsb);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (need_mask) {
                // rare (diagonal blocks, sequence end): zero the dead elements afterwards, behind a real
                // branch, so the common path carries no compares and selects.  NaNs from filler rows
                // past N are discarded here as well.  LAZY_DS: with P zeroed, dS = P (dP - D) formed
                // later is zero too; the (lse, D) pair of a filler row past the sequence end is whatever
                // follows in memory, so its D is replaced to keep 0 * (dP - D) at 0.
                asm volatile("" ::: "memory");
#pragma unroll
                for (int r = 0; r < 16; r++) {
                    const int srow = sb0 + 8 * (r / 4) + 4 * hf + (r % 4);
                    if (srow >= NS || (CAUSAL && srow < ri)) {
                        pb[r / 8][r % 8] = (bf16_t)0.f;
                        if (LAZY_DS) prf[r] = 0.f;
                        else dsb[r / 8][r % 8] = (bf16_t)0.f;
                    }
                    if (LAZY_DS && srow >= NS) vd[r >> 2][r & 3] = 0.f;
                }
            }
            // block i+2 has landed; everyone has left block i-1
            wait_prev_loads(dbias_stores);
            __syncthreads();
            issue_block(i + 4, sl4);
            issue_bias(i + 4, sl4);
            bf16x8 nxt[LA];
#pragma unroll
            for (int n = NA; n < NOPS; n++) {
                if (n + LA < NOPS) opr[(n + LA) % (LA + 1)] = read_op(rb1, tb0, n + LA);
                else nxt[n + LA - NOPS] = read_op(rb2, tb0, n + LA - NOPS);   // row operands of block i+2
                const int m = n - NA;
                if (!LAZY_DS) {
                    if (m < NO1) acc1[m >> 1] = mfma32(opr[n % (LA + 1)], dsb[m & 1], acc1[m >> 1]);
                    else acc2[(m - NO1) >> 1] = mfma32(opr[n % (LA + 1)], pb[(m - NO1) & 1], acc2[(m - NO1) >> 1]);
                } else if (m < NO2) {
                    acc2[m >> 1] = mfma32(opr[n % (LA + 1)], pb[m & 1], acc2[m >> 1]);
                    // dS of block i under the dV MFMAs, 16 / NO2 elements per MFMA
#pragma unroll
                    for (int e = (m * 16) / NO2; e < ((m + 1) * 16) / NO2; e++)
                        dsb[e / 8][e % 8] = (bf16_t)(prf[e] * (dc[e] + vd[e >> 2][e & 3]));
                    __builtin_amdgcn_sched_barrier(0);
                } else {
                    acc1[(m - NO2) >> 1] = mfma32(opr[n % (LA + 1)], dsb[(m - NO2) & 1], acc1[(m - NO2) >> 1]);
                }
            }
            store_ds(dsb, sb0);
            store_dbias(dsb, sb0, sl * kSlotBytes);
#pragma unroll
            for (int n = 0; n < LA; n++) opr[n] = nxt[n];
            read_vec(sl1 * kSlotBytes);
            rb1 = rb2;
            sl = sl1;
        };
        int i = 0;
        if (SV) {      // two steps at a time: the two pairs of score tiles swap roles without copies
            for (; i + 2 <= nIt; i += 2) {
                body(i, sA, dA, sB, dB);
                body(i + 1, sB, dB, sA, dA);
            }
        }
        // (with compiler-placed MFMA results, unrolling by two makes the register allocator shuffle all
        // accumulators between VGPRs and AGPRs; the 32 copies are cheaper there)
        for (; i < nIt; i++) {
            body(i, sA, dA, sB, dB);
            sA = sB;
            dA = dB;
        }
    } else if constexpr (LD) {
        // dS comes from the workspace, 2 KB a wave and block beside the shared operand tile.  Bound by that read, 4.2 TB/s
        // where the dS of a launch is far larger than the last-level cache (C = 128, R 8: 10 matrix instructions a block
        // where the recomputing form has 27; B 2, H 8, N 16384 3110 -> 2040 us).  Eight waves with a ring of 160 KB: 315 us
        // a launch of 2 heads against 254, half the workgroups.  From dBias (B 8, H 12, N 1024, C 64, 200 MB): 45 us, where
        // the recomputing form takes 103; the dkv kernel that writes it 100 instead of 82.
        constexpr int NS_ = kSlotsLd<C, RP, LIMB, CG>;
#pragma unroll
        for (int j = 0; j < NS_ - 1; j++) { issue_block(j, j); issue_bias(j, j); }
        wait_vmcnt<0>();
        __syncthreads();
        auto read_d = [&](int slot_off, int kk, int blk) __attribute__((always_inline)) {
            if (DENSE) {
                const unsigned char* t = smem + (slot_off + kOffBias + wave * kBiasTile);
                const u32x2 lo = *(const u32x2*)(t + boff[2 * kk]), hi = *(const u32x2*)(t + boff[2 * kk + 1]);
                u32x4 w = {lo.x, lo.y, hi.x, hi.y};
                const int left = NS - blk * BT - 16 * kk;      // keys past the last, in whole eights
                if (left < 16) {
                    if (left <= 8) w.z = w.w = 0u;
                    if (left <= 0) w.x = w.y = 0u;
                }
                return as_bf16x8(w);
            }
            const unsigned char* t = smem + (slot_off + kOffBias + wave * kBiasTile + kk * 1024);
            return join_tr(lds_read_tr16((const bf16_t*)(t + tr32[0])), lds_read_tr16((const bf16_t*)(t + tr32[1])));
        };
        constexpr int LB = NO1 < 4 ? NO1 : 4;       // operands read ahead
        bf16x8 opd[LB + 1], dcur[2];
        {
            const TrBase t0 = mk_tr(0);
#pragma unroll
            for (int n = 0; n < LB; n++) opd[n] = tr_read1(t0, n >> 1, n & 1);
#pragma unroll
            for (int kk = 0; kk < 2; kk++) dcur[kk] = read_d(0, kk, blk_of(0));
        }
        static_assert(!CAUSAL || kRows == 128, "the dkv launch leaves dS of whole 128-row tiles on and below the diagonal: the blocks walked here");
        int sl = 0;
        for (int i = 0; i < nIt; i++) {
            const int sln = sl + 1 == NS_ ? 0 : sl + 1, slp = sl == 0 ? NS_ - 1 : sl - 1;
            const int off = sl * kSlotBytes, offn = sln * kSlotBytes;
            const TrBase tb0 = mk_tr(off), tbn = mk_tr(offn);
            wait_vmcnt<(NDW + 2) * (NS_ - 3)>();       // block i + 1 has landed; everyone has left block i - 1
            __syncthreads();
            issue_block(i + NS_ - 1, slp);
            issue_bias(i + NS_ - 1, slp);
            bf16x8 nxt[LB], dn[2];
#pragma unroll
            for (int n = 0; n < NO1; n++) {
                if (n + LB < NO1) opd[(n + LB) % (LB + 1)] = tr_read1(tb0, (n + LB) >> 1, (n + LB) & 1);
                else nxt[n + LB - NO1] = tr_read1(tbn, (n + LB - NO1) >> 1, (n + LB - NO1) & 1);
                if (n >= NO1 - 2) dn[n - (NO1 - 2)] = read_d(offn, n - (NO1 - 2), blk_of(i + 1));
                acc1[n >> 1] = mfma32(opd[n % (LB + 1)], dcur[n & 1], acc1[n >> 1]);
            }
#pragma unroll
            for (int n = 0; n < LB; n++) opd[n] = nxt[n];
#pragma unroll
            for (int kk = 0; kk < 2; kk++) dcur[kk] = dn[kk];
            sl = sln;
        }
    } else {
        // Two or three waves per SIMD: another workgroup's wave fills the gaps.  Iteration i:
        //     S, dP chains of block i | P, dS | wait, barrier | issue block i+3 |
        //     output chains of block i, first operand reads of block i+1
        issue_block(0, 0); issue_bias(0, 0);
        issue_block(1, 1); issue_bias(1, 1);
        issue_block(2, 2); issue_bias(2, 2);
        // This kernel owns every query row once and already holds the row's dO: it forms
        // D = rowsum(dO o O) and lse log2 e itself and leaves the pair for the dkv kernel, which is
        // launched behind it (no separate pass over out and dO).  Placed here so that the row loads
        // are in flight together with the first blocks.
        if (!DKV) {
            const bf16_t* og = (const bf16_t*)p.out + (lbase + rc) * CG;
            float dsum = 0.f;
#pragma unroll
            for (int cs = 0; cs < K::CS; cs++) {
                {
                    const bf16x8 o8 = as_bf16x8(*(const u32x4*)(og + cs * 16 + 8 * hf));
#pragma unroll
                    for (int e = 0; e < 8; e++) dsum = fmaf((float)o8[e], (float)l2reg[cs][e], dsum);
                }
            }
            dsum += __shfl_xor(dsum, 32);
            my_nd = -dsum;
            my_nl = -(p.lse[lbase + rc] * kLog2e);
            if (hf == 0 && ri < NL) {
                vecg[ri] = my_nl;
                vecg[NL + ri] = my_nd;
            }
        }
        wait_vmcnt<0>();
        __syncthreads();
        RowBase rb0 = mk_row(0);
#pragma unroll
        for (int n = 0; n < LA; n++) opr[n] = read_op(rb0, TrBase{}, n);

        // Start values of the tiles.  dkv: dP from -D (and S from -lse2, FOLD), read straight into the accumulators in
        // the second half of the block before.  dq at C = 32: the same from this lane's pair; the wider ones have no
        // registers for it.  A started dP saves its subtraction, FOLD the multiply-add, of about 100 vector
        // instructions a block where the vector ALU is the bound.
        constexpr bool SINIT = K::FOLD, DINIT = DKV || C == 32;
        f32x16 s, dp;
        auto init_tiles = [&](int off) __attribute__((always_inline)) {
            const unsigned char* vp = smem + (off + kOffVec + 16 * hf);
#pragma unroll
            for (int g = 0; g < 4; g++) {
                f32x4 a4 = {0.f, 0.f, 0.f, 0.f}, b4 = {0.f, 0.f, 0.f, 0.f};
                if (DKV) {
                    if (SINIT) a4 = *(const f32x4*)(vp + 32 * g);
                    b4 = *(const f32x4*)(vp + 32 * g + 128);
                } else {
                    if (SINIT) a4 = f32x4{my_nl, my_nl, my_nl, my_nl};
                    if (DINIT) b4 = f32x4{my_nd, my_nd, my_nd, my_nd};
                }
#pragma unroll
                for (int x = 0; x < 4; x++) { s[4 * g + x] = a4[x]; dp[4 * g + x] = b4[x]; }
            }
        };
        init_tiles(0);
        for (int i = 0; i < nIt; i++) {
            const int slot = i & (NSLOT - 1);
            const TrBase tb0 = mk_tr(slot * kSlotBytes);
            const RowBase rbn = mk_row(((i + 1) & (NSLOT - 1)) * kSlotBytes);
            const int sb0 = blk_of(i) * BT;      // first streamed row of the block

            // ---------------- first half: S and dP chains ----------------
            if (DENSE) bias_init(s, slot * kSlotBytes);
#pragma unroll
            for (int n = 0; n < NA; n++) {
                opr[(n + LA) % (LA + 1)] = read_op(rb0, tb0, n + LA);   // n + LA < NOPS: the output operands follow
                if (n < K::KS) s = mfma32(opr[n % (LA + 1)], l1reg[n], s);
                else dp = mfma32(opr[n % (LA + 1)], l2reg[n - K::KS], dp);
            }
            // ---------------- P and dS in accumulator layout ----------------
            bf16x8 pb[2], dsb[2];
            using SAdd = std::integral_constant<bool, !SINIT>;
            using DAdd = std::integral_constant<bool, !DINIT>;
            f32x4 nl4 = {my_nl, my_nl, my_nl, my_nl};
#pragma unroll
            for (int r = 0; r < 16; r++) {
                if (DKV && !SINIT && r % 4 == 0) nl4 = *(const f32x4*)(smem + (slot * kSlotBytes + kOffVec + 16 * hf + 8 * r));
                elem(r, s, dp, nl4[r % 4], my_nd, SAdd{}, DAdd{}, pb, dsb);
            }
            if ((sb0 + BT > NS) || (CAUSAL && (DKV ? sb0 < rw0 + 31 : sb0 + BT - 1 > rw0))) {
                // rare (diagonal blocks, sequence end): zero the dead elements behind a real branch
                asm volatile("" ::: "memory");
#pragma unroll
                for (int r = 0; r < 16; r++) {
                    const int srow = sb0 + 8 * (r / 4) + 4 * hf + (r % 4);
                    if (srow >= NS || (CAUSAL && (DKV ? srow < ri : srow > ri))) {
                        dsb[r / 8][r % 8] = (bf16_t)0.f;
                        if (DKV) pb[r / 8][r % 8] = (bf16_t)0.f;
                    }
                }
            }
            // ---------------- block i+1 has landed; everyone has left block i-1 ----------------
            // (behind them lie the loads of block i+2 and, with a dense bias, the dBias stores of the two blocks before
            // this one)
            wait_prev_loads(dbias_stores);
            __syncthreads();
            issue_block(i + 3, (i + 3) & (NSLOT - 1));
            issue_bias(i + 3, (i + 3) & (NSLOT - 1));

            // ---------------- dBias = dS, issued behind the loads: a store has two blocks' time before anything waits for
            // it (dq, B 8, H 12, N 1024, C 64: 110 -> 100 us) ----------------
            store_dbias(dsb, sb0, slot * kSlotBytes);

            // ---------------- second half: output chains ----------------
            bf16x8 nxt[LA];      // first operands of block i+1 (the window restarts at 0 with every block)
#pragma unroll
            for (int n = NA; n < NOPS; n++) {
                if (n + LA < NOPS) opr[(n + LA) % (LA + 1)] = read_op(rb0, tb0, n + LA);
                else nxt[n + LA - NOPS] = read_op(rbn, tb0, n + LA - NOPS);
                const int m = n - NA;
                if (m < NO1) acc1[m >> 1] = mfma32(opr[n % (LA + 1)], dsb[m & 1], acc1[m >> 1]);
                else acc2[(m - NO1) >> 1] = mfma32(opr[n % (LA + 1)], pb[(m - NO1) & 1], acc2[(m - NO1) >> 1]);
            }
#pragma unroll
            for (int n = 0; n < LA; n++) opr[n] = nxt[n];
            init_tiles(((i + 1) & (NSLOT - 1)) * kSlotBytes);
            rb0 = rbn;
        }
    }
    if (DENSE && !DKV && CAUSAL && ri < NL) {
        // key blocks above the diagonal are never visited: their dBias is zero
        for (int blk = b_end; blk < nblk_all; blk++) {
            bf16_t* drow = dbg + (size_t)ri * p.M + blk * BT + 8 * hf;
#pragma unroll
            for (int gp = 0; gp < 2; gp++)
                if (blk * BT + 16 * gp + 8 * hf < p.M) *(u32x4*)(drow + 16 * gp) = u32x4{0u, 0u, 0u, 0u};
        }
    }
    wait_vmcnt<0>();     // no direct load may outlive this tile's use of the ring
    __syncthreads();

    // ---- epilogue ----
    if (DKV && a.dkv_mul != 1.f) {      // wave-uniform: the q columns carried no scale
#pragma unroll
        for (int mb = 0; mb < K::MB; mb++)
#pragma unroll
            for (int r = 0; r < 16; r++) acc1[mb][r] *= a.dkv_mul;
    }
    const bool rok = ri < NL;
    constexpr int Cg = CG;    // channels of the caller's gradient rows (< C: the rest is not stored)
    const size_t base = (size_t)bh * NL * Cg;
    const bool g32 = p.grad_f32 != 0;      // wave-uniform
    if (rok) {
        if (DKV) {
            bf16_t* dvg = (bf16_t*)p.dv + base + (size_t)ri * Cg;
            bf16_t* dkg = (bf16_t*)p.dk + base + (size_t)ri * Cg;
            float* dkf = (float*)p.dk + base + (size_t)ri * Cg;
#pragma unroll
            for (int mb = 0; mb < K::MBC; mb++)
#pragma unroll
                for (int g = 0; g < 4; g++) {
                    if (mb * 32 + 8 * g >= Cg) continue;
                    bf16x4 a4, b4;
                    f32x4 bf;
#pragma unroll
                    for (int x = 0; x < 4; x++) {
                        a4[x] = (bf16_t)acc2[mb][4 * g + x];
                        b4[x] = (bf16_t)acc1[mb][4 * g + x];
                        bf[x] = acc1[mb][4 * g + x];
                    }
                    *(u32x2*)(dvg + mb * 32 + 8 * g + 4 * hf) = __builtin_bit_cast(u32x2, a4);
                    if (g32) *(f32x4*)(dkf + mb * 32 + 8 * g + 4 * hf) = bf;
                    else *(u32x2*)(dkg + mb * 32 + 8 * g + 4 * hf) = __builtin_bit_cast(u32x2, b4);
                }
        } else {
            bf16_t* dqg = (bf16_t*)p.dq + base + (size_t)ri * Cg;
            float* dqf = (float*)p.dq + base + (size_t)ri * Cg;
#pragma unroll
            for (int mb = 0; mb < K::MBC; mb++)
#pragma unroll
                for (int g = 0; g < 4; g++) {
                    if (mb * 32 + 8 * g >= Cg) continue;
                    bf16x4 o4;
                    f32x4 of;
#pragma unroll
                    for (int x = 0; x < 4; x++) {
                        of[x] = acc1[mb][4 * g + x] * p.scale;
                        o4[x] = (bf16_t)of[x];
                    }
                    if (g32) *(f32x4*)(dqf + mb * 32 + 8 * g + 4 * hf) = of;
                    else *(u32x2*)(dqg + mb * 32 + 8 * g + 4 * hf) = __builtin_bit_cast(u32x2, o4);
                }
        }
    }
    if (RP > 0) {
        const bool f32 = p.phi_f32 != 0;
        const size_t esz = (f32 || g32) ? 4 : 2;
        float* scratch = (float*)smem + wave * 32 * (K::MBP * 32 + 1);
        unsigned char* dst = nullptr;
        unsigned char* const dphi = (unsigned char*)(DKV ? p.dphi_k : p.dphi_q);     // NULL: factor gradients not wanted
        if (rok && dphi != nullptr) dst = dphi + ((size_t)bh * NL + ri) * R * esz;
        // the key-side limb order applies to the key's own gradient and vice versa
        float* dsl = nullptr;
        if (!DKV && rok && p.slopes != nullptr && p.dslope != nullptr) dsl = p.dslope + (size_t)bh * NL + ri;
        store_dphi<K::MBP * 32, !DKV, K::DL>(&acc1[K::MBC], scratch, dst, R, f32, g32, l32, hf, dsl, (float)ri);
    }
}

// Work units: one 128-row tile per workgroup, or when causal the tile pair (n-1-u, u), whose
// streamed ranges add up to the same length for every u (no tail of heavy tiles).
template <int C, int RP, bool CAUSAL, bool DKV, bool DENSE, bool LIMB, int CG, int MODE = RECOMPUTE>
__global__ __launch_bounds__(MODE == LOAD ? kWavesLd * 64 : kThreads, (DKV ? Cfg<C, RP>::PIPE : (MODE == RECOMPUTE && (DENSE || C + RP > 160))) ? 1 : 2) void bwd_main_kernel(BwdParams p, MainArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int L = (blockIdx.x & 7) * p.tiles_per_xcd + (blockIdx.x >> 3);
    if (L >= p.total_tiles) return;
    const int n_units = CAUSAL ? (p.n_tiles + 1) / 2 : p.n_tiles;   // p.n_tiles: 128-row tiles of the lane side
    const int bhl = L / n_units, bh = MODE == RECOMPUTE || DENSE ? bhl : a.head0 + bhl;
    const int u = L - bhl * n_units;
    if (CAUSAL) {
        const int other = p.n_tiles - 1 - u;
        // heavier tile first: high query tiles for dq, low key tiles for dkv
        bwd_tile<C, RP, CAUSAL, DKV, DENSE, LIMB, CG, MODE>(p, a, smem, bh, DKV ? u : other);
        if (u != other) {
            __syncthreads();   // the epilogue's LDS scratch is reused as ring memory
            bwd_tile<C, RP, CAUSAL, DKV, DENSE, LIMB, CG, MODE>(p, a, smem, bh, DKV ? other : u);
        }
    } else {
        bwd_tile<C, RP, CAUSAL, DKV, DENSE, LIMB, CG, MODE>(p, a, smem, bh, u);
    }
}

// Instantiations with a stored dS: where the dq kernel's recomputation takes clearly longer than 4 KB a 32 x 32 block to
// memory and back.  Training, start / stored (us), C = 128: B 2, H 8, N 16384 9590 / 8984; B 4, H 16, N 4096 causal 1377 /
// 1302; B 4, H 8, N 4096 1296 / 1194; B 1, H 2, N 8192 606 / 510; B 8, H 8, N 2048 696 / 661.  C = 64: B 8, H 12, N 1024,
// R 32 204 / 209; B 8, H 8, N 2048, R 16 413 / 418; two columns of 64 (multiplicative) 2060 / 2065: left.
template <int C, int RP, bool DENSE, int CG>
constexpr bool kStored = DENSE ? CG == C : C == 128;
// What is saved grows with the pairs, what the extra launch and the pass over the query rows cost with the call and the rows
// (start / stored, us, C = 128, R 8): 512 heads of N 256 181 / 188, 128 of 512 159 / 164, 32 of 1024 158 / 161 (8.4 M by this
// measure); 64 of 1024 202 / 196 (16.8 M), 256 of 1000 770 / 752, 8 of 2048 172 / 151 (21 M), 2 of 4096 313 / 266, causal 15
// of 3000 288 / 261.
bool stored_pays(long long heads, int N, int M, bool causal) {
    return (double)heads * N * ((causal ? 0.5 : 1.0) * M - 768.0) >= (double)(1 << 24);
}
// With a dense bias dBias is that dS: the dkv kernel writes it, the dq kernel reads it (start / now, us: B 8, H 12, N 1024, C 64
// 272 / 242, causal N 1000 243 / 242; C 128: B 2, H 8, N 2048 296 / 267, causal 318 / 279; C 32: B 8, H 16, N 1024 306 / 286;
// B 1, H 2, N 2048, C 64 161 / 134).  Not in calls that the launches bound, which one more costs 3 us of 140: B 4, H 8,
// N 512, C 64 140 / 143, B 64, H 16, N 128, C 64 146 / 149, B 16, H 16, N 512, C 32 142 / 145,
// B 1, H 2, N 1024, C 64 122 / 125.
bool dense_stored_pays(long long heads, int N, int M, int C) {
    const double pairs = (double)heads * N * M;
    return (N >= 1024 && M >= 1024 && pairs >= (double)(1 << 23)) || pairs * (C == 32 ? 16 : C) >= (double)(1u << 31);
}
constexpr size_t kMaxStored = (size_t)1 << 30;      // at a time
// dS of one head, whole tiles (any int: the size queries come before the limits are checked; at most 2^63).
size_t ds_head_bytes(int N, int M) { return ((size_t)N + 127) / 128 * 128 * (((size_t)M + 127) / 128 * 128) * 2; }
// Heads per launch whose dS fits `room` bytes, 0: recompute.  (256 CUs where there is no device to ask, as in a size query on another host.)
int stored_heads(long long heads, int N, int M, bool causal, size_t room) {
    const size_t per = ds_head_bytes(N, M);
    if (room > kMaxStored) room = kMaxStored;
    const long long fit = (long long)(room / per);
    if (fit <= 0) return 0;
    if (!stored_pays(heads, N, M, causal)) return 0;
    if (fit >= heads) return (int)heads;
    // the dkv launches' rounds of workgroups (one a CU): per head, against those of one launch over all heads
    const int tiles = (M + 127) / 128;
    const int cus = fb_cu_count();
    const long long units = causal ? (tiles + 1) / 2 : tiles, slots = cus > 0 ? cus : 256;
    auto rounds = [&](long long h) { return (double)((h * units + slots - 1) / slots); };
    long long best = 0;
    double cost = 1.1 * rounds(heads);
    // (of the chunks that take equally many rounds the largest is never the worse one: the next smaller one tried is the
    // largest of one round less, a few steps where the head counts of short heads are thousands)
    for (long long c = fit; c >= 1 && c * 4 >= fit; c = ((long long)rounds(c) - 1) * slots / units) {
        const long long whole = heads / c, rest = heads - whole * c;
        const double t = whole * rounds(c) + (rest > 0 ? rounds(rest) : 0.0);
        if (t < cost) { best = c; cost = t; }
    }
    return (int)best;
}

// Pre-pass and the two main kernels.  DENSE: the bias is a dense matrix streamed tile by tile
// (RP = 0) and the dq kernel, or where dBias is read back as dS the dkv kernel, also writes dBias.
template <int C, int RP, bool CAUSAL, bool DENSE, bool LIMB, int CG>
int launch(const BwdParams& pin, hipStream_t stream) {
    using K = Cfg<C, RP, LIMB, CG>;
    constexpr size_t slot = K::T1_BYTES + K::T2::BYTES + (DENSE ? (size_t)kWaves * 32 * 32 * 2 : 0);
    constexpr size_t ring_dq = (size_t)NSLOT * slot;
    constexpr size_t ring_dkv = (size_t)K::NSLOT_DKV * (slot + K::kVecBytes);
    constexpr size_t lds_dq = ring_dq > K::kEpiLds ? ring_dq : K::kEpiLds;
    constexpr size_t lds_dkv = ring_dkv > K::kEpiLds ? ring_dkv : K::kEpiLds;
    auto kdq = bwd_main_kernel<C, RP, CAUSAL, false, DENSE, LIMB, CG>;
    auto kdkv = bwd_main_kernel<C, RP, CAUSAL, true, DENSE, LIMB, CG>;
    static FbLdsOnce once_dq, once_dkv;
    if (!fb_raise_lds_limit((const void*)kdq, lds_dq, once_dq) || !fb_raise_lds_limit((const void*)kdkv, lds_dkv, once_dkv))
        return 1;

    const long long rows = (long long)pin.B * pin.H * pin.N;      // query rows
    const long long rowsk = (long long)pin.B * pin.H * pin.M;     // key rows
    if (pin.Cg != CG || (LIMB && !pin.phi_f32) || (K::DL && pin.R > 10)) return -1;
    // k is read in place.  On the query side the q columns carry the scale; it can move onto the factor columns (as
    // 1/scale) and into the exponent and the dK epilogue, so that q is read in place too -- where the forward formed
    // its scores that way as well (lse and D belong to the forward's scores, and the recomputed ones must be those):
    // C = 64 and 128 with no factors, fp32 factors (scaled before the limb split) and ALiBi factors made in the
    // kernels; and wherever bf16(q scale) = q scale, i.e. for a scale that is a power of two (head dimension 64 at the
    // default scale with bf16 factors, and the multiplicative form, whose prepared rows carry their scale already).
    // Never with a dense bias, which enters the chain unscaled.  Elsewhere the dq kernel, which holds every q row
    // once, leaves the scaled rows for the dkv kernel.
    int mant_exp = 0;
    const bool pow2 = std::frexp(pin.scale, &mant_exp) == 0.5f;
    const bool f32_factors = pin.phi_f32 != 0 || pin.slopes != nullptr;
    const bool raw_q = !DENSE && (score_raw_q(CG, RP > 0 && !f32_factors) || (C % 64 == 0 && pow2));
    const float qscale = K::FOLD ? pin.scale * kLog2e : pin.scale;      // the forward's product
    const float qmul = raw_q ? 1.f / pin.scale : (K::FOLD ? kLog2e : 1.f);
    // workspace: vec [rows][2] float | Aq: scaled rows of C channels, factor rows | Ak: (head dimension 16: widened
    // rows), factor rows | head dimension 16: widened v, dO  (each a multiple of 16 bytes)
    unsigned char* ws = (unsigned char*)pin.workspace;
    MainArgs a;
    a.vec = (float*)ws;
    bf16_t* next = (bf16_t*)(ws + (((size_t)rows * 8 + 15) & ~(size_t)15));
    auto take = [&](long long n_rows, int width) {
        bf16_t* r = next;
        next += (size_t)n_rows * width;
        return r;
    };
    const int shared_q = pin.slopes != nullptr || pin.phi_bstride == 0, shared_k = pin.slopes != nullptr || pin.phik_bstride == 0;
    const long long prows_q = RP == 0 ? 0 : shared_q ? (long long)pin.H * pin.N : rows;
    const long long prows_k = RP == 0 ? 0 : shared_k ? (long long)pin.H * pin.M : rowsk;
    bf16_t* aqm = raw_q ? nullptr : take(rows, C);
    bf16_t* aqp = take(prows_q, K::RP2);
    bf16_t* akm = CG < C ? take(rowsk, C) : nullptr;
    bf16_t* akp = take(prows_k, K::RP2);
    a.aq = OperandRows{raw_q ? (const bf16_t*)pin.q : aqm, aqp, shared_q};
    a.ak = OperandRows{CG < C ? akm : (const bf16_t*)pin.k, akp, shared_k};
    a.q_out = raw_q || CG < C ? nullptr : aqm;
    a.q_mul = qscale;
    a.k_mul = 1.f;
    a.exp_mul = raw_q ? kLog2e * pin.scale : kLog2e;
    a.dkv_mul = raw_q ? pin.scale : (K::FOLD ? kLn2 : 1.f);

    BwdParams p = pin;
    if constexpr (CG < C) {
        // out and dO keep their 16-channel rows for the row sums
        const Widen16 w{aqm, take(rows, C), akm, take(rowsk, C)};
        const long long most = rows > rowsk ? rows : rowsk;
        hipLaunchKernelGGL(bwd_widen16_kernel, dim3((unsigned)((most * 4 + 255) / 256), 4), dim3(256), 0, stream, pin, w,
                           rows, rowsk, qscale);
        p.v = w.v;
        p.dout = w.dout;
    }
    if constexpr (RP > 0) {
        constexpr int RPB = kPrepRows<K::RP2>;
        const unsigned nb_q = (unsigned)((prows_q + RPB - 1) / RPB), nb_k = (unsigned)((prows_k + RPB - 1) / RPB);
        hipLaunchKernelGGL((bwd_pre_kernel<K::RP2, K::DL>), dim3(nb_q + nb_k), dim3(256), 0, stream, pin, aqp, akp, nb_q,
                           prows_q, prows_k, qmul);
    }
    if (hipGetLastError() != hipSuccess) return 1;

    const int all_heads = p.B * p.H;
    auto set_tiles = [](BwdParams& p, int lane_rows, int heads, int tile_rows = 128) {
        p.n_tiles = (lane_rows + tile_rows - 1) / tile_rows;
        const int n_units = CAUSAL ? (p.n_tiles + 1) / 2 : p.n_tiles;
        p.total_tiles = heads * n_units;
        p.tiles_per_xcd = (p.total_tiles + 7) / 8;
    };
    a.ds = nullptr;
    a.ds_pitch = a.ds_rows = 0;
    a.head0 = 0;
    if constexpr (kStored<C, RP, DENSE, CG>) {
        // dkv first, chunk by chunk of heads, leaving dS for dq
        const size_t least = (fb_bwd_workspace_bytes(rows, rowsk, CG, pin.R) + 255) & ~(size_t)255;
        const size_t room = pin.workspace_bytes > least ? pin.workspace_bytes - least : 0;
        const int chunk = DENSE ? (dense_stored_pays(all_heads, pin.N, pin.M, C) ? all_heads : 0) : stored_heads(all_heads, pin.N, pin.M, CAUSAL, room);
        if (chunk > 0) {
            constexpr size_t lds_load = (size_t)kSlotsLd<C, RP, LIMB, CG> * kSlotBytesLd<C, RP, LIMB, CG>;
            static_assert(kSlotsLd<C, RP, LIMB, CG> >= 4 && lds_load >= K::kEpiLds, "ring and epilogue");
            auto kst = bwd_main_kernel<C, RP, CAUSAL, true, DENSE, LIMB, CG, STORE>;
            auto kld = bwd_main_kernel<C, RP, CAUSAL, false, DENSE, LIMB, CG, LOAD>;
            static FbLdsOnce once_st, once_ld;
            if (!fb_raise_lds_limit((const void*)kst, lds_dkv, once_st) || !fb_raise_lds_limit((const void*)kld, lds_load, once_ld)) return 1;
            a.ds = (bf16_t*)(ws + least);
            a.ds_pitch = (unsigned)((p.N + 127) / 128 * 128);
            a.ds_rows = (unsigned)((p.M + 127) / 128 * 128);
            if (DENSE && pow2 && !K::FOLD) {      // bf16(k scale) = k scale: the key rows take it, once a wave, and q is read in place
                a.aq.main = (const bf16_t*)pin.q;
                a.q_out = nullptr;
                a.k_mul = a.dkv_mul = pin.scale;
            }
            hipLaunchKernelGGL((bwd_rows_kernel<C>), dim3((unsigned)((rows * 2 + 255) / 256)), dim3(256), 0, stream, pin, a.vec, a.q_out,
                               a.q_mul, rows);
            a.q_out = nullptr;
            for (a.head0 = 0; a.head0 < all_heads; a.head0 += chunk) {
                const int n = all_heads - a.head0 < chunk ? all_heads - a.head0 : chunk;
                set_tiles(p, p.M, n);
                hipLaunchKernelGGL(kst, dim3(8 * p.tiles_per_xcd), dim3(kThreads), lds_dkv, stream, p, a);
                set_tiles(p, p.N, n, kWavesLd * 32);
                hipLaunchKernelGGL(kld, dim3(8 * p.tiles_per_xcd), dim3(kWavesLd * 64), lds_load, stream, p, a);
                if (hipGetLastError() != hipSuccess) return 1;
            }
            return 0;
        }
    }
    // dq first: it also leaves (lse log2 e, D) of every query row for the dkv kernel
    set_tiles(p, p.N, all_heads);
    hipLaunchKernelGGL(kdq, dim3(8 * p.tiles_per_xcd), dim3(kThreads), lds_dq, stream, p, a);
    if (hipGetLastError() != hipSuccess) return 1;
    set_tiles(p, p.M, all_heads);
    hipLaunchKernelGGL(kdkv, dim3(8 * p.tiles_per_xcd), dim3(kThreads), lds_dkv, stream, p, a);
    return hipGetLastError() == hipSuccess ? 0 : 1;
}

template <int C, int CG, int RP, bool LIMB = false>
int dispatch_causal(const BwdParams& p, hipStream_t stream) {
    return p.causal ? launch<C, RP, true, false, LIMB, CG>(p, stream) : launch<C, RP, false, false, LIMB, CG>(p, stream);
}

template <int C, int CG>
int dispatch_rp(const BwdParams& p, int rp, hipStream_t stream) {
    if (p.phi_f32 && rp > 32) return rp <= 64 ? dispatch_causal<C, CG, 64, true>(p, stream) : -1;     // DL
    if constexpr (score_log2e(CG, true)) {      // FOLD
        if (p.phi_f32 && rp == 16) return dispatch_causal<C, CG, 16, true>(p, stream);
        if (p.phi_f32 && rp == 32) return dispatch_causal<C, CG, 32, true>(p, stream);
    }
    switch (rp) {
        case 0: return dispatch_causal<C, CG, 0>(p, stream);
        case 16: return dispatch_causal<C, CG, 16>(p, stream);
        case 32: return dispatch_causal<C, CG, 32>(p, stream);
        case 48: return dispatch_causal<C, CG, 48>(p, stream);
        case 64: return dispatch_causal<C, CG, 64>(p, stream);
        default: break;
    }
    // wider rows: the C (R - 1) extra channels of the multiplicative form (bf16 columns)
    if constexpr (C <= 64) {
        if (p.phi_f32) return -1;
        if (rp == 96) return dispatch_causal<C, CG, 96>(p, stream);
        if (rp == 128) return dispatch_causal<C, CG, 128>(p, stream);
    }
    return -1;
}

template <int C, int CG>
int dispatch_dense(const BwdParams& p, hipStream_t stream) {
    return p.causal ? launch<C, 0, true, true, false, CG>(p, stream) : launch<C, 0, false, true, false, CG>(p, stream);
}

}  // namespace

size_t fb_bwd_workspace_bytes(long long rows_q, long long rows_k, int C, int R) {
    // R alone does not say whether the factors are fp32 (6 R columns): size for the widest rows.
    // Head dimension 16 runs on 32-channel operand rows and adds widened copies of v and dO.
    const int w = (C == 16 ? 32 : C) + (R > 64 ? 128 : (R > 0 ? 64 : 0)) + (C == 16 ? 32 : 0);
    return (((size_t)rows_q * 8 + 15) & ~(size_t)15) + (size_t)(rows_q + rows_k) * w * 2;
}

size_t fb_bwd_stored_bytes(long long heads, int N, int M, int C, bool causal) {
    const int chunk = C != 128 ? 0 : stored_heads(heads, N, M, causal, kMaxStored);
    return chunk > 0 ? 256 + (size_t)chunk * ds_head_bytes(N, M) : 0;
}

int fb_launch_bwd_dense_bf16(const BwdParams& p, int C, hipStream_t stream) {
    switch (C) {
        case 16: return dispatch_dense<32, 16>(p, stream);
        case 32: return dispatch_dense<32, 32>(p, stream);
        case 64: return dispatch_dense<64, 64>(p, stream);
        case 128: return dispatch_dense<128, 128>(p, stream);
        default: return -1;
    }
}

int fb_launch_bwd_bf16(const BwdParams& p, int C, int rp, hipStream_t stream) {
    switch (C) {
        case 16: return dispatch_rp<32, 16>(p, rp, stream);
        case 32: return dispatch_rp<32, 32>(p, rp, stream);
        case 64: return dispatch_rp<64, 64>(p, rp, stream);
        case 128: return dispatch_rp<128, 128>(p, rp, stream);
        default: return -1;
    }
}
