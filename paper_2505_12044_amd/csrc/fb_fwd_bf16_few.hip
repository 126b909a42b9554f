// bf16 forward for few queries against many keys (decode: the new tokens of cached sequences), gfx950.
//
// Bound by memory: K, V and phi_k are read once and each key meets at most 8 queries, so the work per byte is
// far below what a matrix tile needs and the 128-row tiles of fwd_bf16_kernel leave three of four waves and,
// with fewer heads than CUs, most of the chip idle.  Here the keys of one (b, h) are split over the grid and over
// the waves of a workgroup, and everything is fp32 vector arithmetic on rows read straight from memory:
//   a key's C channels lie in C / 8 adjacent lanes (16 bytes each, whole rows per load instruction);
//   a group of C / 8 lanes walks its own keys with its own online softmax (m, l, o), U keys at a time with
//   all 2 U row loads in flight, and needs no exchange but the sum over its lanes of the score (DPP adds);
//   the groups of a wave, then the waves of a workgroup, are merged once at the end; the splits of a (b, h) leave
//   (m, l, o) in the workspace and a second kernel merges them (in a fixed order).
// B 8, H 16, N 1, M 4096, C 128, R 2, inputs from memory: 127 -> 51 us a call, 5.3 TB/s of K and V (a large reduction
// reads at 6.1); 43 us where they lie in the Infinity Cache.
// The factor product is a chain of fp32 multiply-adds on the stored factors (no limbs).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "fb_device.h"
#include "fb_launch.h"
#include "fb_params.h"

namespace {

constexpr int kFewWaves = 4;
constexpr int kFewThreads = kFewWaves * 64;

template <int C, int NQ>
struct FewCfg {
    static constexpr int LPK = C / 8;                 // lanes per key
    static constexpr int KPC = 64 / LPK;              // keys per load instruction of a wave
    static constexpr int U = NQ <= 2 ? 8 : 4;         // keys per group and step (registers: 8 U of rows, U NQ scores)
    static constexpr int KI = U * KPC;                // keys per wave and step
    static constexpr int UNIT = kFewWaves * KI;       // keys per workgroup and step
};

// sum over the LPK lanes of a group, the same value in all of them
template <int LPK>
FB_DEV float group_sum(float x) {
    auto dpp = [](float v, auto ctrl) __attribute__((always_inline)) {
        return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    x += dpp(x, std::integral_constant<int, 0xB1>{});                        // lane ^ 1
    if constexpr (LPK >= 4) x += dpp(x, std::integral_constant<int, 0x4E>{});    // lane ^ 2
    if constexpr (LPK >= 8) x += dpp(x, std::integral_constant<int, 0x141>{});   // lane 7 - i of eight
    if constexpr (LPK >= 16) x += dpp(x, std::integral_constant<int, 0x140>{});  // lane 15 - i of sixteen
    return x;
}

FB_DEV void unpack8(float (&x)[8], const u32x4& r) {
#pragma unroll
    for (int i = 0; i < 4; i++) {
        x[2 * i] = __builtin_bit_cast(float, r[i] << 16);
        x[2 * i + 1] = __builtin_bit_cast(float, r[i] & 0xffff0000u);
    }
}

// RT: number of factors when known at compile time (0, 2), -1: p.R of them.
template <int C, int NQ, int RT, bool PF32>
__global__ __launch_bounds__(kFewThreads, 2) void fwd_few_kernel(FwdParams p, int n_split, int units_per_split,
                                                                 float* __restrict__ part_o, float2* __restrict__ part_ml) {
    using K = FewCfg<C, NQ>;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane % K::LPK, g = lane / K::LPK;
    const int bh = blockIdx.x / n_split, split = blockIdx.x - bh * n_split;
    const int b = bh / p.H, h = bh - b * p.H;
    const int N = p.N, M = p.M, R = RT >= 0 ? RT : p.R;

    const bf16_t* kg = (const bf16_t*)p.k + (size_t)bh * M * C + c * 8;
    const bf16_t* vg = (const bf16_t*)p.v + (size_t)bh * M * C + c * 8;
    using PT = std::conditional_t<PF32, float, bf16_t>;
    const PT* pqg = (const PT*)p.phi_q + (size_t)b * p.phi_bstride + (size_t)h * N * R;
    const PT* pkg = (const PT*)p.phi_k + (size_t)b * p.phik_bstride + (size_t)h * M * R;

    // The rounding of the query that the backward repeats
    constexpr bool RAWQ = score_raw_q(C, !PF32), LOG2E = score_log2e(C, PF32 && RT != 0);
    const float qscale = LOG2E ? p.scale * kLog2e : p.scale;
    u32x4 q[NQ];
    const PT* pq[NQ];                    // wave-uniform rows; queries past N repeat the last one and are not stored
#pragma unroll
    for (int n = 0; n < NQ; n++) {
        const int qi = min(n, N - 1);
        q[n] = *(const u32x4*)((const bf16_t*)p.q + ((size_t)bh * N + qi) * C + c * 8);
        if (!RAWQ) {
            bf16x8 x = as_bf16x8(q[n]);
#pragma unroll
            for (int e = 0; e < 8; e++) x[e] = (bf16_t)((float)x[e] * qscale);
            q[n] = as_uint4(x);
        }
        pq[n] = pqg + (size_t)qi * R;
    }
    float m[NQ], l[NQ], o[NQ][8];
#pragma unroll
    for (int n = 0; n < NQ; n++) {
        m[n] = -1e30f;
        l[n] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; e++) o[n][e] = 0.f;
    }
    const float emul = RAWQ ? p.scale * kLog2e : (LOG2E ? 1.f : kLog2e);

    const int u_begin = split * units_per_split;
    const int u_end = min(u_begin + units_per_split, (M + K::UNIT - 1) / K::UNIT);
    for (int unit = u_begin; unit < u_end; unit++) {
        const int k0 = unit * K::UNIT + wave * K::KI;          // wave-uniform
        if (k0 >= M) break;
        u32x4 kr[K::U], vr[K::U];
        int key[K::U];
#pragma unroll
        for (int u = 0; u < K::U; u++) key[u] = min(k0 + u * K::KPC + g, M - 1);
#pragma unroll
        for (int u = 0; u < K::U; u++) kr[u] = *(const u32x4*)(kg + (size_t)key[u] * C);
        float s[K::U][NQ];
#pragma unroll
        for (int u = 0; u < K::U; u++)
#pragma unroll
            for (int n = 0; n < NQ; n++) s[u][n] = 0.f;
        auto add_factor = [&](int r) __attribute__((always_inline)) {
            float pk[K::U];
#pragma unroll
            for (int u = 0; u < K::U; u++) pk[u] = (float)pkg[(size_t)key[u] * R + r];
#pragma unroll
            for (int n = 0; n < NQ; n++) {
                const float a = (float)pq[n][r];
#pragma unroll
                for (int u = 0; u < K::U; u++) s[u][n] = fmaf(a, pk[u], s[u][n]);
            }
        };
        if constexpr (RT >= 0) {
#pragma unroll
            for (int r = 0; r < RT; r++) add_factor(r);
        } else {
            int r = 0;
            for (; r + 4 <= R; r += 4) {
                add_factor(r); add_factor(r + 1); add_factor(r + 2); add_factor(r + 3);
            }
            for (; r < R; r++) add_factor(r);
        }
#pragma unroll
        for (int u = 0; u < K::U; u++) vr[u] = *(const u32x4*)(vg + (size_t)key[u] * C);
        // scores in units of log 2
#pragma unroll
        for (int u = 0; u < K::U; u++)
#pragma unroll
            for (int n = 0; n < NQ; n++) {
                float d = 0.f;
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const unsigned kw = kr[u][i], qw = q[n][i];     // (a bit cast of the element itself reads element 0)
                    d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, kw), __builtin_bit_cast(bf16x2, qw), d, false);
                }
                s[u][n] = fmaf(group_sum<K::LPK>(d), emul, s[u][n] * kLog2e);
            }
        if (k0 + K::KI > M) {            // sequence end: the repeats of the last key do not count
#pragma unroll
            for (int u = 0; u < K::U; u++)
                if (k0 + u * K::KPC + g >= M) {
                    vr[u] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
                    for (int n = 0; n < NQ; n++) s[u][n] = -INFINITY;
                }
        }
#pragma unroll
        for (int n = 0; n < NQ; n++) {
            float mx = m[n];
#pragma unroll
            for (int u = 0; u < K::U; u++) mx = fmaxf(mx, s[u][n]);
            const float alpha = fast_exp2(m[n] - mx);
            m[n] = mx;
            l[n] *= alpha;
#pragma unroll
            for (int e = 0; e < 8; e++) o[n][e] *= alpha;
#pragma unroll
            for (int u = 0; u < K::U; u++) {
                s[u][n] = fast_exp2(s[u][n] - mx);
                l[n] += s[u][n];
            }
        }
#pragma unroll
        for (int u = 0; u < K::U; u++) {
            float x[8];
            unpack8(x, vr[u]);
#pragma unroll
            for (int n = 0; n < NQ; n++)
#pragma unroll
                for (int e = 0; e < 8; e++) o[n][e] = fmaf(s[u][n], x[e], o[n][e]);
        }
    }

    // ---- the groups of the wave ----
#pragma unroll
    for (int n = 0; n < NQ; n++) {
        float mx = m[n];
#pragma unroll
        for (int d = K::LPK; d < 64; d *= 2) mx = fmaxf(mx, __shfl_xor(mx, d));
        const float alpha = fast_exp2(m[n] - mx);
        m[n] = mx;
        l[n] *= alpha;
#pragma unroll
        for (int e = 0; e < 8; e++) o[n][e] *= alpha;
#pragma unroll
        for (int d = K::LPK; d < 64; d *= 2) {
            l[n] += __shfl_xor(l[n], d);
#pragma unroll
            for (int e = 0; e < 8; e++) o[n][e] += __shfl_xor(o[n][e], d);
        }
    }
    // ---- the waves of the workgroup ----
    __shared__ float sm_o[kFewWaves][NQ][C];
    __shared__ float sm_m[kFewWaves][NQ], sm_l[kFewWaves][NQ];
    if (g == 0) {
#pragma unroll
        for (int n = 0; n < NQ; n++)
#pragma unroll
            for (int e = 0; e < 8; e++) sm_o[wave][n][c * 8 + e] = o[n][e];
    }
    if (lane == 0) {
#pragma unroll
        for (int n = 0; n < NQ; n++) { sm_m[wave][n] = m[n]; sm_l[wave][n] = l[n]; }
    }
    __syncthreads();
    for (int i = tid; i < NQ * C; i += kFewThreads) {
        const int n = i / C, ch = i % C;
        if (n >= N) break;
        float mx = sm_m[0][n];
#pragma unroll
        for (int w = 1; w < kFewWaves; w++) mx = fmaxf(mx, sm_m[w][n]);
        float lt = 0.f, ot = 0.f;
#pragma unroll
        for (int w = 0; w < kFewWaves; w++) {
            const float a = fast_exp2(sm_m[w][n] - mx);
            lt = fmaf(a, sm_l[w][n], lt);
            ot = fmaf(a, sm_o[w][n][ch], ot);
        }
        if (n_split == 1) {
            const size_t row = (size_t)bh * N + n;
            ((bf16_t*)p.out)[row * C + ch] = (bf16_t)(ot / lt);
            if (ch == 0) p.lse[row] = (mx + __log2f(lt)) * kLn2;
        } else {
            const size_t row = ((size_t)bh * n_split + split) * N + n;
            part_o[row * C + ch] = ot;
            if (ch == 0) part_ml[row] = make_float2(mx, lt);
        }
    }
}

// Merges the splits: one thread per four channels of a query row.
template <int C>
__global__ __launch_bounds__(256) void few_merge_kernel(const float* __restrict__ part_o, const float2* __restrict__ part_ml,
                                                        bf16_t* __restrict__ out, float* __restrict__ lse, int N, int n_split, int rows) {
    const int gid = blockIdx.x * 256 + threadIdx.x;
    const int row = gid / (C / 4), c4 = gid % (C / 4);
    if (row >= rows) return;
    const int bh = row / N, n = row - bh * N;
    const size_t r0 = (size_t)bh * n_split * N + n;
    float mx = -1e30f;
    for (int s = 0; s < n_split; s++) mx = fmaxf(mx, part_ml[r0 + (size_t)s * N].x);
    float lt = 0.f;
    f32x4 ot = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int s = 0; s < n_split; s++) {
        const float2 ml = part_ml[r0 + (size_t)s * N];
        const f32x4 x = *(const f32x4*)(part_o + (r0 + (size_t)s * N) * C + c4 * 4);
        const float a = fast_exp2(ml.x - mx);
        lt = fmaf(a, ml.y, lt);
#pragma unroll
        for (int e = 0; e < 4; e++) ot[e] = fmaf(a, x[e], ot[e]);
    }
    const float inv = 1.f / lt;
    bf16x4 o4;
#pragma unroll
    for (int e = 0; e < 4; e++) o4[e] = (bf16_t)(ot[e] * inv);
    *(u32x2*)(out + (size_t)row * C + c4 * 4) = __builtin_bit_cast(u32x2, o4);
    if (c4 == 0) lse[row] = (mx + __log2f(lt)) * kLn2;
}

struct FewPlan { int nq, n_split, units_per_split; };

// Splits: enough workgroups to keep the memory system busy (kFewGroups of four waves).  us with 256, 512, 1024, 2048, inputs
// from memory, R 2: 128 heads, N 1, M 4096, C 128 48, 50, 51, 53; 16 heads, N 8, M 16384, C 128 53, 49, 61, 84; 128 heads,
// N 8, M 2048, C 64 29, 26, 32, 32 (a split's merge and prologue weigh more with more queries).
// A workgroup walks at least kFewSteps steps, and heads of fewer than eight steps are not split: the merge is a
// second launch (3 us of the GPU, as much of the host), which M = 300 keys (5 us in one workgroup) do not repay.
constexpr int kFewGroups = 512;
constexpr int kFewSteps = 2;

FewPlan few_plan(long long BH, int N, int M, int C, bool scratch) {
    FewPlan f;
    f.nq = N == 1 ? 1 : (N == 2 ? 2 : (N <= 4 ? 4 : 8));
    const int unit = kFewWaves * (f.nq <= 2 ? 8 : 4) * (512 / C);       // FewCfg::UNIT
    const int units = (M + unit - 1) / unit;
    long long want = (kFewGroups + BH - 1) / BH;
    const int most = units < 8 || !scratch ? 1 : units / kFewSteps;
    if (want > most) want = most;
    f.units_per_split = (int)((units + want - 1) / want);
    f.n_split = (units + f.units_per_split - 1) / f.units_per_split;
    return f;
}

template <int C, int NQ, int RT, bool PF32>
int launch_few(const FwdParams& p, const FewPlan& f, void* ws, hipStream_t stream) {
    static_assert(FewCfg<C, NQ>::UNIT == kFewWaves * (NQ <= 2 ? 8 : 4) * (512 / C), "few_plan");
    const long long blocks = (long long)p.B * p.H * f.n_split;
    if (blocks >= (1LL << 31)) return -1;
    const size_t rows = (size_t)p.B * p.H * f.n_split * p.N;
    float2* ml = (float2*)((float*)ws + (ws ? rows * C : 0));
    hipLaunchKernelGGL((fwd_few_kernel<C, NQ, RT, PF32>), dim3((unsigned)blocks), dim3(kFewThreads), 0, stream, p, f.n_split,
                       f.units_per_split, (float*)ws, ml);
    if (hipGetLastError() != hipSuccess) return 1;
    if (f.n_split > 1) {
        const int orows = p.B * p.H * p.N;
        const unsigned nb = (unsigned)(((long long)orows * (C / 4) + 255) / 256);
        hipLaunchKernelGGL((few_merge_kernel<C>), dim3(nb), dim3(256), 0, stream, (const float*)ws, ml, (bf16_t*)p.out, p.lse, p.N,
                           f.n_split, orows);
        if (hipGetLastError() != hipSuccess) return 1;
    }
    return 0;
}

template <int C, int NQ>
int few_factors(const FwdParams& p, const FewPlan& f, void* ws, hipStream_t stream) {
    if (p.R == 0) return launch_few<C, NQ, 0, true>(p, f, ws, stream);
    if (p.phi_f32) return p.R == 2 ? launch_few<C, NQ, 2, true>(p, f, ws, stream) : launch_few<C, NQ, -1, true>(p, f, ws, stream);
    return launch_few<C, NQ, -1, false>(p, f, ws, stream);
}

template <int C>
int few_queries(const FwdParams& p, const FewPlan& f, void* ws, hipStream_t stream) {
    switch (f.nq) {
        case 1: return few_factors<C, 1>(p, f, ws, stream);
        case 2: return few_factors<C, 2>(p, f, ws, stream);
        case 4: return few_factors<C, 4>(p, f, ws, stream);
        default: return few_factors<C, 8>(p, f, ws, stream);
    }
}

}  // namespace

// Which calls: the kernel that takes less time by the two estimates below, in ns, fitted to 5629 calls of 1 to 4096
// heads, 16 to 16384 keys, N 1, 2, 4, 8, every head dimension and factor form, with scratch and without.  Chosen by them,
// one call in a hundred is more than 3 % slower than on the tile kernel (worst 1.3x, at 15 us), and the average call is
// within 0.6 % of the faster kernel.  us on the tile kernel / here in one workgroup a head / here with the split:
//   8 heads, M 16384, C 128:   N 1 R 2 355 / 198 / 25;   N 8 R 16 bf16 349 / 1115 / 55
//   8 heads, M 300:            C 16 N 1 R 2 7.1 / 3.7;   C 16 N 8 R 16 bf16 5.9 / 11.5
//   1024 heads, M 2048, C 128: N 1 R 2 187 / 177;   N 8 R 2 191 / 255
namespace {

// A workgroup: prologue and merges (a shuffle per group level and query), then its steps, each with the factor chain.
// Past one round of 320 workgroups the waves that have keys count (the last step of a short sequence leaves some idle).
double few_ns(long long BH, int M, int C, int R, const FewPlan& f) {
    static constexpr double kStep[4] = {1150, 1500, 1250, 1950}, kFactor[4] = {130, 160, 100, 150};
    const int i = f.nq == 1 ? 0 : (f.nq == 2 ? 1 : (f.nq == 4 ? 2 : 3));
    const int levels = C == 16 ? 5 : (C == 32 ? 4 : (C == 64 ? 3 : 2));
    const int wave_keys = (f.nq <= 2 ? 8 : 4) * (512 / C);
    const double fixed = 140.0 * f.nq * levels;
    const double steps = f.units_per_split * (kStep[i] + kFactor[i] * R);
    const int units = (M + kFewWaves * wave_keys - 1) / (kFewWaves * wave_keys);
    const double fill = (double)((M + wave_keys - 1) / wave_keys) / ((double)units * kFewWaves);
    const double one = fixed + steps, busy = (fixed + steps * fill) * (double)BH * f.n_split / 320.0;
    return 1800 + (f.n_split > 1 ? 4000 : 0) + (busy > one ? busy : one);
}

// The tile kernel: a workgroup a head, a prologue and a ring step per 32 keys.  fp32 factors take six columns a rank (one,
// two or three to four k-steps), and bf16 ranks that are no multiple of eight are gathered one by one.
double tile_ns(long long BH, int M, int C, int R, bool phi_f32) {
    const int c = C == 16 ? 0 : (C == 32 ? 1 : (C == 64 ? 2 : 3));
    static constexpr double kBlock[4] = {290, 380, 500, 640};            // ns per 32 keys, no or whole-chunk factors
    static constexpr double kMid[4] = {1.25, 1.25, 1.1, 1.7}, kWide[4] = {1.35, 1.35, 1.3, 2.4};      // fp32, R 3..8, 9..10
    double fixed = c == 3 ? 1000 : 600, step = kBlock[c];
    if (!phi_f32) {
        if ((R & 7) != 0) step *= 1.6;
    } else if (R > 0) {
        fixed += R <= 2 ? 800 : (R <= 8 ? 1700 : 4200);
        if (R > 2) step *= R <= 8 ? kMid[c] : kWide[c];
    }
    const double rounds = (double)BH / (c == 3 ? 300 : 400);
    return 2200 + (fixed + (M + 31) / 32 * step) * (rounds > 1 ? rounds : 1);
}

}  // namespace

bool fb_few_queries(long long BH, int N, int M, int C, int R, bool phi_f32, bool scratch) {
    if (N > 8 || N >= M || R > 16) return false;
    return few_ns(BH, M, C, R, few_plan(BH, N, M, C, scratch)) < tile_ns(BH, M, C, R, phi_f32);
}

size_t fb_few_workspace_bytes(long long BH, int N, int M, int C) {
    const FewPlan f = few_plan(BH, N, M, C, true);
    return f.n_split > 1 ? (size_t)BH * f.n_split * N * (C + 2) * sizeof(float) : 0;
}

int fb_launch_fwd_bf16_few(const FwdParams& p, int C, void* ws, hipStream_t stream) {
    const FewPlan f = few_plan((long long)p.B * p.H, p.N, p.M, C, ws != nullptr);
    switch (C) {
        case 16: return few_queries<16>(p, f, ws, stream);
        case 32: return few_queries<32>(p, f, ws, stream);
        case 64: return few_queries<64>(p, f, ws, stream);
        case 128: return few_queries<128>(p, f, ws, stream);
        default: return -1;
    }
}
