// Internal launchers (one per kernel family); defined in the matching .hip file.
// Each returns 0 on success, 1 when the HIP runtime rejected the launch, -1 when the
// requested shape has no instantiation.
#ifndef FB_LAUNCH_H_
#define FB_LAUNCH_H_

#include <hip/hip_runtime.h>

#include <atomic>

#include "fb_params.h"

int fb_launch_fwd_f32(const FwdParams& p, int C, bool dense, hipStream_t stream);
int fb_launch_fwd_bf16(const FwdParams& p, int C, int rp, bool dense, int qb, hipStream_t stream);
// ALiBi factors generated in the kernel from p.slopes (p.phi_q / p.phi_k unused); qb = 1 or 2.
int fb_launch_fwd_bf16_alibi(const FwdParams& p, int C, int qb, hipStream_t stream);
// Few queries against many keys (no mask).  fb_few_queries: whether that kernel takes the call, with scratch for the
// splits or without; ws: device scratch of fb_few_workspace_bytes(B*H, N, M, C) bytes for the partial results of a head's
// splits, or NULL (no splits).
bool fb_few_queries(long long BH, int N, int M, int C, int R, bool phi_f32, bool scratch);
size_t fb_few_workspace_bytes(long long BH, int N, int M, int C);
int fb_launch_fwd_bf16_few(const FwdParams& p, int C, void* ws, hipStream_t stream);
// Short sequences on the 32-channel tiles (N = M): a head's keys and values in LDS whole.  fb_short_fwd: whether that
// kernel takes the call.
bool fb_short_fwd(const FwdParams& p, int C, int rp);
int fb_launch_fwd_bf16_short(const FwdParams& p, int C, int rp, hipStream_t stream);
// p.workspace points at fb_bwd_workspace_bytes(B*H*N, B*H*M, C, R) bytes of device scratch.
int fb_launch_bwd_bf16(const BwdParams& p, int C, int rp, hipStream_t stream);
// Short key sequences on the 32-channel tiles: one kernel, no workspace.  fb_short_bwd: whether it takes the call.
bool fb_short_bwd(const BwdParams& p, int C, int rp);
int fb_launch_bwd_bf16_short(const BwdParams& p, int C, int rp, hipStream_t stream);
size_t fb_bwd_workspace_bytes(long long rows_q, long long rows_k, int C, int R);
// Room behind that size (from the next multiple of 256 bytes on) with which the dq kernel takes dS from the dkv kernel,
// 0: no use for it.  The launch decides by the same rule from p.workspace_bytes.
size_t fb_bwd_stored_bytes(long long heads, int N, int M, int C, bool causal);
// fp32 tensors and fp32 factors: p.workspace holds one float per query row (a prefix of the size above) and, where
// p.workspace_bytes allows it (fb_bwd_f32_workspace_bytes; 0: no use for more), dS of some or all heads behind them.
size_t fb_bwd_f32_workspace_bytes(long long heads, int N, int M, int C, bool causal);
int fb_launch_bwd_f32(const BwdParams& p, int C, hipStream_t stream);
int fb_launch_bwd_dense_f32(const BwdParams& p, int C, hipStream_t stream);
// Dense-bias backward (p.bias, p.dbias, p.bias_bstride set; p.R = 0; workspace as above with R = 0).
int fb_launch_bwd_dense_bf16(const BwdParams& p, int C, hipStream_t stream);

// Multiplicative bias pre-pass: head[row][C] = x * phi[:, 0] * mul, rest[row][C (R-1)] = the other
// repeats, bf16, for the B * rows_per_batch rows of x (rows_per_batch = H * sequence length);
// phi is [Bp, rows_per_batch, R] with phi_bstride elements between batch items (0 when shared).
int fb_launch_mulbias_prep(const void* x, const void* phi, void* head, void* rest, int B, long long rows_per_batch,
                           int C, int R, int phi_f32, long long phi_bstride, float mul, hipStream_t stream);

// Multiplicative bias backward fold: dx[row][C] = mul * sum_r phi_r g_r, dphi[row][R] = mul * sum_c x_c g_r,c
// from g_head [rows][C], g_rest [rows][C (R-1)] (float gradients of the reweighted repeats); dphi is per batch element.
int fb_launch_mulbias_fold(const void* x, const void* phi, const void* g_head, const void* g_rest, void* dx,
                           void* dphi, int B, long long rows_per_batch, int C, int R, int phi_f32,
                           long long phi_bstride, float mul, hipStream_t stream);

// d0[i] = sum_b s0[b * n0 + i] for i < n0, and the same for (s1, d1, n1); n1 = 0: one tensor only.
int fb_launch_fold_batch(const void* s0, void* d0, long long n0, const void* s1, void* d1, long long n1, int B, bool f32,
                         hipStream_t stream);

// A kernel's dynamic-LDS limit is an attribute of the (kernel, device) pair: raise it on the
// first launch on each device.  Racing first launches all set the same value; the flag is
// published only after the attribute call has returned.
constexpr int kFbMaxDevices = 64;
struct FbLdsOnce { std::atomic<bool> done[kFbMaxDevices] = {}; };
inline bool fb_raise_lds_limit(const void* kern, size_t bytes, FbLdsOnce& once) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    const bool tracked = dev >= 0 && dev < kFbMaxDevices;
    if (tracked && once.done[dev].load(std::memory_order_acquire)) return true;
    if (hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess) return false;
    if (tracked) once.done[dev].store(true, std::memory_order_release);
    return true;
}

// Heads dealt to one workgroup a CU, head after head: how many the busiest CU gets, and how much of that all of them get.
struct FbHeadRounds {
    long long rounds;
    double fill;
};
inline FbHeadRounds fb_head_rounds(long long heads, int cus) {
    const long long rounds = (heads + cus - 1) / cus;
    return {rounds, (double)heads / ((double)rounds * cus)};
}

// Compute units of the current device (0 on failure), asked once per device.
inline int fb_cu_count() {
    static std::atomic<int> known[kFbMaxDevices] = {};
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    const bool tracked = dev >= 0 && dev < kFbMaxDevices;
    if (tracked && (n = known[dev].load(std::memory_order_relaxed)) > 0) return n;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (tracked) known[dev].store(n, std::memory_order_relaxed);
    return n;
}

#endif
