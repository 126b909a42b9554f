// Sum over the batch of the per-batch-element gradients of a tensor that is shared over the batch (factors or
// a dense bias): dst[i] = sum_b src[b * n + i], fp32 sums in a fixed order, one rounding at the end.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "fb_device.h"
#include "fb_launch.h"

namespace {

constexpr int kFoldThreads = 256;

// V consecutive values of type T as floats
template <typename T, int V>
struct Vec {
    T v[V];
};
template <typename T, int V>
FB_DEV void load_vec(float (&x)[V], const T* p) {
    if constexpr (V == 1) {
        x[0] = (float)p[0];
    } else {
        static_assert(sizeof(Vec<T, V>) == 16, "16-byte pieces");
        const Vec<T, V> t = __builtin_bit_cast(Vec<T, V>, *(const u32x4*)p);
#pragma unroll
        for (int e = 0; e < V; e++) x[e] = (float)t.v[e];
    }
}
template <typename T, int V>
FB_DEV void store_vec(T* p, const float (&x)[V]) {
    if constexpr (V == 1) {
        p[0] = (T)x[0];
    } else {
        Vec<T, V> t;
#pragma unroll
        for (int e = 0; e < V; e++) t.v[e] = (T)x[e];
        *(u32x4*)p = __builtin_bit_cast(u32x4, t);
    }
}

// Bound by memory: every source value is read once, in pieces of V values (16 bytes where n allows it).  A
// workgroup covers 256 / G consecutive pieces; G groups of threads share the batch (group g takes elements
// g, g + G, ...) and meet in LDS.  G = 1 where the pieces alone fill the chip, 16 where they do not.  Eight
// loads in flight per thread.
// Training steps with it against torch's sum and conversion per tensor: B 384, H 4, N 384, C 32, R 16 bf16
// 407 -> 368 us (the two sums took 69 us), dense bias B 8, H 12, N 1024, C 64 341 -> 315 us (71 us), relative
// positions B 8, H 12, N 1024, R 32 225 -> 216 us.
// Two tensors (phi_q and phi_k) in one launch: workgroups [0, nb0) belong to the first.  block0: workgroups of the
// launches before this one.
template <typename T, int V, int G>
__global__ __launch_bounds__(kFoldThreads) void fold_batch_kernel(const T* __restrict__ src0, T* __restrict__ dst0, long long n0,
                                                                  const T* __restrict__ src1, T* __restrict__ dst1, long long n1,
                                                                  long long block0, long long nb0, int B) {
    constexpr int P = kFoldThreads / G;        // pieces per workgroup
    const long long block = block0 + blockIdx.x;
    const bool second = block >= nb0;
    const T* const src = second ? src1 : src0;
    T* const dst = second ? dst1 : dst0;
    const long long n = second ? n1 : n0;
    const int piece = threadIdx.x % P, g = threadIdx.x / P;
    const long long i = ((block - (second ? nb0 : 0)) * P + piece) * V;
    float acc[V];
#pragma unroll
    for (int e = 0; e < V; e++) acc[e] = 0.f;
    if (i < n) {                               // V divides n: a piece is wholly inside or outside
        const T* s = src + (long long)g * n + i;
        const long long step = (long long)G * n;
        int b = g;
        // U elements at a time: U loads in flight, summed as a tree
        auto take = [&](auto u_tag) __attribute__((always_inline)) {
            constexpr int U = decltype(u_tag)::value;
            float x[U][V];
#pragma unroll
            for (int u = 0; u < U; u++) load_vec<T, V>(x[u], s + u * step);
            s += U * step;
            b += U * G;
#pragma unroll
            for (int w = 1; w < U; w *= 2)
#pragma unroll
                for (int u = 0; u + w < U; u += 2 * w)
#pragma unroll
                    for (int e = 0; e < V; e++) x[u][e] += x[u + w][e];
#pragma unroll
            for (int e = 0; e < V; e++) acc[e] += x[0][e];
        };
        while (b + 7 * G < B) take(std::integral_constant<int, 8>{});
        if (b + 3 * G < B) take(std::integral_constant<int, 4>{});
        if (b + G < B) take(std::integral_constant<int, 2>{});
        if (b < B) take(std::integral_constant<int, 1>{});
    }
    if constexpr (G > 1) {
        __shared__ float part[G][V][P];
#pragma unroll
        for (int e = 0; e < V; e++) part[g][e][piece] = acc[e];
        __syncthreads();
        if (g != 0) return;
#pragma unroll
        for (int e = 0; e < V; e++) {
            float t = 0.f;
#pragma unroll
            for (int k = 0; k < G; k++) t += part[k][e][piece];
            acc[e] = t;
        }
    }
    if (i < n) store_vec<T, V>(dst + i, acc);
}

template <typename T, int V, int G>
int launch_fold(const void* s0, void* d0, long long n0, const void* s1, void* d1, long long n1, int B, hipStream_t stream) {
    constexpr int P = kFoldThreads / G;
    auto blocks = [](long long n) { return (n / V + P - 1) / P; };
    const long long nb0 = blocks(n0), nb = nb0 + blocks(n1);
    // a launch takes fewer than 2^32 threads: larger tensors (from 2^28 values of an odd length on) in several, each long
    // enough that the gap between them does not show
    constexpr long long kMost = 1LL << 20;
    for (long long block0 = 0; block0 < nb; block0 += kMost) {
        hipLaunchKernelGGL((fold_batch_kernel<T, V, G>), dim3((unsigned)(nb - block0 < kMost ? nb - block0 : kMost)),
                           dim3(kFoldThreads), 0, stream, (const T*)s0, (T*)d0, n0, (const T*)s1, (T*)d1, n1, block0, nb0, B);
        if (hipGetLastError() != hipSuccess) return 1;
    }
    return 0;
}

template <typename T, int V>
int dispatch_split(const void* s0, void* d0, long long n0, const void* s1, void* d1, long long n1, int B, hipStream_t stream) {
    // Threads of the unsplit form against what the chip keeps in flight (256 CUs of 2048 threads).  Measured in
    // the training step: B 8, H 12, N 1024 dense (1.6 M pieces) G = 1; B 384, H 4, N 384, R 16 (2 x 3072
    // pieces) G = 16.
    if (n0 / V + n1 / V >= 256LL * 1024 || B < 4) return launch_fold<T, V, 1>(s0, d0, n0, s1, d1, n1, B, stream);
    return launch_fold<T, V, 16>(s0, d0, n0, s1, d1, n1, B, stream);
}

template <typename T>
int dispatch_vec(const void* s0, void* d0, long long n0, const void* s1, void* d1, long long n1, int B, hipStream_t stream) {
    constexpr int V = 16 / sizeof(T);
    const uintptr_t bits = reinterpret_cast<uintptr_t>(s0) | reinterpret_cast<uintptr_t>(d0) | reinterpret_cast<uintptr_t>(s1) |
                           reinterpret_cast<uintptr_t>(d1);
    // 16-byte pieces need every batch element's row to start on 16 bytes
    if ((bits & 15u) == 0 && n0 % V == 0 && n1 % V == 0) return dispatch_split<T, V>(s0, d0, n0, s1, d1, n1, B, stream);
    return dispatch_split<T, 1>(s0, d0, n0, s1, d1, n1, B, stream);
}

}  // namespace

int fb_launch_fold_batch(const void* s0, void* d0, long long n0, const void* s1, void* d1, long long n1, int B, bool f32,
                         hipStream_t stream) {
    return f32 ? dispatch_vec<float>(s0, d0, n0, s1, d1, n1, B, stream) : dispatch_vec<bf16_t>(s0, d0, n0, s1, d1, n1, B, stream);
}
