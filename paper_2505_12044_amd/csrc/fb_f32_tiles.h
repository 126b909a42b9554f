// Building blocks of the fp32 kernels: the fp32 matrix instruction, operand rows read straight from
// global memory in its layouts, and the choice of how many waves share a tile.
//
// v_mfma_f32_32x32x2_f32, D[32x32] += A[32x2] B[2x32], full fp32 products and sums.  Lane l, hf = l / 32:
//   A: row l % 32, k-slot hf       B: column l % 32, k-slot hf
//   D: column l % 32, rows 8*(r/4) + 4*hf + (r%4) for register r = 0..15
// It runs at 256 flop per CU and cycle, twice what scalar v_fma_f32 reaches, and one instruction holds the
// matrix pipe for 64 cycles, so a wave can feed its operands from the vector cache without an LDS stage:
// per 32 x 32 block and contraction it reads 4 KB per 32 columns against 1024 pipe cycles.
#ifndef FB_F32_TILES_H_
#define FB_F32_TILES_H_

#include "fb_device.h"

FB_DEV f32x16 mfma32f(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

// A lane-side row [x | phi | 0] of one query or key, chunk i (columns 8i + 4hf .. + 3).
template <int C>
FB_DEV f32x4 own_chunk(const float* x, const float* phi, int R, int i, int hf) {
    if (8 * i < C) return *(const f32x4*)(x + 8 * i + 4 * hf);
    const int c = 8 * i - C + 4 * hf;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < 4; e++)
        if (c + e < R) v[e] = phi[c + e];
    return v;
}

// A streamed array as a raw buffer of `bytes` bytes: reads past its end return zero, so rows behind the
// sequence end need no clamp, and a row operand is one address register plus immediates.
typedef __amdgpu_buffer_rsrc_t f32_buf;
FB_DEV f32_buf make_buf(const float* ptr, size_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)ptr, 0, (int)(unsigned)bytes, 0x00020000);
}
FB_DEV float buf_f32(f32_buf b, unsigned off) {
    return __builtin_bit_cast(float, (unsigned)__builtin_amdgcn_raw_buffer_load_b32(b, (int)off, 0, 0));
}
FB_DEV f32x4 buf_f32x4(f32_buf b, unsigned off) {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(b, (int)off, 0, 0));
}

// Streamed operand rows [x | phi | 0].
struct F32Rows {
    f32_buf x, phi;
    int R;
};

// Chunk i of streamed row `row` (columns 8i + 4hf .. + 3): the row operand of four k-steps.
template <int C>
FB_DEV f32x4 row_chunk(const F32Rows& s, unsigned row, int i, int hf) {
    if (8 * i < C) return buf_f32x4(s.x, row * (C * 4u) + 16u * hf + 32u * i);
    const int c = 8 * i - C + 4 * hf;
    f32x4 v;
#pragma unroll
    for (int e = 0; e < 4; e++) {
        const float t = buf_f32(s.phi, (row * (unsigned)s.R + (unsigned)c) * 4u + 4u * e);
        v[e] = c + e < s.R ? t : 0.f;      // the columns past R belong to the next row
    }
    return v;
}

// Row that accumulator register r of this half stands for inside a 32-row block.
FB_DEV int acc_row(int r, int hf) { return 8 * (r / 4) + 4 * hf + (r % 4); }

// Waves that share one 32-row tile, each taking every KW-th block of the other side (a power of two).
// One wave per tile where the tiles alone give every SIMD its two waves; else the streamed side is
// split until they do, or until a wave has a single block left.
inline int f32_split(long long tiles, int blocks, int max_kw) {
    int kw = 1;
    while (kw < max_kw && tiles * kw < 2048 && 2 * kw <= blocks) kw *= 2;
    return kw;
}

#endif
