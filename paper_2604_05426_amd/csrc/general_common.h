// Device helpers of the general kernels (fp32, and bf16 with rows that start at any element).
#pragma once

#include "mfma_common.h"

namespace mlora {

template <typename T> constexpr int kEpc = 16 / (int)sizeof(T);     // elements of a 16-byte piece

// 16 bytes from any element boundary; the first `valid` elements are read, the rest are zero
template <typename T> __device__ __forceinline__ uint4 load16(const T* p, int valid) {
    uint4 v = zero4();
    if (valid >= kEpc<T>) {
        __builtin_memcpy(&v, p, 16);
    } else if (valid > 0) {
        uint32_t w[4] = {0u, 0u, 0u, 0u};
        T o[kEpc<T>];
#pragma unroll
        for (int e = 0; e < kEpc<T>; ++e) o[e] = p[min(e, valid - 1)];      // all in flight together
#pragma unroll
        for (int e = 0; e < kEpc<T>; ++e) {
            if constexpr (sizeof(T) == 4) w[e] = e < valid ? __float_as_uint(o[e]) : 0u;
            else w[e >> 1] |= e < valid ? (uint32_t)o[e] << ((e & 1) * 16) : 0u;
        }
        v = make_uint4(w[0], w[1], w[2], w[3]);
    }
    return v;
}

template <typename T> __device__ __forceinline__ float to_f32(T v) {
    if constexpr (sizeof(T) == 4) return v; else return bf2f(v);
}
template <typename T> __device__ __forceinline__ T from_f32(float v) {
    if constexpr (sizeof(T) == 4) return v; else return f2bf(v);
}

// One lane's share of a 16 x 16 block product over 16 (fp32) or 32 (bf16) contraction elements: 16 bytes per operand.  bf16: the
// eight elements 8 g .. 8 g + 7 of row / column l % 16, g = l / 16; fp32: the elements 4 g .. 4 g + 3, multiplied in four steps
// (step j takes element 4 g + j of every g: the order inside the sum is free as long as both operands agree).
template <typename T> __device__ __forceinline__ f32x4 block_mma(uint4 a, uint4 b, f32x4 c) {
    if constexpr (sizeof(T) == 4) {
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
        return c;
    } else {
        return mfma16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c);
    }
}
template <typename T> constexpr int kBlockK = sizeof(T) == 4 ? 16 : 32;   // contraction of one block_mma

// Four adjacent elements of a row whose columns are spread over four blocks (block x takes the columns 4 l + x).  `whole`
// (uniform): all four are inside the row; else each is clamped to the last of `valid` (>= 1) by itself.
template <typename T> using quad_t = uint32_t __attribute__((ext_vector_type(sizeof(T) == 4 ? 4 : 2)));
template <typename T> __device__ __forceinline__ quad_t<T> load_quad(const T* p, bool whole, int valid) {
    quad_t<T> v;
    if (whole) {
        __builtin_memcpy(&v, p, sizeof(v));
    } else {
        T o[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) o[c] = p[min(c, valid - 1)];
        __builtin_memcpy(&v, o, sizeof(v));
    }
    return v;
}
constexpr int kQuadRows32 = 4, kQuadRows16 = 8;
template <typename T> constexpr int kQuadRows = sizeof(T) == 4 ? kQuadRows32 : kQuadRows16;   // rows (contraction) per lane and piece
// column x of a lane's quads as MFMA operand bytes
template <typename T> __device__ __forceinline__ uint4 quad_column(const quad_t<T> (&q)[kQuadRows<T>], int x) {
    uint32_t w[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        if constexpr (sizeof(T) == 4) w[p] = q[p][x];
        else w[p] = __builtin_amdgcn_perm(q[2 * p + 1][x >> 1], q[2 * p][x >> 1], (x & 1) ? 0x07060302u : 0x05040100u);
    }
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// the 16 bytes a lane supplies when its elements lie `ld` apart: elements k .. of a column at p
template <typename T> __device__ __forceinline__ uint4 gather16(const T* p, int64_t ld, int valid) {
    uint32_t w[4] = {0u, 0u, 0u, 0u};
    if (valid <= 0) return zero4();
    T o[kEpc<T>];
#pragma unroll
    for (int e = 0; e < kEpc<T>; ++e) o[e] = p[min(e, valid - 1) * ld];
#pragma unroll
    for (int e = 0; e < kEpc<T>; ++e) {
        if constexpr (sizeof(T) == 4) w[e] = e < valid ? __float_as_uint(o[e]) : 0u;
        else w[e >> 1] |= e < valid ? (uint32_t)o[e] << ((e & 1) * 16) : 0u;
    }
    return make_uint4(w[0], w[1], w[2], w[3]);
}

}  // namespace mlora
